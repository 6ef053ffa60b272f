"""Planning a batch of many short reads: the transition constants of one read
(three logarithms and exponentials) are computed while those of others still are.
Host time of a call per read, less that of a call whose reads are empty, against a
C loop on the same processor in which each read's constants wait for the last
one's."""

import ctypes
import subprocess
import time

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth

pytestmark = pytest.mark.gpu

CHAIN = r"""
#include <math.h>
double chain(int n, double *out) {
  double wait = 0.0;
  for (int i = 0; i < n; ++i) {
    const double epk = (70.0 + (i & 7) + wait) / 40.0;
    const double stay = log(1.0 - 1.0 / (epk + 1.0));
    out[i & 63] = log(1.0 - 1e-10 - exp(stay));
    wait = out[i & 63] * 1e-300; /* 0 beside the sum, but it has to be known */
  }
  return wait;
}
"""


def best(fn, reps=40):
    t = np.inf
    for _ in range(reps):
        t0 = time.perf_counter()
        fn()
        t = min(t, time.perf_counter() - t0)
    return t


def test_reads_do_not_wait_for_one_another(tmp_path):
    import torch

    n = 20000
    src, so = tmp_path / "chain.c", tmp_path / "chain.so"
    src.write_text(CHAIN)
    subprocess.check_call(["gcc", "-O2", "-shared", "-fPIC", str(src), "-o", str(so), "-lm"])
    lib = ctypes.CDLL(str(so))
    lib.chain.restype = ctypes.c_double
    buf = (ctypes.c_double * 64)()
    chain = best(lambda: lib.chain(n, buf)) / n

    m = synth.pore_model(6)
    rng = np.random.default_rng(5)
    ne = np.full(n, 72)  # alike, so that sorting them takes what sorting empty ones does

    def batch(empty):
        eo = np.concatenate([[0], np.cumsum(ne)]).astype(np.uint64)
        ko = (np.arange(n + 1) * 40).astype(np.uint64)
        if empty:
            eo[:] = 0
        ev = np.zeros((int(ne.sum()), 3), np.float32)
        ev[:, 0] = rng.normal(90, 12, ev.shape[0])
        rk = rng.integers(0, 4096, n * 40).astype(np.int32)
        one, zero = torch.ones(n, device="cuda"), torch.zeros(n, device="cuda")
        return abea.DeviceBatch(n, torch.from_numpy(ev).cuda(), torch.from_numpy(rk).cuda(), one, zero, eo, ko)

    def host_time(db):
        al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=100)
        dr = abea.DeviceResult.empty(db)
        t = np.inf
        for _ in range(40):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            al.align_device(db, dr)
            t = min(t, time.perf_counter() - t0)
        torch.cuda.synchronize()
        al.close()
        return t / n

    print("gpu: host time of a call, 20000 reads and 20000 empty reads", flush=True)
    full, none = host_time(batch(False)), host_time(batch(True))
    print(f"a read {full * 1e9:.1f} ns, an empty one {none * 1e9:.1f} ns, constants in a chain {chain * 1e9:.1f} ns")
    assert full - none < 0.8 * chain
