"""Events that run through hundreds of tiles: bit for bit against the oracle, and
their samples are read once.  An event's sum is made by the wavefront of the tile it
starts in, a tile in which none starts adds none up."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_detect import compare, gpu_events_device, oracle_events

pytestmark = pytest.mark.gpu

TILE = 1024


def steps(n, at):
    """n samples of small noise whose level rises by 300 at each of `at`."""
    x = 200 + (np.arange(n) % 2)
    for a in at:
        x[a:] += 300
    return x.astype(np.int16)


def raw_batch(signals):
    return synth.make_raw_batch([synth.RawRead(x, np.zeros(0, np.uint32), np.float32(3), np.float32(0.17), np.float32(1),
                                               np.float32(0), np.zeros(0, np.int64)) for x in signals])


def test_long_events(oracle_mod):
    n = 300 * TILE + 77
    b = raw_batch([steps(n, at) for at in ([], [n - 40], [n - 5000], [200 * TILE], [200 * TILE - 1], [150 * TILE + 500],
                                           [60], [1030, 66 * TILE + 3, 131 * TILE, n - 1500])]
                  + [np.full(n, -32768, np.int16), np.full(64 * TILE, 32767, np.int16), np.full(65 * TILE + 1, 9, np.int16)])
    m = synth.pore_model(6)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6)
    for params in (None, (3, 9, 1.4, 9.0)):
        print(f"gpu: long events params={params}", flush=True)
        pa = abea.detect_params(*params) if params else None
        po = oracle_mod.ed_params(params[0], params[2], params[1], params[3]) if params else None
        ev, eo = gpu_events_device(al, b, pa)
        want_ev, want_eo = oracle_events(oracle_mod, b, po)
        compare(f"long events {params}", ev, eo, want_ev, want_eo)
    al.close()


def test_long_events_are_read_once():
    """1024 reads of 117 tiles without a change point against 16: the chain of
    the one wavefront that sums an event is the same, and 245 MB are read once
    in 0.3 ms at 1 TB/s.  Read again by every tile they are 14 GB.  (With 128 tiles a
    read, 32 workgroups, every chain would be on the same one of the eight XCDs.)"""
    import torch

    m = synth.pore_model(6)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6, timing=True)
    n = 116 * TILE + 301

    def event_kernel_ms(reads):
        x = torch.full((reads * n,), 400, dtype=torch.int16, device="cuda")
        d = abea.DeviceRawBatch(reads, x, torch.zeros(reads, device="cuda"), torch.ones(reads, device="cuda"),
                                np.arange(reads + 1, dtype=np.uint64) * np.uint64(n))
        ev = torch.zeros((reads, 3), device="cuda")
        eo = torch.zeros(reads + 1, dtype=torch.int64, device="cuda")
        best = np.inf
        for _ in range(4):
            al.detect_events_device(d, ev, eo)
            torch.cuda.synchronize()
            best = min(best, float(al.detect_timings()[1]))
        assert int(eo[-1]) == reads and bool((ev[:, 2] == n).all())
        return best

    print("gpu: long events, 16 and 1024 reads", flush=True)
    few, many = event_kernel_ms(16), event_kernel_ms(1024)
    print(f"event kernel {few:.3f} ms, {many:.3f} ms")
    al.close()
    assert many < 4 * few + 0.6
