"""Batches of few tiles and many reads, most of them empty: the reads' offsets come
from the block that scans the tiles up to 1024 reads, from a launch of their own
beyond."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_detect import compare, gpu_events_device, oracle_events

pytestmark = pytest.mark.gpu


def mixed(rng, reads, full, n):
    """`reads` reads, `full` of them of n samples, the others empty."""
    has = np.zeros(reads, bool)
    has[rng.permutation(reads)[:full]] = True
    return [np.clip(np.round(rng.normal(500, 60, n if h else 0)), 0, 1000).astype(np.int16) for h in has]


@pytest.mark.parametrize("reads", [255, 256, 257, 1022, 1023, 1024, 1025, 1026, 4000])
def test_offsets(oracle_mod, reads):
    rng = np.random.default_rng(reads)
    b = synth.make_raw_batch([synth.RawRead(x, np.zeros(0, np.uint32), np.float32(3), np.float32(0.17), np.float32(1),
                                            np.float32(0), np.zeros(0, np.int64)) for x in mixed(rng, reads, 250, 2500)])
    m = synth.pore_model(6)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6)
    print(f"gpu: detect {reads} reads, 250 with samples", flush=True)
    ev, eo = gpu_events_device(al, b)
    al.close()
    want_ev, want_eo = oracle_events(oracle_mod, b)
    compare(f"{reads} reads", ev, eo, want_ev, want_eo)


def test_many_empty_reads_are_not_slow():
    """200000 reads of which 1000 hold samples against those 1000: the offsets
    of 200000 reads are 1.6 MB, a few times a small batch's launches; one
    workgroup that makes them takes 27 times as long."""
    import torch

    m = synth.pore_model(6)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6, timing=True)

    def whole_ms(reads):
        n = np.zeros(reads, np.int64)
        n[:1000] = 900
        so = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
        x = torch.randint(300, 700, (int(so[-1]),), dtype=torch.int16, device="cuda")
        d = abea.DeviceRawBatch(reads, x, torch.zeros(reads, device="cuda"), torch.ones(reads, device="cuda"), so)
        ev = torch.zeros((int(so[-1]), 3), device="cuda")
        eo = torch.zeros(reads + 1, dtype=torch.int64, device="cuda")
        best = np.inf
        for _ in range(8):
            al.detect_events_device(d, ev, eo)
            torch.cuda.synchronize()
            best = min(best, float(al.detect_timings()[2]))
        return best

    print("gpu: detect 1000 and 200000 reads", flush=True)
    few, many = whole_ms(1000), whole_ms(200000)
    print(f"{few:.3f} ms, {many:.3f} ms")
    al.close()
    assert many < 10 * few
