"""Time per band of a read that has a wavefront and a SIMD to itself, against that of
an interior band at W = 100 on the same device: bands with cells outside the
table (a read of fewer k-mers than the band is wide has no others) at two and four
slots per lane, globally and with trim states, and interior bands at one and eight slots.
The bounds lie between what the bands' code takes and what it took with two wait
states of their own for each trace bit and one band's instructions at a time."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth

pytestmark = pytest.mark.gpu


def one_read(m, n_k, n_e):
    rng = np.random.default_rng(n_k + n_e)
    ranks = rng.integers(0, m.level_mean.shape[0], n_k).astype(np.uint32)
    ev = np.zeros((n_e, 3), np.float32)
    r = ranks[np.sort(rng.integers(0, n_k, n_e))]
    ev[:, 0] = rng.normal(m.level_mean[r], m.level_stdv[r])
    return synth.make_batch([synth.Read(ev, ranks, np.float32(1), np.float32(0))])


def band_kernel_ns(m, b, W, trim):
    import torch

    al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, timing=True, workers=abea.ABEA_WORKERS_SPLIT)
    db = abea.to_device(b)
    dr = abea.DeviceResult.empty(db)
    best = np.inf
    for _ in range(6):
        al.align_device(db, dr)
        torch.cuda.synchronize()
        best = min(best, float(al.timings()[1]) * 1e6)
    al.close()
    return best


def per_band(m, W, edge, trim=False):
    """From two lengths, so that what a call costs besides drops out."""
    sizes = [(W // 2, 8000), (W // 2, 16000)] if edge else [(8000, 14400), (16000, 28800)]
    t = [band_kernel_ns(m, one_read(m, *s), W, trim) for s in sizes]
    return (t[1] - t[0]) / (sum(sizes[1]) - sum(sizes[0]))


def test_time_per_band():
    m = synth.pore_model(6)
    print("gpu: time per band", flush=True)
    unit = per_band(m, 100, False)
    got = {
        "W=100 edge": (per_band(m, 100, True) / unit, 1.95),
        "W=100 edge, trim": (per_band(m, 100, True, True) / unit, 3.6),
        "W=200 edge": (per_band(m, 200, True) / unit, 3.4),
        "W=200 edge, trim": (per_band(m, 200, True, True) / unit, 6.2),
        "W=30 interior": (per_band(m, 30, False) / unit, 0.745),
        "W=300 interior": (per_band(m, 300, False) / unit, 5.35),
    }
    print(f"interior band at W=100 {unit:.1f} ns; times it:",
          ", ".join(f"{k} {v:.2f} (bound {b})" for k, (v, b) in got.items()))
    for k, (v, b) in got.items():
        assert v < b, k
