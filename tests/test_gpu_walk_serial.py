"""The walk of one segment at a time: paths just short enough for it and just too
long, at every number of slots per lane, globally and with trim states, bit for bit
against the oracle; and the time of walks whose segments do not meet, and of short
reads, against that of the band fill of the same reads."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_walk import make_read

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trim", [False, True])
@pytest.mark.parametrize("W,cpl", [(30, 1), (100, 2), (101, 4), (200, 4), (300, 8), (120, 16), (512, 16)])
def test_lengths_around_the_choice(oracle_mod, W, cpl, trim):
    m = synth.pore_model(6)
    rng = np.random.default_rng(W + cpl + trim)
    bands = (1024 if cpl <= 4 else 2048)
    G = 32 // cpl
    reads = []
    for b in (bands - 1, bands, bands + 1, bands + G, bands + G + 1, 2 * bands + 3 * G + 1, 5 * bands):
        for how in ("read", "flat", "noise"):
            n_k = max(1, int((b + 1) * (0.37 if how != "noise" else rng.uniform(0.3, 0.7))))
            reads.append(make_read(rng, m, max(1, b + 1 - n_k), n_k, how))
    # half a read, then noise (segments that meet above ones that do not), and the reverse
    for a, b in (("read", "noise"), ("noise", "read")):
        x, y = make_read(rng, m, 3000, 1700, a), make_read(rng, m, 3000, 1700, b)
        reads.append(synth.Read(np.concatenate([x.events, y.events]), np.concatenate([x.ranks, y.ranks]), x.scale, x.shift))
    if trim:  # the path ends many segments above the first group
        r = make_read(rng, m, 1500, 800, "read")
        pore = np.full((6000, 3), 220, np.float32)
        reads.append(synth.Read(np.concatenate([pore, r.events]), r.ranks, r.scale, r.shift))
    batch = synth.make_batch(reads)
    o = oracle_mod.align_batch(batch, oracle_mod.Model(m.level_mean, m.level_stdv), W, n_threads=8,
                               flags=oracle_mod.TRIM if trim else 0)
    for workers in (0, abea.ABEA_WORKERS_SPLIT):
        print(f"gpu: serial walk W={W} cpl={cpl} trim={trim} workers={workers}", flush=True)
        al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, workers=workers, cells_per_lane=cpl)
        g = al.align(batch)
        al.close()
        assert np.array_equal(g.status, o.status)
        for r in range(batch.n_reads):
            if o.status[r] == 0:
                assert g.log_likelihood[r] == o.score[r], r
                assert np.array_equal(g.read_pairs(r), o.read_pairs(r)), r


def walk_over_band(m, batch, W):
    import torch

    al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, timing=True, workers=abea.ABEA_WORKERS_SPLIT)
    db = abea.to_device(batch)
    dr = abea.DeviceResult.empty(db)
    best = np.full(2, np.inf)
    for _ in range(6):
        al.align_device(db, dr)
        torch.cuda.synchronize()
        best = np.minimum(best, al.timings()[1:3])
    al.close()
    return float(best[1] / best[0])


def test_walk_time():
    """Bounds between this walk and one that has segments only, in which such reads
    are walked segment after segment by one lane."""
    m = synth.pore_model(6)
    rng = np.random.default_rng(3)
    flat = synth.make_batch([make_read(rng, m, 14400, 8000, "flat")] * 64)
    tiny = synth.make_batch([make_read(rng, m, 72, 40, "read") for _ in range(500)] * 40)
    print("gpu: walk times", flush=True)
    got = {
        "flat W=30": (walk_over_band(m, flat, 30), 0.50),
        "flat W=100": (walk_over_band(m, flat, 100), 0.36),
        "flat W=500": (walk_over_band(m, flat, 500), 0.145),
        "short W=30": (walk_over_band(m, tiny, 30), 0.56),
        "short W=400": (walk_over_band(m, tiny, 400), 0.22),
    }
    print("walk / band fill:", ", ".join(f"{k} {v:.3f} (bound {b})" for k, (v, b) in got.items()))
    for k, (v, b) in got.items():
        assert v < b, k
