"""Events, scales and shifts that leave no finite score behind them: infinite,
NaN, and so large that an emission or a sum of them overflows, as single events
and runs at the start, inside and at the end of a read.  The kernels for two and
four slots per lane take their interior bands from code for finite scores and
must give every output (the cell count of a lost read too) of the kernels that
clear every slot, which eight slots per lane run at any width, and of the oracle
where no NaN event is in the read."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth

pytestmark = pytest.mark.gpu

VALUES = (np.inf, -np.inf, np.nan, 1e25, 3e18, -1e19, 2.0**24 * 1.5, -(2.0**24))


def ordinary(rng, m, n_k, n_e):
    ranks = rng.integers(0, m.level_mean.shape[0], n_k).astype(np.uint32)
    ev = np.zeros((n_e, 3), np.float32)
    r = ranks[np.minimum((np.arange(n_e) * n_k) // n_e, n_k - 1)]
    ev[:, 0] = rng.normal(m.level_mean[r], m.level_stdv[r])
    return ev, ranks


def make_reads(m, W):
    """(has a NaN, read)"""
    rng = np.random.default_rng(77 + W)
    out = []
    n_k, n_e = 5 * W, 9 * W
    # before, at and after the first interior group, inside, near the end
    for at in (0, 1, W // 2, 2 * W, 2 * W + 17, 5 * W, 8 * W, n_e - 1):
        for v in VALUES:
            for run in (1, 40):
                ev, ranks = ordinary(rng, m, n_k, n_e)
                ev[at : at + run, 0] = v
                out.append((bool(np.isnan(v)), synth.Read(ev, ranks, np.float32(1), np.float32(0))))
    for scale, shift in ((np.inf, 0), (np.nan, 0), (1, np.inf), (1, 1e30), (-1e30, 0), (1e18, 1), (0, 0)):
        ev, ranks = ordinary(rng, m, n_k, n_e)
        nan = not (np.isfinite(scale) and np.isfinite(shift))
        out.append((nan, synth.Read(ev, ranks, np.float32(scale), np.float32(shift))))
    out.append((False, synth.Read(*ordinary(rng, m, n_k, n_e), np.float32(1), np.float32(0))))
    return out


def read_outputs(g, r):
    return (int(g.status[r]), int(g.cells[r]), g.log_likelihood[r : r + 1].view(np.uint32)[0],
            g.read_pairs(r).tobytes())


@pytest.mark.parametrize("trim", [False, True])
@pytest.mark.parametrize("W", [100, 101, 120, 200, 201, 250])
def test_nonfinite_and_huge_events(oracle_mod, W, trim):
    assert abea.min_cells_per_lane(W) in (2, 4)
    m = synth.pore_model(6)
    reads = make_reads(m, W)
    batch = synth.make_batch([r for _, r in reads])
    o = oracle_mod.align_batch(batch, oracle_mod.Model(m.level_mean, m.level_stdv), W, n_threads=8,
                               flags=oracle_mod.TRIM if trim else 0)
    print(f"gpu: non-finite W={W} trim={trim} cpl=8 reads={batch.n_reads}", flush=True)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, cells_per_lane=8)
    ref = al.align(batch)
    al.close()
    for r in range(batch.n_reads):
        if not reads[r][0]:
            assert ref.status[r] == o.status[r] and int(ref.cells[r]) == int(o.cells[r]), r
            if o.status[r] == 0:
                assert ref.log_likelihood[r] == o.score[r], r
                assert np.array_equal(ref.read_pairs(r), o.read_pairs(r)), r
    assert {0, 2} <= set(ref.status.tolist())
    for workers in (0, 7, abea.ABEA_WORKERS_SPLIT):
        print(f"gpu: non-finite W={W} trim={trim} workers={workers}", flush=True)
        al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, workers=workers)
        g = al.align(batch)
        al.close()
        for r in range(batch.n_reads):
            assert read_outputs(g, r) == read_outputs(ref, r), r
