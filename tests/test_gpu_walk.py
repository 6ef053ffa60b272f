"""The segmented walk and the expansion of its path bits: reads whose band
counts sit at the edges of trace groups, of segments and of the largest
segment count, at every number of slots per lane, globally and with trim
states, bit for bit against the oracle.  Besides ordinary reads: events all
alike (every cell ties, so paths from different cells of a band meet late and
segments walk again) and events unrelated to the reference."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth

pytestmark = pytest.mark.gpu


def make_read(rng, model, n_e, n_k, how):
    ranks = rng.integers(0, model.level_mean.shape[0], n_k).astype(np.uint32)
    ev = np.zeros((n_e, 3), np.float32)
    if how == "flat":
        ranks[:] = ranks[0]
        ev[:, 0] = model.level_mean[ranks[0]]
    elif how == "noise":
        ev[:, 0] = rng.uniform(50, 140, n_e)
    else:
        r = ranks[np.minimum((np.arange(n_e) * n_k) // n_e, n_k - 1)]
        ev[:, 0] = rng.normal(model.level_mean[r], model.level_stdv[r])
    return synth.Read(ev, ranks, np.float32(1), np.float32(0))


def band_counts(cpl):
    G = 32 // cpl
    groups = (1, 2, 7, 8, 9, 255, 256, 257, 64 * 5 - 1, 64 * 5, 64 * 5 + 1, 64 * 9 + 3)
    return sorted({b for g in groups for b in (g * G - 1, g * G, g * G + 1) if b >= 1})


@pytest.mark.parametrize("trim", [False, True])
@pytest.mark.parametrize("W", [30, 100, 101, 200, 300, 500])
def test_band_counts_at_segment_edges(oracle_mod, W, trim):
    m = synth.pore_model(6)
    rng = np.random.default_rng(W * 2 + trim)
    reads = []
    for b in band_counts(abea.min_cells_per_lane(W)):
        for how in ("read", "flat", "noise"):
            # b = n_e + n_k - 1
            n_k = max(1, int((b + 1) * (0.37 if how != "noise" else rng.uniform(0.3, 0.7))))
            reads.append(make_read(rng, m, max(1, b + 1 - n_k), n_k, how))
    if trim:  # open pore longer than several segments before and after a read
        r = make_read(rng, m, 900, 400, "read")
        pore = np.full((1500, 3), 220, np.float32)
        reads.append(synth.Read(np.concatenate([pore, r.events, pore[:700]]), r.ranks, r.scale, r.shift))
    batch = synth.make_batch(reads)
    o = oracle_mod.align_batch(batch, oracle_mod.Model(m.level_mean, m.level_stdv), W, n_threads=8,
                               flags=oracle_mod.TRIM if trim else 0)
    for workers in (0, 5, abea.ABEA_WORKERS_SPLIT):
        print(f"gpu: walk W={W} trim={trim} workers={workers} reads={batch.n_reads}", flush=True)
        al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, workers=workers)
        g = al.align(batch)
        al.close()
        assert np.array_equal(g.status, o.status)
        for r in range(batch.n_reads):
            if o.status[r] == 0:
                assert g.log_likelihood[r] == o.score[r], r
                assert np.array_equal(g.read_pairs(r), o.read_pairs(r)), r
            else:
                assert g.pair_offset[r] == g.pair_offset[r + 1], r
