"""Interior bands at two and four slots per lane (abea_interior.h): every
refill interval length, residue of W and order of the end cells' registers, at
the widths where they change, for reads with no interior group, with one, and
with many, with k-mer moves in a row (few events per k-mer) and event moves in
a row (many), globally and with trim states, bit for bit against the oracle."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth

pytestmark = pytest.mark.gpu

# (W, cells_per_lane).  Two slots: the interval is 16 bands to W = 111, 8 to 119,
# 4 at 120.  Four: 8 bands to W = 245, 4 to 249, 2 to 251; the window at 252.
SHAPES = [(2, 2), (3, 2), (30, 2), (63, 0), (64, 0), (100, 0), (101, 0), (111, 0), (112, 0), (119, 0), (120, 0),
          (2, 4), (3, 4), (5, 4), (100, 4), (121, 0), (200, 0), (201, 0), (202, 0), (203, 0), (244, 0), (245, 0),
          (246, 0), (247, 0), (248, 0), (249, 0), (250, 0), (251, 0), (252, 0)]


def reads_for(model, W, seed):
    rng = np.random.default_rng(seed)
    out = []
    for n_k in (max(1, W - 1), W, W + 1, W + 17, W + 40, 3 * W + 61, 1500):
        for per in (0.6, 1.0, 1.8, 4.0):
            n_e = max(1, int(n_k * per) + int(rng.integers(0, 9)))
            ranks = rng.integers(0, model.level_mean.shape[0], n_k).astype(np.uint32)
            r = ranks[np.minimum((np.arange(n_e) * n_k) // n_e, n_k - 1)]
            ev = np.zeros((n_e, 3), np.float32)
            ev[:, 0] = rng.normal(model.level_mean[r], model.level_stdv[r])
            out.append(synth.Read(ev, ranks, np.float32(1), np.float32(0)))
    return out


@pytest.mark.parametrize("trim", [False, True])
@pytest.mark.parametrize("W,cpl", SHAPES)
def test_interior_bands(oracle_mod, W, cpl, trim):
    m = synth.pore_model(6)
    reads = reads_for(m, W, 1000 * W + cpl)
    batch = synth.make_batch(reads)
    o = oracle_mod.align_batch(batch, oracle_mod.Model(m.level_mean, m.level_stdv), W, n_threads=8,
                               flags=oracle_mod.TRIM if trim else 0)
    # the 256 longest reads of a batch run the form for lone wavefronts: all of
    # these, or none beside 256 copies of a longer one
    r0 = reads[-1]
    longer = synth.Read(np.concatenate([r0.events, r0.events[-100:]]), r0.ranks, r0.scale, r0.shift)
    beside = synth.make_batch(reads + [longer] * 256)
    for b, workers in ((batch, 0), (batch, 5), (beside, 0), (beside, abea.ABEA_WORKERS_SPLIT)):
        print(f"gpu: interior W={W} cells_per_lane={cpl} trim={trim} workers={workers} reads={b.n_reads}", flush=True)
        al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, workers=workers, cells_per_lane=cpl)
        g = al.align(b)
        al.close()
        assert np.array_equal(g.status[: len(reads)], o.status)
        for r in range(len(reads)):
            assert g.log_likelihood[r] == o.score[r], r
            assert np.array_equal(g.read_pairs(r), o.read_pairs(r)), r
