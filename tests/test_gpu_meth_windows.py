"""Methylation windows at the edges of what the scoring kernels hold: every
window length that has a form of its own (k = 5 and 6 with the models in LDS, 9)
and those of the general form (2, 3, 7), windows cut off by the read's start, reads
of one k-mer to a few more than a wavefront's run of pairs or a thread's four
k-mers, trim states (paths that begin past event 0) and events scaled to the
model; LLRs bit for bit against the oracle."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_meth import compare, gpu_scores, oracle_scores

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 63, 64, 65, 250, 511, 512, 513, 1023, 1024, 1025, 1027, 2100]


@pytest.mark.parametrize("form", ["plain", "trim", "scale"])
@pytest.mark.parametrize("k", [2, 3, 5, 6, 7, 9])
def test_window_lengths(oracle_mod, k, form):
    m = synth.pore_model(k)
    mm = synth.methylated_model(m)
    rng = np.random.default_rng(10 * k)
    cg = (1 << (2 * (k - 1))) | (2 << (2 * (k - 2)))
    reads = []
    for n_k in LENGTHS:
        for dense in (False, True):  # bases at random; every k-mer a site
            ranks = rng.integers(0, 4**k, n_k)
            if dense:
                ranks = cg | (ranks & (4 ** (k - 2) - 1))
            ranks = ranks.astype(np.uint32)
            n_e = max(1, int(n_k * rng.uniform(1.0, 2.4)))
            r = ranks[np.minimum((np.arange(n_e) * n_k) // n_e, n_k - 1)]
            ev = np.ones((n_e, 3), np.float32)
            ev[:, 0] = rng.normal(m.level_mean[r], m.level_stdv[r])
            reads.append(synth.Read(ev, ranks, np.float32(1), np.float32(0)))
    b = synth.make_batch(reads)
    print(f"gpu: methylation windows k={k} {form}", flush=True)
    flags = {"plain": 0, "trim": oracle_mod.TRIM, "scale": oracle_mod.SCALE_EVENTS}[form]
    al = abea.Aligner(m.level_mean, m.level_stdv, k, W=100, trim=form == "trim", scale_events=form == "scale")
    al.set_methylated_model(mm.level_mean, mm.level_stdv)
    got = gpu_scores(al, b)
    al.close()
    assert compare(f"k={k} {form}", got, oracle_scores(oracle_mod, b, m, mm, flags=flags)) > 1000
