"""The pool's cap by residency at two slots per lane: five wavefronts per SIMD, in
single-wavefront workgroups and in those of four, however few registers the kernel
needs (a launch of five a SIMD is to fill each with five)."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_walk import make_read

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trim", [False, True])
@pytest.mark.parametrize("W", [100, 101])
@pytest.mark.parametrize("wpg", [1, 4])
def test_five_per_simd(oracle_mod, W, wpg, trim):
    import torch

    m = synth.pore_model(6)
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    one = make_read(np.random.default_rng(W), m, 60, 40, "read")
    n = 6 * simds + 7
    o = oracle_mod.align_batch(synth.make_batch([one]), oracle_mod.Model(m.level_mean, m.level_stdv), W, n_threads=1,
                               flags=oracle_mod.TRIM if trim else 0)
    print(f"gpu: resident W={W} wpg={wpg} trim={trim} n={n}", flush=True)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, trim=trim, workers=n, waves_per_group=wpg, cells_per_lane=2)
    g = al.align(synth.make_batch([one] * n))
    workers = al.plan_info()["workers"]
    al.close()
    assert workers == 5 * simds
    assert np.array_equal(g.status, np.full(n, o.status[0]))
    assert (g.log_likelihood == o.score[0]).all()
    for r in (0, 5 * simds - 1, 5 * simds, n - 1):
        assert np.array_equal(g.read_pairs(r), o.read_pairs(0)), r
