"""abea_launch_t.band_clear selects no kernel: for every value eager calls and graph
replays give the oracle's results, the kernels' own clearing included (the widths
at which the refill intervals of the interior code change, the one at four slots per
lane that clears every slot, and slot counts above the least)."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,cpl", [(100, 0), (100, 4), (112, 0), (113, 0), (120, 0), (121, 0), (200, 0), (245, 0), (246, 0),
                                   (250, 0), (251, 0), (252, 0)])
def test_every_value_matches_the_oracle(oracle_mod, W, cpl):
    import torch

    m = synth.pore_model(6)
    b = synth.workload_batch("plain-4000-lognormal5kb", m, read_ids=range(40))
    o = oracle_mod.align_batch(b, oracle_mod.Model(m.level_mean, m.level_stdv), W, n_threads=8)
    assert (o.status == 0).all()

    def check(g, what):
        assert np.array_equal(g.status, o.status), what
        assert np.array_equal(g.cells.astype(np.int64), o.cells.astype(np.int64)), what
        assert np.array_equal(g.log_likelihood, o.score), what
        for r in range(b.n_reads):
            assert np.array_equal(g.read_pairs(r), o.read_pairs(r)), (what, r)

    for clear in (abea.ABEA_CLEAR_AUTO, abea.ABEA_CLEAR_WINDOW, abea.ABEA_CLEAR_EDGES):
        print(f"gpu: W={W} cpl={cpl} band_clear={clear}", flush=True)
        al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=W, cells_per_lane=cpl, band_clear=clear)
        check(al.align(b), "eager")
        db = abea.to_device(b)
        dr = abea.DeviceResult.empty(db)
        g = al.graph(db, dr)
        st = torch.cuda.Stream()
        for _ in range(3):
            dr.log_likelihood.fill_(0.0)
            dr.pairs.fill_(-1)
            torch.cuda.synchronize()
            g.launch(st)
            st.synchronize()
            check(dr.to_host(b.n_reads), "graph")
        g.close()
        al.close()
