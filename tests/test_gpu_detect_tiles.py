"""Change points with the windows of 3 and 8, a wavefront per tile of 1024
boundaries: read lengths around a tile's edges, samples whose span within a
tile is just inside and just beyond what the 32-bit sums hold (4096 around a
sample of the tile) and the whole 16-bit range, at the tile's edges and inside,
flat runs (a zero variance, equal statistics), events that end tiles later, and
batches at the ends of the scan's range.  Events and offsets bit for bit against
the oracle."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_detect import compare, gpu_events_device, oracle_events

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 5, 6, 15, 16, 17, 63, 1023, 1024, 1025, 1032, 1039, 1040, 1041, 2047, 2048, 2049, 3071, 3072, 3100, 5200]


def signal(rng, n, kind):
    k = max(1, n // 9)
    x = np.repeat(rng.integers(300, 900, k + 1), rng.integers(2, 18, k + 1))[:n]
    x = np.resize(x, n) if n else x
    x = x + np.round(rng.normal(0, 12, n)).astype(np.int64)
    if kind == "flat":
        x = (np.arange(n) // 40 % 3) * 50 + 400
    elif kind == "one":  # no change point in any tile
        x = np.full(n, 7)
    elif kind == "full":
        x = rng.integers(-32768, 32768, n)
    elif kind == "ends":
        x = np.where(rng.random(n) < 0.5, -32768, 32767)
    elif kind == "negative":
        x = x - 33300
    elif isinstance(kind, int) and n:  # a step of `kind` from some sample on, and back
        a = int(rng.integers(0, n))
        x = np.full(n, 100)
        x[a : a + int(rng.integers(1, 40))] += kind
        x = x + rng.integers(0, 2, n)
    return np.clip(x, -32768, 32767).astype(np.int16)


def batch(seed, kinds, lengths=LENGTHS):
    rng = np.random.default_rng(seed)
    return synth.make_raw_batch([synth.RawRead(signal(rng, n, k), np.zeros(0, np.uint32), np.float32(rng.integers(-20, 20)),
                                               np.float32(0.17), np.float32(1), np.float32(0), np.zeros(0, np.int64))
                                 for k in kinds for n in lengths])


@pytest.fixture(scope="module")
def aligner():
    m = synth.pore_model(6)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6, W=100)
    yield al
    al.close()


@pytest.mark.parametrize("params", [None, (3, 8, 0.0, 0.0), (3, 8, 1.4, 9.0), (3, 9, 1.4, 9.0)])
@pytest.mark.parametrize("kinds", [["read"] * 4, ["flat", "one"], ["full", "ends"], ["negative", "read", "full"],
                                   [1900, 2040, 2046, 2047, 2048, 2049, 2100, 4000, 4200, 32000]])
def test_tiles(aligner, oracle_mod, kinds, params):
    b = batch(len(kinds), kinds)
    print(f"gpu: detect tiles kinds={kinds} params={params} reads={b.n_reads}", flush=True)
    pa = po = None
    if params:
        pa = abea.detect_params(*params)
        po = oracle_mod.ed_params(params[0], params[2], params[1], params[3])
    ev, eo = gpu_events_device(aligner, b, pa)
    want_ev, want_eo = oracle_events(oracle_mod, b, po)
    compare(f"tiles {kinds} {params}", ev, eo, want_ev, want_eo)


@pytest.mark.parametrize("tiles", [1, 1023, 1024, 1025, 4095, 4097])
def test_tile_counts(aligner, oracle_mod, tiles):
    rng = np.random.default_rng(tiles)
    lengths = [1024 * 5 - 3] * (tiles // 5) + [1000] * (tiles % 5)
    b = batch(tiles, ["read"], [lengths[i] for i in rng.permutation(len(lengths))])
    print(f"gpu: detect {tiles} tiles", flush=True)
    ev, eo = gpu_events_device(aligner, b)
    want_ev, want_eo = oracle_events(oracle_mod, b)
    compare(f"{tiles} tiles", ev, eo, want_ev, want_eo)
