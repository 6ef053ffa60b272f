"""The change-point kernel's float32 sums, up to their limit: a lane takes them while
the squares around its boundaries, less a constant near their mean, add up to less
than 2^21, and a tile in which a lane's do not is taken in double.  Signals whose
largest lane lies just below, at and just above that limit (a single sample beside a
lane's boundaries, one between them, square waves of a lane's period), at every
place in a tile and its halo, bit for bit against the oracle; that the limit is met
is checked on the signals themselves."""

import numpy as np
import pytest

from paper_2101_05012_amd import abea, synth
from test_gpu_detect import compare, gpu_events_device, oracle_events

pytestmark = pytest.mark.gpu

TILE, LANE, HALO = 1024, 16, 8
LIMIT = 2.0**21


def lane_sums(x):
    """The sums of 24 squares (two overlapping of 16) that the lanes of the
    signal's inner tiles compare with the limit."""
    f = np.float32
    out = []
    for t0 in range(TILE, len(x) - TILE - 32, TILE):
        s = np.stack([x[t0 + LANE * l - HALO : t0 + LANE * l - HALO + 32] for l in range(TILE // LANE)])
        y = (s.astype(np.int64) + 32768 + 2**23).astype(f)
        c = ((y[:, 4] + y[:, 12]) + (y[:, 20] + y[:, 28])) * f(0.25)
        y = (y - c[:, None]).astype(np.float64) ** 2
        q0, q8, q16 = y[:, 0:16].sum(1), y[:, 8:24].sum(1), y[:, 16:32].sum(1)
        out += [q0 + q8, q8 + q16]
    return np.concatenate(out)


def flat(n, rng, noise):
    return 500 + rng.integers(-noise, noise + 1, n)


def signals():
    rng = np.random.default_rng(21)
    out = []
    for noise in (0, 1):
        for at in (0, 1, 7, 8, 9, 500, 503, 511, 519, 1015, 1016, 1022, 1023):
            # one sample counts once or twice in a lane's two sums
            for d in (1023, 1024, 1025, 1447, 1448, 1449, 1450):
                x = flat(4 * TILE, rng, noise)
                x[TILE + at] += d
                out.append(x)
        for d in (254, 255, 256, 257, 361, 362, 363):
            for phase in range(0, 16, 3):
                x = flat(4 * TILE, rng, noise)
                x[TILE - 32 : 2 * TILE + 32] += np.where((np.arange(TILE + 64) + phase) // 8 % 2 == 0, d, -d)
                out.append(x)
    return [x.astype(np.int16) for x in out]


def test_around_the_limit(oracle_mod):
    xs = signals()
    top = np.array([lane_sums(x).max() for x in xs])
    assert ((top >= LIMIT - 8192) & (top < LIMIT)).sum() >= 20
    assert (top == LIMIT).sum() >= 5
    assert ((top > LIMIT) & (top <= LIMIT + 8192)).sum() >= 20
    b = synth.make_raw_batch([synth.RawRead(x, np.zeros(0, np.uint32), np.float32(-7), np.float32(0.17), np.float32(1),
                                            np.float32(0), np.zeros(0, np.int64)) for x in xs])
    m = synth.pore_model(6)
    al = abea.Aligner(m.level_mean, m.level_stdv, 6)
    for params in (None, (3, 8, 0.0, 0.0), (3, 8, 0.7, 30.0)):
        print(f"gpu: detect around the limit of the float32 sums, params={params}, {len(xs)} reads", flush=True)
        pa = abea.detect_params(*params) if params else None
        po = oracle_mod.ed_params(params[0], params[2], params[1], params[3]) if params else None
        ev, eo = gpu_events_device(al, b, pa)
        want_ev, want_eo = oracle_events(oracle_mod, b, po)
        compare(f"limit {params}", ev, eo, want_ev, want_eo)
    al.close()
