"""The step kernel's single-copy tiles: workgroups whose patches do not fit
the two-copy tile keep one tile (doubles, or floats where it is larger), per
workgroup or, where even that does not fit, per wave; a wave whose box fits no
tile reads the frame. Placed particles at the edges of each choice, some of
their patches over the frame's border, weights flattened so that every
particle counts; one step against the oracle's weights, and gradient mode
against the plain step bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1310_5045_amd import synth

from parity import GpuState, check_propagate, check_weights, pair, snapshot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

W, H = 230, 200
# doubles of LDS a workgroup of each shape (and wider patches) keeps its tile in
ALL = {0: 3072, 1: 2688}


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


def cells(way, shape, P):
    """The boxes of patch centres (x0, y0, columns, rows) that the waves of a
    workgroup of 256 particles are placed in, in order."""
    cap = ALL[shape]

    def box(pixels, tw, x0=-4, y0=-6):  # tile of tw columns and at most `pixels` pixels
        return x0, y0, tw - P + 1, pixels // tw - P + 1

    corners = [(-4, -6), (W - 60, -6), (-4, H - 60), (W - 60, H - 60)]
    return {
        "double": [box(2500, 50)] * 4,
        "double_full": [box(cap, 64)] * 4,
        "float": [box(cap + 64, 64)] * 4,
        "float_full": [box(2 * cap, 64)] * 4,
        "wave_double": [box(cap // 4, 26, x, y) for x, y in corners],
        "wave_float": [box(cap // 2, 32, x, y) for x, y in corners],
        "frame": [(0, 0, W - 20, H - 20)] * 4,
        # one wave whose box fits no tile beside three that keep theirs
        "mixed": [box(cap // 4, 26, x, y) for x, y in corners[:3]] + [(0, 0, W - 20, H - 20)],
    }[way]


def layout(way, shape, P, n):
    rng = np.random.default_rng(P)
    x = np.empty((5, n))
    where = cells(way, shape, P)
    for j in range(0, n, 64):
        x0, y0, cols, rows = where[(j // 64) % 4]
        k = min(64, n - j)
        cx, cy = rng.integers(0, cols, k), rng.integers(0, rows, k)
        cx[:2], cy[:2] = (0, cols - 1), (0, rows - 1)  # the box's corners are taken
        x[0, j:j + k] = x0 + cx + rng.uniform(-0.45, 0.45, k)
        x[1, j:j + k] = y0 + cy + rng.uniform(-0.45, 0.45, k)
    x[2:4] = 0.0
    x[4] = rng.uniform(20, 40, n)
    return x.astype(np.float32)


@pytest.mark.parametrize("way", ["double", "double_full", "float", "float_full", "wave_double",
                                 "wave_float", "frame", "mixed"])
@pytest.mark.parametrize("P,shape", [(9, 0), (9, 1), (13, 0), (13, 1), (25, 0)])
def test_single_copy_tiles(ppf, way, P, shape):
    s = {9: 1.5, 13: 2.0, 25: 4.0}[P]
    mv = synth.render_movie(W, H, 1, intensity=30.0, sigma=s, start_box=(20, 60, 20, 60), seed=8)
    n = 2 * 256 + 2 * 64  # the last workgroup ends after its second wave
    kw = dict(n=n, width=W, height=H, s=s, b=10.0, sigma=3.0, q=(1e-3,) * 5, seed=3)
    p, m = pair(ppf, **kw)
    assert m.P == P
    x = layout(way, shape, P, n)
    a = -oracle.loglik(m, mv.frames[0], x.astype(np.float64))
    lw = a - a.max() - np.log(np.exp(a - a.max()).sum())
    z = torch.from_numpy(mv.frames[0]).cuda()
    f = ppf.Filter(p)
    f.set_shape(shape)
    f.set_particles(x, lw)
    f.step(z)
    cur, st = snapshot(f, n, None)
    f.close()
    check_propagate(m, 1, GpuState(x, lw, np.arange(n), False, lw), cur.x)
    check_weights(m, mv.frames[0], lw, cur.x, cur.lw, st)
    if shape == 0:
        g = ppf.Filter(pair(ppf, grad=1, **kw)[0])
        g.set_particles(x, lw)
        g.step(z)
        gx, glw, ganc = g.particles()
        g.close()
        assert np.array_equal(gx, cur.x) and np.array_equal(glw, cur.lw)
        assert np.array_equal(ganc, cur.anc)
