"""The step of a spread-out cloud, whose workgroups' boxes of patch centres pass the
two-copy tile: timed, so that no way of reading the pixels is much slower than another
one that serves a like cloud, and against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1310_5045_amd import synth

from parity import GpuState, check_propagate, check_weights, pair, snapshot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 1 << 22


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def frame():
    mv = synth.render_movie(512, 512, 1, start_box=(60, 120, 60, 120), seed=2)
    return torch.from_numpy(mv.frames[0]).cuda()


def step_us(ppf, frame, P, side, reps=10):
    """The step kernel's time for particles spread over a square of `side` pixels, which
    never resample and hardly move."""
    p = ppf.params(n_particles=N, width=512, height=512, psf_sigma=max(0.4, P / 6.0), patch=P,
                   seed=3, ess_threshold=0.0, q=(0.01, 0.01, 0.001, 0.001, 0.1),
                   init_a=(50, 50, 0, 0, 15), init_b=(50 + side, 50 + side, 0.001, 0.001, 45))
    f = ppf.Filter(p)
    for _ in range(3):
        f.step(frame)
    f.profile(True)
    for _ in range(reps):
        f.step(frame)
    n, ms = f.kernel_times()["k_step"]
    f.close()
    return ms / n * 1e3


@pytest.mark.parametrize("P,bound", [(1, 1.25), (3, 1.05)])
def test_small_patches_on_middling_boxes(ppf, frame, P, bound):
    """Boxes that would fit one copy against ones that do not: measured 0.98 and 0.89
    times their step for 1 x 1 and 3 x 3 patches; 1.7 and 1.09 with the boxes staged."""
    best = min(step_us(ppf, frame, P, 68) / step_us(ppf, frame, P, 90) for _ in range(3))
    assert best < bound, best


@pytest.mark.parametrize("P,bound", [(5, 1.4), (7, 1.6), (9, 1.8), (11, 1.8)])
def test_boxes_that_fit_no_tile(ppf, frame, P, bound):
    """Boxes too large for one copy against boxes of a like size that may be staged:
    measured 1.2 to 1.3 times their step; 1.6 to 3.8 with a wait for every pixel."""
    best = min(step_us(ppf, frame, P, 84) / step_us(ppf, frame, P, 56) for _ in range(3))
    assert best < bound, best


W, H = 231, 197


@pytest.mark.parametrize("shape", [0, 1])
@pytest.mark.parametrize("P", [5, 7, 9, 11, 13])
@pytest.mark.parametrize("border", ["inside", "touching", "over"])
def test_patches_from_the_frame(ppf, P, shape, border):
    """Waves spread over the frame, all of whose patches lie inside it, touch its borders,
    or with one lane's patch in each wave a pixel over one of them; one step against the
    oracle's weights, and gradient mode bit for bit."""
    h = (P - 1) // 2
    mv = synth.render_movie(W, H, 1, intensity=30.0, sigma=P / 6.0, start_box=(60, 90, 60, 90),
                            seed=8)
    n = 3 * 256 + 100
    rng = np.random.default_rng(P)
    edge = {"inside": 1, "touching": 0, "over": 0}[border]
    x0, x1, y0, y1 = h + edge, W - 1 - h - edge, h + edge, H - 1 - h - edge
    cx, cy = rng.integers(x0, x1 + 1, n), rng.integers(y0, y1 + 1, n)
    corners = [(x0, y0), (x1, y1), (x0, y1), (x1, y0)]
    for j in range(0, n, 64):  # every wave's box is the whole range
        for k, (u, v) in enumerate(corners[:max(1, min(4, n - j))]):
            cx[j + k], cy[j + k] = u, v
        if border == "over":
            side = (j // 64) % 4
            cx[j] += (-1, 1, 0, 0)[side] if side != 1 else x1 - x0 + 1
            cy[j] += (0, 0, -1, y1 - y0 + 1)[side]
    x = np.empty((5, n))
    x[0], x[1] = cx + rng.uniform(-0.45, 0.45, n), cy + rng.uniform(-0.45, 0.45, n)
    x[2:4] = 0.0
    x[4] = rng.uniform(20, 40, n)
    x = x.astype(np.float32)
    kw = dict(n=n, width=W, height=H, s=P / 6.0, patch=P, b=10.0, sigma=3.0, q=(1e-3,) * 5, seed=3)
    p, m = pair(ppf, **kw)
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
    g = ppf.Filter(pair(ppf, grad=1, **kw)[0])
    g.set_particles(x, lw)
    g.step(z)
    gx, glw, ganc = g.particles()
    g.close()
    assert np.array_equal(gx, cur.x) and np.array_equal(glw, cur.lw)
    assert np.array_equal(ganc, cur.anc)
