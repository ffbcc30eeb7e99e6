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


@pytest.mark.parametrize("P,bound", [(5, 1.5), (7, 2.0), (9, 2.6), (11, 3.2)])
def test_waves_over_the_border(ppf, frame, P, bound):
    """A cloud over the whole frame and past its borders against one as wide inside it, both
    read from the frame: measured 1.1 to 1.8 times its step; 2.3 to 4.8 with a wait for every
    pixel of a wave that has one patch over a border."""
    def gauss_us(sd, reps=10):
        p = ppf.params(n_particles=N // 2, width=512, height=512, psf_sigma=max(0.4, P / 6.0),
                       patch=P, seed=3, ess_threshold=0.0, q=(0.5, 0.5, 0.1, 0.1, 1.0), init_kind=1,
                       init_a=(256, 256, 0, 0, 30), init_b=(sd, sd, 1.0, 1.0, 5))
        f = ppf.Filter(p)
        for _ in range(10):
            f.step(frame)
        f.profile(True)
        for _ in range(reps):
            f.step(frame)
        n, ms = f.kernel_times()["k_step"]
        f.close()
        return ms / n * 1e3
    best = min(gauss_us(200) * 2 / step_us(ppf, frame, P, 200) for _ in range(3))
    assert best < bound, best


def clustered(rng, n, W, H, gap):
    """Patch centres whose workgroups are four waves, each on a spot of 3 x 3 pixels, `gap`
    pixels apart (the corners of a square)."""
    blk, wave = np.arange(n) // 256, np.arange(n) // 64 % 4
    x0, y0 = (blk * 7) % (W - gap - 40) + 20, (blk * 13) % (H - gap - 40) + 20
    cx = x0 + gap * (wave & 1) + rng.integers(0, 3, n)
    cy = y0 + gap * (wave >> 1) + rng.integers(0, 3, n)
    return cx, cy


def cluster_us(ppf, frame, P, gap, reps=10):
    n = 1 << 20
    rng = np.random.default_rng(1)
    cx, cy = clustered(rng, n, 512, 512, gap)
    x = np.zeros((5, n), np.float32)
    x[0], x[1], x[4] = cx, cy, 30.0
    p = ppf.params(n_particles=n, width=512, height=512, psf_sigma=P / 6.0, patch=P, seed=3,
                   ess_threshold=0.0, q=(0.01, 0.01, 0.0, 0.0, 0.1))
    f = ppf.Filter(p)
    f.set_particles(x, np.full(n, -np.log(n)))
    for _ in range(3):
        f.step(frame)
    f.profile(True)
    for _ in range(reps):
        f.step(frame)
    k, ms = f.kernel_times()["k_step"]
    f.close()
    return ms / k * 1e3


@pytest.mark.parametrize("P,bound", [(9, 1.3), (11, 1.4), (25, 2.0)])
def test_workgroups_of_distant_clusters(ppf, frame, P, bound):
    """Waves on spots of their own inside the frame, whose boxes are staged each for itself,
    against workgroups on one spot: measured 1.1 to 1.5 times their step; 1.6 to 2.9 from the
    frame."""
    best = min(cluster_us(ppf, frame, P, 90) / cluster_us(ppf, frame, P, 0) for _ in range(3))
    assert best < bound, best


@pytest.mark.parametrize("gap", [0, 24, 40, 52, 70])
@pytest.mark.parametrize("P", [7, 9, 13, 15, 25])
def test_clusters_against_the_oracle(ppf, P, gap):
    """Filled boxes (gap 0), boxes staged or not and boxes past any tile; one step against
    the oracle's weights."""
    mv = synth.render_movie(W, H, 1, intensity=30.0, sigma=P / 6.0, start_box=(60, 90, 60, 90),
                            seed=8)
    n = 5 * 256 + 100
    rng = np.random.default_rng(P + gap)
    cx, cy = clustered(rng, n, W, H, gap)
    one_step(ppf, mv.frames[0], cx, cy, rng, 0, n=n, width=W, height=H, s=P / 6.0, patch=P, b=10.0,
             sigma=3.0, q=(1e-3,) * 5, seed=3)


@pytest.mark.parametrize("shape", [0, 1])
@pytest.mark.parametrize("P", [1, 3, 5, 7, 9, 11, 13, 15, 25])
@pytest.mark.parametrize("size", [(200, 160), (7, 300), (300, 7), (90, 90)])
def test_clouds_past_every_border(ppf, P, size, shape):
    """Waves with patches inside, over and past the borders, on frames wider and narrower
    than a patch; one step against the oracle's weights."""
    w, h = size
    rng = np.random.default_rng(P)
    z = (10.0 + 3.0 * rng.standard_normal((h, w))).astype(np.float32)
    n = 3 * 256 + 100
    cx = rng.integers(-P - 3, w + P + 3, n)
    cy = rng.integers(-P - 3, h + P + 3, n)
    cx[256:320], cy[320:384] = w, -1  # a wave on one column, one on one row
    cx[384:448] = np.arange(64) % 3 - 1
    one_step(ppf, z, cx, cy, rng, shape, n=n, width=w, height=h, s=max(0.4, P / 6.0), patch=P,
             b=10.0, sigma=3.0, q=(1e-3,) * 5, seed=3)


def one_step(ppf, z, cx, cy, rng, shape, n, **kw):
    x = np.zeros((5, n))
    x[0], x[1] = cx + rng.uniform(-0.45, 0.45, n), cy + rng.uniform(-0.45, 0.45, n)
    x[4] = rng.uniform(20, 40, n)
    x = x.astype(np.float32)
    p, m = pair(ppf, n=n, **kw)
    a = -oracle.loglik(m, z, x.astype(np.float64))
    lw = a - a.max() - np.log(np.exp(a - a.max()).sum())
    f = ppf.Filter(p)
    f.set_shape(shape)
    f.set_particles(x, lw)
    f.step(torch.from_numpy(z).cuda())
    cur, st = snapshot(f, n, None)
    f.close()
    check_propagate(m, 1, GpuState(x, lw, np.arange(n), False, lw), cur.x)
    check_weights(m, z, lw, cur.x, cur.lw, st)
