"""Heavy resampling segments on both sides of the limit where one launch does
the whole pass (2^20 weights: 1024 segments): the weight on one, two or many
particles, at the first, a middle and the last one, ancestors against the
oracle; through the standalone resampler and through a filter's own weights."""
import math

import numpy as np
import pytest

from parity import check_step, check_systematic, pair, snapshot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LIMIT = 1 << 20


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


def weights(kind, n):
    rng = np.random.default_rng(n)
    if kind == "ramp":  # every segment about as heavy, few of them at the limit of it
        return np.log(np.linspace(1e-3, 1.0, n))
    l = np.full(n, -80.0)
    where = {"first": [0], "last": [n - 1], "two": [n // 2, n // 2 + 1],
             "spread": np.linspace(0, n - 1, 37).astype(int)}[kind]
    l[where] = rng.normal(0.0, 0.5, len(where))
    return l


@pytest.mark.parametrize("n", [5000, 64 * 1024, 64 * 1024 + 1, LIMIT, LIMIT + 1])
@pytest.mark.parametrize("kind", ["first", "last", "two", "spread", "ramp"])
def test_standalone(ppf, n, kind):
    l32 = weights(kind, n).astype(np.float32)
    w = np.exp(l32.astype(np.float64) - l32.max())
    w /= w.sum()
    for u in (0.0, 0.61):
        anc = ppf.resample_systematic(torch.from_numpy(l32).cuda(), u).cpu().numpy()
        assert check_systematic(w, u, anc)[1] == 0


@pytest.mark.parametrize("n", [3000, 64 * 1024 + 1, LIMIT, LIMIT + 1])
@pytest.mark.parametrize("kind", ["last", "spread"])
def test_filter(ppf, n, kind):
    # a flat likelihood, so that the weights set are the weights resampled
    p, m = pair(ppf, n=n, obs_model=1, q=(0.1,) * 5, lg_r=(1e3,) * 3, init_kind=1,
                init_a=(40, 30, 0, 0, 20), init_b=(1,) * 5, seed=5)
    f = ppf.Filter(p)
    l = weights(kind, n)
    lw = l - l.max() - math.log(np.exp(l - l.max()).sum())
    x, _, _ = f.particles()
    f.set_particles(x, lw)
    prev, _ = snapshot(f, n, lw)
    prev.lw_next, prev.resampled = lw, False
    obs = np.array([40, 30, 20], dtype=np.float32)
    f.step(torch.from_numpy(obs).cuda())
    cur, st = snapshot(f, n, None)
    check_step(m, 1, prev, cur, st, obs, False)
    f.close()
