"""The merge in one launch, with derivatives and for batches, on both sides of its
limit of four chunks of 256 records."""
import math

import numpy as np
import pytest

import oracle
from paper_1310_5045_amd import synth

from parity import pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CHUNK = 256 * 256  # particles of a merge chunk
W, H = 96, 80
KW = dict(width=W, height=H, s=1.5, b=10.0, sigma=3.0, init_a=(36, 30, -1, -1, 20),
          init_b=(56, 50, 1, 1, 40), q=(0.5, 0.5, 0.2, 0.2, 1.0), seed=3)


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def movie():
    return synth.render_movie(W, H, 3, intensity=30.0, sigma=1.5, start_box=(40, 52, 34, 46),
                              seed=8)


@pytest.mark.parametrize("n", [1, 257, CHUNK + 1, 3 * CHUNK - 255, 4 * CHUNK, 4 * CHUNK + 1])
def test_derivatives_at_the_merge_limits(ppf, movie, n):
    """One step's derivatives on the device's own states, against the oracle; each sum's
    scale is the sum of its terms' magnitudes (terms of fp32 likelihoods)."""
    p, m = pair(ppf, n=n, grad=1, **KW)
    f = ppf.Filter(p)
    obs = movie.frames[0]
    f.step(torch.from_numpy(obs).cuda())
    x = f.particles()[0].astype(np.float64)
    st = f.stats()
    tang = oracle.propagate_tangent(m, 1, np.zeros((7, n)), None)
    w, _ = oracle.normalize(oracle.loglik(m, obs, x) - math.log(n))
    dll = oracle.loglik_grad(m, obs, x)
    want = oracle.step_grad(w, dll, tang)
    v = np.stack([dll[3], dll[4], dll[5], dll[0] * tang[0], dll[1] * tang[1], dll[0] * tang[3],
                  dll[1] * tang[5], dll[2] * tang[6], dll[2]])
    scale = (w[None, :] * np.abs(v)).sum(axis=1)
    got = f.grad()[1]
    assert np.all(np.abs(got - want) <= 2e-5 * (np.abs(want) + scale) + 1e-9), (got, want)
    mean = (w[None, :] * x).sum(axis=1)
    dev = (w[None, :] * np.abs(x)).sum(axis=1)
    assert np.all(np.abs(st["mean"] - mean) <= 2e-5 * dev), (st["mean"], mean)
    f.close()


@pytest.mark.parametrize("sizes", [(1, 1000, CHUNK + 1, 4 * CHUNK), (300, 4 * CHUNK + 1)])
def test_batches_at_the_merge_limits(ppf, movie, sizes):
    ps = [pair(ppf, n=n, **dict(KW, seed=3 + i))[0] for i, n in enumerate(sizes)]
    b = ppf.Batch(ps)
    singles = [ppf.Filter(p) for p in ps]
    frames = torch.from_numpy(movie.frames).cuda()
    for k in range(2):
        b.step(frames[k])
        for f in singles:
            f.step(frames[k])
        for t, (f, sb) in enumerate(zip(singles, b.stats())):
            st = f.stats()
            for key in ("k", "resampled", "ess", "max_logw", "log_sum", "delta", "cum"):
                assert sb[key] == st[key], (t, key)
            assert np.array_equal(sb["mean"], st["mean"]), t
            for u, v in zip(b.particles(t), f.particles()):
                assert np.array_equal(u, v), t
    b.close()
    for f in singles:
        f.close()
