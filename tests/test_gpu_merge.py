"""The merge's launch shapes: one workgroup for up to four chunks of 256
records, chunk launches with a one-wave final merge up to 64 chunks, and with
a four-wave one beyond. Filters of the linear-Gaussian model on both sides of
each limit, two steps each against the oracle."""
import math

import numpy as np
import pytest

from parity import check_step, pair, snapshot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CHUNK = 256 * 256  # particles of a merge chunk
LG = dict(obs_model=1, q=(0.5, 0.5, 0.3, 0.3, 1.0), lg_r=(2.0, 2.0, 4.0), init_kind=1,
          init_a=(40, 30, 0.5, -0.3, 20), init_b=(4, 4, 0.5, 0.5, 4), seed=5)


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.mark.parametrize("n", [1, CHUNK, CHUNK + 1, 3 * CHUNK - 255, 4 * CHUNK, 4 * CHUNK + 1,
                               64 * CHUNK, 64 * CHUNK + 1])
def test_steps_at_the_merge_limits(ppf, n):
    p, m = pair(ppf, n=n, **LG)
    f = ppf.Filter(p)
    obs = np.array([[40.5, 29.6, 20.3], [41.1, 29.1, 19.2]], dtype=np.float32)
    prev, _ = snapshot(f, n, np.full(n, -math.log(n)))
    for k in (1, 2):
        f.step(torch.from_numpy(obs[k - 1]).cuda())
        cur, st = snapshot(f, n, None)
        check_step(m, k, prev, cur, st, obs[k - 1], False)
        prev = cur
    f.close()
