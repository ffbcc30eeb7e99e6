"""The radix sort's two tile sizes, through the initialisation that sorts by
Z order: the cloud must be the stable order of the particles' Morton keys at
the edges of the tiles of both sizes, and where the wide tiles begin."""
import numpy as np
import pytest

import oracle

from parity import pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.mark.parametrize("n", [1, 63, 256, 1023, 1024, 1025, 40_961, (1 << 22) - 1, 1 << 22,
                               (1 << 22) + 4097])
def test_zorder_init_is_the_stable_key_order(ppf, n):
    kw = dict(n=n, width=256, height=256, s=1.5, seed=5, init_a=(0, 0, -1, -1, 15),
              init_b=(256, 256, 1, 1, 45))
    f = ppf.Filter(pair(ppf, init_kind=3, **kw)[0])
    got = f.gather().cpu().numpy()
    f.close()
    u = ppf.Filter(pair(ppf, init_kind=0, **kw)[0])
    draws = u.gather().cpu().numpy()  # the same draws in draw order
    u.close()
    m = oracle.Model(init_kind=3, **kw)
    assert np.array_equal(got, draws[:, oracle.zorder_perm(m, n)])
