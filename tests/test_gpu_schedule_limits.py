"""DLB schedules at the edges of their lists' tiles and of the sort's tile sizes
(up to 2^19 entries of both sides in tiles of 4096 whose counts the scatter adds
up itself, above in tiles of 1024), with surplus and deficit unbalanced either
way, one side empty, one sender for all receivers, and equal values; entry for
entry against the oracle. The sort through the Z-ordered initialisation too."""
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


def counts(kind, G, n):
    rng = np.random.default_rng(G)
    if kind == "random":
        return rng.integers(0, 3 * n, G)
    if kind == "senders":
        return np.full(G, n + 3)
    if kind == "receivers":
        return rng.integers(0, n, G)
    c = np.zeros(G, dtype=np.int64)
    c[G // 2] = G * n  # one sender, every other group a receiver of n
    return c


@pytest.mark.parametrize("G", [1, 2, 511, 512, 1023, 1024, 1025, 2049, 1 << 18,
                               (1 << 18) + 1])
@pytest.mark.parametrize("kind", ["random", "senders", "receivers", "one"])
def test_schedules(ppf, G, kind):
    n = 7
    c = counts(kind, G, n).astype(np.int32)
    ct = torch.from_numpy(c).cuda()
    kinds = (ppf.DLB_GS, ppf.DLB_SGS, ppf.DLB_LGS)
    if G >= 1 << 18:  # (the oracle's sorted lists are slow)
        kinds = (ppf.DLB_GS, ppf.DLB_SGS) if kind == "random" else (ppf.DLB_GS,)
    for sched in kinds:
        got = ppf.dlb_schedule(sched, ct, n).cpu().numpy()
        assert np.array_equal(got, oracle.dlb_schedule(sched, c, n)), sched


@pytest.mark.parametrize("n", [4095, 4096, 4097, (1 << 19) - 1, 1 << 19, (1 << 19) + 1])
def test_zorder_init(ppf, n):
    kw = dict(n=n, width=256, height=256, s=1.5, seed=5, init_a=(0, 0, -1, -1, 15),
              init_b=(256, 256, 1, 1, 45))
    f = ppf.Filter(pair(ppf, init_kind=3, **kw)[0])
    u = ppf.Filter(pair(ppf, init_kind=0, **kw)[0])
    got, draws = f.gather().cpu().numpy(), u.gather().cpu().numpy()
    f.close()
    u.close()
    assert np.array_equal(got, draws[:, oracle.zorder_perm(oracle.Model(init_kind=3, **kw), n)])
