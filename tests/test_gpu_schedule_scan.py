"""DLB schedules of so many groups that the tile sums are scanned by a launch of their
own: over 4096 tiles of 256 senders (2^20 groups) for the entries' prefixes, over 4096
tiles of 1024 positions (2^22 groups) for the lists'. Entry for entry against the
schedules' definitions: greedy matching as the overlap of the surplus and deficit
intervals laid end to end in list order, and rank pairing."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


def want(ppf, kind, counts, n):
    d = counts.astype(np.int64) - n
    lists = []
    for v in (np.maximum(d, 0), np.maximum(-d, 0)):
        g = np.flatnonzero(v)
        if kind != ppf.DLB_GS:
            g = g[np.argsort(-v[g], kind="stable")]
        lists.append((g, v[g]))
    (sg, sv), (rg, rv) = lists
    if kind == ppf.DLB_LGS:
        m = min(len(sg), len(rg))
        return np.stack([sg[:m], rg[:m], np.minimum(sv[:m], rv[:m])], axis=1)
    cs, cr = np.cumsum(sv), np.cumsum(rv)
    total = min(cs[-1], cr[-1])
    # the cuts of both lists up to the smaller total: an entry between each two
    cuts = np.union1d(cs, cr)
    cuts = cuts[:np.searchsorted(cuts, total) + 1]
    lo = np.concatenate([[0], cuts[:-1]])
    return np.stack([sg[np.searchsorted(cs, lo, side="right")],
                     rg[np.searchsorted(cr, lo, side="right")], cuts - lo], axis=1)


@pytest.mark.parametrize("G", [1025, 1 << 20, (1 << 20) + 1, (1 << 22) - 1, (1 << 22) + 1])
@pytest.mark.parametrize("more", [0, 2])  # offspring equal to or above the groups' slots on average
def test_schedules_of_many_groups(ppf, G, more):
    n = 5
    counts = np.random.default_rng(G).integers(0, 2 * n + 1 + more, G).astype(np.int32)
    ct = torch.from_numpy(counts).cuda()
    for kind in (ppf.DLB_GS, ppf.DLB_SGS, ppf.DLB_LGS):
        got = ppf.dlb_schedule(kind, ct, n).cpu().numpy()
        assert np.array_equal(got, want(ppf, kind, counts, n)), kind
