"""RPA where its launches change: ranking by counting up to 8192 groups and
sorted lists beyond, and the groups' offspring ranges by a look at every slot up
to 2^22 particles and by search beyond; with one group, groups of one particle
and numbers of slots that are no multiple of four. The resampled multiset is the
systematic one and the placement the oracle's routing, also where all the weight
lies in a few groups."""
import numpy as np
import pytest

import oracle
from paper_1310_5045_amd import synth

from parity import check_systematic, pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.mark.parametrize("dlb", [0, 1])
@pytest.mark.parametrize("groups,group", [(1, 999), (15, 67), (17, 1), (63, 5), (4097, 3), (8191, 4),
                                          (8192, 5), (8193, 4), (8192, 512), (8193, 512)])
def test_routing(ppf, dlb, groups, group):
    n = groups * group
    mv = synth.render_movie(96, 96, 2, intensity=30.0, sigma=0.8, start_box=(40, 56, 40, 56),
                            seed=23)
    p, m = pair(ppf, n=n, width=96, height=96, s=0.8, b=10.0, sigma=3.0,
                init_a=(24, 24, -1, -1, 15), init_b=(72, 72, 1, 1, 45), resample=0, seed=6)
    p.resample, p.rna_group, p.dlb = ppf.RESAMPLE_RPA, group, dlb
    f = ppf.Filter(p)
    frames = torch.from_numpy(mv.frames).cuda()
    for k in range(1, 3):
        f.step(frames[k - 1])
        x, lw, anc = f.particles()
        assert f.stats()["resampled"]
        sys_anc = np.sort(anc)
        check_systematic(np.exp(lw), oracle.resample_uniform(m, k), sys_anc)
        assert np.array_equal(anc, oracle.route_rpa(sys_anc, group, dlb)), k
    f.close()
