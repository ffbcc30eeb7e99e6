"""RPA under the greedy schedule on both sides of the number of groups up to which its
plan is made by counting: the routing against the oracle, and no jump in its time, as
the counting grows with the square of the groups."""
import numpy as np
import pytest

import oracle
from paper_1310_5045_amd import synth

from parity import check_systematic, pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LIMIT = 4096  # groups planned by counting


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def frames():
    mv = synth.render_movie(96, 96, 2, intensity=30.0, sigma=0.8, start_box=(40, 56, 40, 56),
                            seed=23)
    return torch.from_numpy(mv.frames).cuda()


def make(ppf, groups, group):
    p, m = pair(ppf, n=groups * group, width=96, height=96, s=0.8, b=10.0, sigma=3.0,
                init_a=(24, 24, -1, -1, 15), init_b=(72, 72, 1, 1, 45), resample=0, seed=6)
    p.resample, p.rna_group, p.dlb = ppf.RESAMPLE_RPA, group, ppf.DLB_GS
    return ppf.Filter(p), m


@pytest.mark.parametrize("groups,group", [(LIMIT - 1, 5), (LIMIT, 1), (LIMIT, 7), (LIMIT + 1, 1),
                                          (LIMIT + 1, 6), (5000, 33)])
def test_routing_at_the_limit(ppf, frames, groups, group):
    f, m = make(ppf, groups, group)
    for k in range(1, 3):
        f.step(frames[k - 1])
        _, lw, anc = f.particles()
        assert f.stats()["resampled"]
        sys_anc = np.sort(anc)
        check_systematic(np.exp(lw), oracle.resample_uniform(m, k), sys_anc)
        assert np.array_equal(anc, oracle.route_rpa(sys_anc, group, ppf.DLB_GS)), k
    f.close()


def test_time_of_many_groups(ppf, frames):
    """8192 groups of 4 against 4096: measured 0.9 to 1.2 times the routing; 1.4 to 1.5 by
    counting."""
    def us(groups):
        f, _ = make(ppf, groups, 4)
        for _ in range(3):
            f.step(frames[1])
        f.profile(True)
        for _ in range(50):
            f.step(frames[1])
        n, ms = f.kernel_times()["k_rpa"]
        f.close()
        return ms / n * 1e3

    best = min(us(8192) / us(LIMIT) for _ in range(3))
    assert best < 1.3, best
