"""RNA's and ARNA's local resampling at the edges of its work split: groups of
one wave up to 256 particles and of four waves beyond, four particles to a lane,
group sizes that are no multiple of four or of a record block, a last workgroup
with fewer groups than it has waves, groups without weight and all the weight on
a group's last particle."""
import math

import numpy as np
import pytest

import oracle

from parity import check_rna, check_step, pair, snapshot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(1, 9), (3, 5), (4, 6), (63, 3), (64, 2), (65, 7), (255, 5), (256, 9), (257, 3), (511, 2),
         (1000, 3), (1021, 1), (1024, 2)]


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.mark.parametrize("group,G", SIZES)
@pytest.mark.parametrize("rho", [0.0, 0.1, 1.0])
def test_standalone(ppf, group, G, rho):
    rng = np.random.default_rng(group)
    n, moved = group * G, int(rho * group)
    l = rng.normal(0, 2, n).astype(np.float32)
    if G > 2:
        l[group:2 * group] = -np.inf          # a group without weight
        l[2 * group:3 * group - 1] = -np.inf  # all of a group's weight on its last particle
    buf = torch.from_numpy(np.concatenate([np.zeros(3, np.float32), l])).cuda()
    ug = rng.random(n // group)
    for at in (0, 3):  # aligned for vector loads, and not
        lw = buf[at:at + n].clone() if at == 0 else buf[at:]
        ls = lw.cpu().numpy().astype(np.float64)
        if at == 0:
            ls[:3] = 0.0
        anc, lwg = ppf.resample_rna(lw, group, moved, torch.from_numpy(ug).cuda())
        w = np.exp(ls - ls.max())
        w /= w.sum()
        check_rna(w, group, moved, ug, anc.cpu().numpy())
        with np.errstate(divide="ignore"):
            assert np.allclose(lwg.cpu().numpy(), np.log(w.reshape(-1, group).sum(1) / group),
                               rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("group,G", SIZES)
@pytest.mark.parametrize("resample", [1, 3])
def test_filter(ppf, group, G, resample):
    n = group * G
    kw = dict(n=n, width=64, height=64, s=0.8, b=10.0, sigma=3.0, init_a=(20, 20, -1, -1, 15),
              init_b=(44, 44, 1, 1, 45), seed=9, resample=1, rna_group=group, rna_exchange=0.3)
    frames = np.random.default_rng(1).normal(10, 3, (3, 64, 64)).astype(np.float32)
    p, m = pair(ppf, **kw)
    if resample == 3:  # ARNA that never adapts is RNA
        p.resample, p.arna_min, p.arna_lost = 3, p.rna_exchange, math.inf
    f = ppf.Filter(p)
    prev, _ = snapshot(f, n, np.full(n, -math.log(n)))
    for k in range(1, 4):
        f.step(torch.from_numpy(frames[k - 1]).cuda())
        cur, st = snapshot(f, n, None)
        check_step(m, k, prev, cur, st, frames[k - 1], True)
        prev = cur
    f.close()
