"""Steps that graph mode replays: RPA over more sorted lists than are ranked by counting
(many launches), and batches with four or more step launches of 4096 workgroups or more
(their step launches side by side). Each test asks which way its steps run, and every
replay gives bit for bit what a plainly stepped twin gives, with host work and
synchronisation between the replays, the frames in alternating buffers, and a reset."""
import numpy as np
import pytest

from paper_1310_5045_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

W, H = 96, 80


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def movie():
    return synth.render_movie(W, H, 4, start_box=(30, 66, 30, 50), seed=13).frames


def box(**kw):
    return dict(width=W, height=H, init_a=(26, 26, -1, -1, 15), init_b=(70, 54, 1, 1, 45), seed=3,
                **kw)


def spots(ppf, sizes, n):
    return [ppf.params(n_particles=n, psf_sigma=max(0.8, P / 6.0), patch=P, track_id=P, **box())
            for P in sizes]


def run_twins(a, b, movie, particles):
    bufs = [torch.empty((H, W), device="cuda") for _ in range(2)]
    a.graph(True)
    assert a.graph_launches() == 0  # nothing recorded yet
    launches = set()
    for rep in range(2):
        for k, z in enumerate(movie):
            buf = bufs[k % 2]
            buf.copy_(torch.from_numpy(z))
            a.step(buf)
            b.step(buf)
            launches.add(a.graph_launches())
            torch.cuda.synchronize()
            for u, v in zip(particles(a), particles(b)):
                assert np.array_equal(u, v), (rep, k)
        a.reset()
        b.reset()
    assert b.graph_launches() == 0 and len(launches) == 1
    a.graph(False)
    assert a.graph_launches() == 0
    a.close()
    b.close()
    return launches.pop()


@pytest.mark.parametrize("groups,dlb,replayed", [(8192, 1, False), (8193, 0, False),
                                                 (8193, 1, True)])
def test_rpa(ppf, movie, groups, dlb, replayed):
    p = ppf.params(n_particles=4 * groups, psf_sigma=0.8, resample=ppf.RESAMPLE_RPA, rna_group=4,
                   dlb=dlb, ess_threshold=float(groups), **box())
    n = run_twins(ppf.Filter(p), ppf.Filter(p), movie, lambda f: f.particles())
    assert (n > 12) if replayed else n == 0


@pytest.mark.parametrize("sizes,shapes,n,replayed", [
    (range(15, 26, 2), 0, 180_000, True),    # six wide sizes
    (range(9, 26, 2), 2, 117_000, True),     # two fused launches and six wide sizes
    (range(15, 26, 2), 0, 170_000, False),   # too few workgroups
    (range(19, 26, 2), 0, 263_000, True),    # four wide sizes
    (range(21, 26, 2), 0, 400_000, False),   # three launches
])
def test_batch_over_many_sizes(ppf, movie, sizes, shapes, n, replayed):
    ps = spots(ppf, sizes, n)
    a, b = ppf.Batch(ps), ppf.Batch(ps)
    for x in (a, b):
        x.set_shapes(shapes)
    launches = run_twins(a, b, movie[:2],
                         lambda x: [u for t in range(len(ps)) for u in x.particles(t)])
    # its step launches, one or two of the merge, and two of the resampling
    assert 0 < launches <= 12 if replayed else launches == 0


def test_dropped_graph(ppf, movie):
    """Changing the launches drops the graph; the next step records them again."""
    b = ppf.Batch(spots(ppf, range(9, 26, 2), 117_000))
    z = torch.from_numpy(movie[0]).cuda()
    b.graph(True)
    b.step(z)
    one = b.graph_launches()
    b.set_shapes(2)
    assert b.graph_launches() == 0
    b.step(z)
    assert b.graph_launches() == one + 1
    b.close()
