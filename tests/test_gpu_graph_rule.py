"""Graph mode on both sides of its rule: steps of at most 12 launches are
launched directly, longer ones (RPA with sorted lists over more than 8192 groups,
a batch over every patch size) replay a HIP graph; either way every step gives
bit for bit what a plainly stepped twin gives, with the frames in alternating
buffers, host work and synchronisation between the steps, and a reset."""
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
    return synth.render_movie(W, H, 5, start_box=(30, 66, 30, 50), seed=13).frames


def box(**kw):
    return dict(width=W, height=H, init_a=(26, 26, -1, -1, 15), init_b=(70, 54, 1, 1, 45), **kw)


def twins(a, b, movie, same):
    bufs = [torch.empty((H, W), device="cuda") for _ in range(2)]
    a.graph(True)
    for rep in range(2):
        for k, z in enumerate(movie):
            buf = bufs[k % 2]
            buf.copy_(torch.from_numpy(z))
            a.step(buf)
            b.step(buf)
            torch.cuda.synchronize()
            same(a, b)
        a.reset()
        b.reset()
    a.close()
    b.close()


def same_filter(a, b):
    for u, v in zip(a.particles(), b.particles()):
        assert np.array_equal(u, v)
    assert a.stats()["cum"] == b.stats()["cum"]


@pytest.mark.parametrize("groups,dlb", [(4096, 1), (8192, 0), (8193, 0), (8193, 1), (20_000, 1)])
def test_rpa(ppf, movie, groups, dlb):
    p = ppf.params(n_particles=4 * groups, psf_sigma=0.8, resample=ppf.RESAMPLE_RPA, rna_group=4,
                   dlb=dlb, seed=3, **box())
    twins(ppf.Filter(p), ppf.Filter(p), movie, same_filter)


def test_batch_of_every_patch_size(ppf, movie):
    ps = [ppf.params(n_particles=700 + 40 * P, psf_sigma=max(0.8, P / 6.0), patch=P, track_id=P,
                     seed=3, **box()) for P in range(7, 26, 2)]
    ps.append(ppf.params(n_particles=1024, resample=ppf.RESAMPLE_RNA, rna_group=64, seed=3,
                         track_id=99, **box()))

    def same(a, b):
        for t in range(len(ps)):
            for u, v in zip(a.particles(t), b.particles(t)):
                assert np.array_equal(u, v)

    a, b = ppf.Batch(ps), ppf.Batch(ps)
    for x in (a, b):
        x.set_shapes(2)
    twins(a, b, movie, same)
