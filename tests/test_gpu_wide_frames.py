"""Frames whose width or height plus a patch passes the largest 32-bit integer: a
filter on such a frame gives bit for bit what it gives on a frame of 4096 pixels
with the same pixels near the particles (no patch reaches the narrow frame's end)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LONG = 2**31 - 1
SHORT = 4096


@pytest.fixture(scope="module")
def ppf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1310_5045_amd as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def pixels():
    z = torch.full((LONG,), 10.0, device="cuda")  # 8.6 GB, one row or one column
    z[2000:2040] += torch.linspace(0, 30, 40, device="cuda")
    return z


@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("sigma", [0.3, 1.5, 4.0])  # 1 x 1, 9 x 9 and 25 x 25 patches
def test_frame_of_the_largest_side(ppf, pixels, wide, sigma):
    def run(side, z):
        w, h = (side, 1) if wide else (1, side)
        a, b = [2020.0, 0.0], [6.0, 0.3]  # along the frame, and across it
        if not wide:
            a, b = a[::-1], b[::-1]
        p = ppf.params(n_particles=700, width=w, height=h, psf_sigma=sigma, seed=5, init_kind=1,
                       init_a=(*a, 0, 0, 30), init_b=(*b, 0.3, 0.3, 5))
        f = ppf.Filter(p)
        for _ in range(3):
            f.step(z.view(h, w))
        out = f.particles(), f.stats()
        f.close()
        return out

    (x, lw, anc), st = run(SHORT, pixels[:SHORT].clone())
    (gx, glw, ganc), gst = run(LONG, pixels)
    assert np.ptp(lw) > 1.0  # the pixels tell the particles apart
    assert np.array_equal(gx, x) and np.array_equal(glw, lw) and np.array_equal(ganc, anc)
    assert gst["cum"] == st["cum"] and gst["k"] == st["k"] == 3
