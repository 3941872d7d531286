"""Codesign and layer-norm kernels at the edges of their lane groups, pieces and chunks.

Level counts on both sides of every group width, odd pixel counts, arrays on
16-byte boundaries and off them; maps of one value, of one chunk and one value
more, of more chunks than the last kernel merges itself, in place and off
16-byte boundaries.  Against float64 on the same float32 inputs: 1e-6 in
relative 2-norm on phases and maps, 3e-6 on gradients (sums of up to 1024
float32 terms, a few 1e-7 measured); hard phases exactly.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lrb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_11268_amd import binding
    binding.load()
    return binding


def rel(a, b):
    return float(torch.linalg.vector_norm(a.double() - b) / torch.linalg.vector_norm(b).clamp(min=1e-30))


def placed(t, off):
    """A contiguous copy of t that starts `off` floats into its allocation."""
    buf = torch.empty(t.numel() + off, device="cuda")
    v = buf[off:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 36, 63, 64, 65, 100, 128, 132, 255, 256, 257, 260, 512,
                               516, 1000, 1023, 1024])
def test_codesign_levels(lrb, k):
    print(f"levels {k}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    tau = 0.7
    for count, off in ((1, 0), (77, 0), (130, 1), (519, 0), (2100, 0)):
        lg = placed(torch.randn((count, k), generator=g, device="cuda") * 2, off)
        nz = placed(torch.randn((count, k), generator=g, device="cuda"), off)
        lv = placed(torch.rand((k,), generator=g, device="cuda") * 6.28, off)
        gp = torch.randn((count,), generator=g, device="cuda")
        if k > 2:  # a tie for the largest score: the first level wins
            lg[:, 1] = 9.0 - nz[:, 1]
            lg[:, k - 1] = lg[:, 1]
            nz[:, k - 1] = nz[:, 1]
        w = torch.softmax((lg.double() + nz.double()) / float(np.float32(tau)), -1)
        mean = (w * lv.double()).sum(-1)
        assert rel(lrb.lr_codesign_phase(lg, nz, lv, tau), mean) < 1e-6
        assert torch.equal(lrb.lr_codesign_phase(lg, nz, lv, tau, hard=True), lv[(lg + nz).argmax(-1)])
        ref = w * (lv.double() - mean[:, None]) * (gp.double() / float(np.float32(tau)))[:, None]
        out = placed(torch.zeros((count, k), device="cuda"), off)
        lrb.lr_codesign_backward(lg, nz, lv, tau, gp, out=out)
        if k == 1:
            # zero but for rounding: the mean is fl(fl(e l) fl(1/e)), within 3 ulp of the one level l <= 6.28
            assert float((out.abs() / gp.abs()[:, None].clamp(min=1e-30)).max()) <= 3 * 2.0 ** -23 * 6.28 / tau
        else:
            # (a spread of the levels far below their size leaves rounding: compare on the gradient's scale)
            scale = torch.linalg.vector_norm(w * lv.double() * (gp.double() / tau)[:, None])
            assert float(torch.linalg.vector_norm(out.double() - ref) / scale) < 3e-6


@pytest.mark.parametrize("count", [1, 3, 4, 255, 4095, 4096, 4097, 4100, 12288, 122500, 1048576, 1048580, 1200001])
def test_layer_norm_chunks(lrb, count):
    print(f"count {count}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(count)
    for batch, off in ((1, 0), (3, 0), (2, 1)):
        x = placed(torch.rand((batch, count), generator=g, device="cuda") * 3 + 5, off)
        gy = placed(torch.randn((batch, count), generator=g, device="cuda"), off)
        d = x.double()
        mean = d.mean(1, keepdim=True)
        rstd = 1 / torch.sqrt(((d - mean) ** 2).mean(1, keepdim=True) + 1e-5)
        ref = (d - mean) * rstd
        y, stats = lrb.lr_layer_norm(x, out=placed(torch.zeros_like(x), off))
        if count > 1:
            assert rel(y, ref) < 1e-6
        assert rel(stats, torch.cat([mean, rstd], 1)) < 1e-6
        in_place = placed(x, off)
        again, stats2 = lrb.lr_layer_norm(in_place, out=in_place)
        assert torch.equal(again, y) and torch.equal(stats, stats2)
        yd, gd = y.double(), gy.double()
        want = stats.double()[:, 1:] * (gd - gd.mean(1, keepdim=True) - yd * (gd * yd).mean(1, keepdim=True))
        dx = lrb.lr_layer_norm_backward(gy, y, stats, out=placed(torch.zeros_like(x), off))
        if count > 4:
            assert rel(dx, want) < 3e-6
        gi = placed(gy, off)
        assert torch.equal(lrb.lr_layer_norm_backward(gi, y, stats, out=gi), dx)
