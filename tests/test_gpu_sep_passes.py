"""Separable passes on register-resident items, every FFT length with the layer filling the grid.

One to three layers (row and column layer passes of both directions, detector
plane along rows and along columns) at odd batches: region sums (regions that
share rows, one at the plane's corner), the full map, the field, accumulation,
the skip field, and both seeds of the backward pass, against torch's
complex128 transforms.  Tolerance in relative 2-norm: 6e-6 on outputs, 1.2e-5
on dL/dphi, a few times what float32 transforms of these lengths measure
(1.5e-6 and 2.5e-6 at 500 and 1000 points).
"""

import numpy as np
import pytest

import oracle.donn as od

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SIZES = (64, 100, 128, 200, 256, 350, 400, 500, 512, 1000, 1024)
LAM, DX, Z = 532e-9, 36e-6, 0.3


@pytest.fixture(scope="module")
def lrb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_11268_amd import binding
    binding.load()
    return binding


def rel(a, b):
    return float(torch.linalg.vector_norm(a.to(b.dtype) - b) / torch.linalg.vector_norm(b))


@pytest.mark.parametrize("m", SIZES)
@pytest.mark.parametrize("layers", [1, 2, 3])
def test_full_aperture_step(lrb, m, layers):
    h = torch.from_numpy(od.transfer_function(LAM, DX, Z, od.FRESNEL, m)).cuda()
    hop = lambda u: torch.fft.ifft2(torch.fft.fft2(u) * h)  # noqa: E731
    b = 5 if m <= 256 else (3 if m <= 512 else 1)
    print(f"m {m} layers {layers} batch {b}", flush=True)
    g = np.random.default_rng([m, layers])
    size = max(2, m // 9)
    y0 = [0, m // 3, m // 3, m - size]
    x0 = [0, m // 5, m // 2, m - size]
    net = lrb.Network(LAM, DX, Z, lrb.LR_FRESNEL, m, m, layers, 0.95, lrb.Detector(size, y0, x0))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).cuda()  # noqa: E731
    amp, phi = dev(g.random((b, m, m))), dev(g.random((layers, m, m)) * 6.28)
    gs, gi = dev(g.standard_normal((b, 4))), dev(g.standard_normal((b, m, m)))
    skip = torch.complex(dev(g.random((b, m, m))), dev(g.random((b, m, m))))

    p = phi.double().requires_grad_()
    u = amp.double() + 0j
    for layer in range(layers):
        u = hop(u) * (float(np.float32(0.95)) * torch.polar(torch.ones_like(p[layer]), p[layer]))
    plain = hop(u)

    def region_sums(i):
        return torch.stack([i[:, y:y + size, x:x + size].sum((1, 2)) for y, x in zip(y0, x0)], 1)

    for sk in (None, skip):
        ud = plain if sk is None else plain + sk.to(torch.complex128)
        inten = ud.real ** 2 + ud.imag ** 2
        sums = region_sums(inten)
        ref_s, = torch.autograd.grad((sums * gs.double()).sum(), p, retain_graph=True)
        ref_i, = torch.autograd.grad((inten * gi.double()).sum(), p, retain_graph=True)
        saved = net.new_saved(b)
        out = lrb.lr_donn_forward(net, amp, phi, saved=saved, sums=True, intensity=True, field=True, skip=sk)
        assert rel(out["sums"], sums.detach()) < 6e-6
        assert rel(out["intensity"], inten.detach()) < 6e-6
        assert rel(out["field"], ud.detach()) < 6e-6
        assert rel(lrb.lr_donn_backward(net, phi, saved, grad_sums=gs, skip=sk)[0], ref_s) < 1.2e-5
        assert rel(lrb.lr_donn_backward(net, phi, saved, grad_intensity=gi, skip=sk)[0], ref_i) < 1.2e-5
        alone = lrb.lr_donn_forward(net, amp, phi, saved=saved, sums=True, skip=sk)["sums"]
        assert rel(alone, sums.detach()) < 6e-6
        assert rel(lrb.lr_donn_backward(net, phi, saved, grad_sums=gs, skip=sk)[0], ref_s) < 1.2e-5
        twice = lrb.lr_donn_forward(net, amp, phi, saved=saved, sums=True, intensity=True, skip=sk, accumulate=True,
                                    out_sums=alone.clone(), out_intensity=out["intensity"].clone())
        assert rel(twice["sums"], 2 * sums.detach()) < 6e-6
        assert rel(twice["intensity"], 2 * inten.detach()) < 6e-6
