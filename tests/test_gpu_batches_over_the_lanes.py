"""Backward passes whose persistent workgroups take several samples each.

The accumulating passes keep one tile per workgroup and share a batch among
as many lanes of workgroups as fit on the device (CUs * 16 waves / tiles of a sample, or
fewer); BATCH is larger at every length and a multiple of none.  dL/dphi of three-layer
Fresnel and two-layer angular-spectrum and Rayleigh-Sommerfeld networks
against torch's complex128 transforms, to 1.2e-5 in relative 2-norm (2.5e-6
measured at 500 and 1000 points).  The sum over the batch runs in a fixed
order: a second call gives the same bits.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BATCH = {64: 1031, 100: 701, 128: 521, 200: 271, 256: 131, 350: 103, 400: 71, 500: 53, 512: 67, 1000: 17, 1024: 19}
VISIBLE, INFRARED = (532e-9, 36e-6, 0.3), (1550e-9, 8e-6, 0.05)


@pytest.fixture(scope="module")
def lrb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_11268_amd import binding
    binding.load()
    return binding


def hop(u, h, n, m):
    o = (m - n) // 2
    p = u.new_zeros((u.shape[0], m, m))
    p[:, o:o + n, o:o + n] = u
    return torch.fft.ifft2(torch.fft.fft2(p) * h)[:, o:o + n, o:o + n]


def check(lrb, approx, optics, n, m, layers, seed, b=0):
    b = b or BATCH[m]
    print(f"approx {approx} n {n} m {m} layers {layers} batch {b}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * m + n)
    net = lrb.Network(*optics, approx, n, m, layers, 0.95, lrb.Detector(max(2, n // 6), [0, n // 2], [n // 3, n // 2]))
    h = net.H.to(torch.complex128)
    amp = torch.rand((b, n, n), generator=g, device="cuda")
    phi = torch.rand((layers, n, n), generator=g, device="cuda") * 6.28
    gi = torch.randn((b, n, n), generator=g, device="cuda")
    gs = torch.randn((b, 2), generator=g, device="cuda")
    p = phi.double().requires_grad_()
    step = max(1, 8_000_000 // (m * m))
    size = net.detector.size
    for lo in range(0, b, step):
        u = amp[lo:lo + step].double() + 0j
        for layer in range(layers):
            u = hop(u, h, n, m) * (float(np.float32(0.95)) * torch.polar(torch.ones_like(p[layer]), p[layer]))
        u = hop(u, h, n, m)
        i = u.real ** 2 + u.imag ** 2
        if seed == "map":
            loss = (i * gi[lo:lo + step].double()).sum()
        else:
            s = torch.stack([i[:, y:y + size, x:x + size].sum((1, 2)) for y, x in ((0, n // 3), (n // 2, n // 2))], 1)
            loss = (s * gs[lo:lo + step].double()).sum()
        loss.backward()
    saved = net.new_saved(b)
    lrb.lr_donn_forward(net, amp, phi, saved=saved, sums=True)
    kw = {"grad_intensity": gi} if seed == "map" else {"grad_sums": gs}
    got = lrb.lr_donn_backward(net, phi, saved, **kw)[0]
    for layer in range(layers):
        err = torch.linalg.vector_norm(got[layer].double() - p.grad[layer]) / torch.linalg.vector_norm(p.grad[layer])
        assert float(err) < 1.2e-5, (layer, float(err))
    assert torch.equal(lrb.lr_donn_backward(net, phi, saved, **kw)[0], got)


@pytest.mark.parametrize("m", sorted(BATCH))
@pytest.mark.parametrize("seed", ["map", "sums"])
def test_separable(lrb, m, seed):
    check(lrb, lrb.LR_FRESNEL, VISIBLE, m, m, 3, seed)


@pytest.mark.parametrize("m", sorted(BATCH))
def test_padded_separable(lrb, m):
    check(lrb, lrb.LR_FRESNEL, VISIBLE, m - 2 * (m // 7), m, 3, "map")


@pytest.mark.parametrize("m", sorted(BATCH))
@pytest.mark.parametrize("half", [False, True])
def test_angular_spectrum(lrb, m, half):
    n = m // 2 - (m // 2 - m) % 2 if half else m
    check(lrb, lrb.LR_ANGULAR_SPECTRUM, INFRARED, n, m, 2, "sums" if half else "map")


@pytest.mark.parametrize("m", [m for m in sorted(BATCH) if m != 350])  # (a sampled kernel takes factors 2, 3 and 5)
def test_sampled_kernel(lrb, m):
    n = m // 2 - (m // 2 - m) % 2
    check(lrb, lrb.LR_RS_IR, INFRARED, n, m, 1, "map")


# (the column passes change kernels between the two batches of a pair, on 256 CUs)
@pytest.mark.parametrize("m,b", [(64, 255), (64, 256), (100, 255), (100, 256), (128, 127), (128, 128), (256, 31),
                                 (256, 32), (400, 20), (400, 21), (500, 30), (500, 31), (500, 127), (500, 128),
                                 (512, 15), (512, 16), (512, 128), (512, 129), (1000, 6), (1000, 7)])
def test_both_sides_of_the_batch_rule(lrb, m, b):
    check(lrb, lrb.LR_FRESNEL, VISIBLE, m, m, 3, "map", b)
