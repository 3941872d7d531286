"""Angular-spectrum passes at the edges of their tiles and of the half-aperture branch.

Every FFT length with the aperture at exactly half the grid (the HalfDft
branch), one step beside it (the general branch), a few pixels wide (fewer
rows than one tile) and ragged; two-layer networks with region sums, the full
map, the skip field, gamma and both seeds of the backward pass, at odd
batches, against torch's complex128 transforms.  Tolerance: 3e-6 on outputs
and 1e-5 on dL/dphi in relative 2-norm, about four times what float32
transforms of these lengths measure (7e-7 and 2e-6).
"""

import numpy as np
import pytest

import oracle.donn as od
from paper_2306_11268_amd import workloads as wl

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SIZES = (64, 100, 128, 200, 256, 350, 400, 500, 512, 1000, 1024)
LAM, DX, Z = 1550e-9, 8e-6, 0.05


@pytest.fixture(scope="module")
def lrb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_11268_amd import binding
    binding.load()
    return binding


def rel(a, b):
    return float(torch.linalg.vector_norm(a.to(b.dtype) - b) / torch.linalg.vector_norm(b))


def hop(u, h, n, m):
    o = (m - n) // 2
    p = u.new_zeros((u.shape[0], m, m))
    p[:, o:o + n, o:o + n] = u
    return torch.fft.ifft2(torch.fft.fft2(p) * h)[:, o:o + n, o:o + n]


def apertures(m):
    half = m // 2 - (m // 2 - m) % 2
    return sorted({half, half + 2, half - 2, 6 + m % 2, m - 2})


@pytest.mark.parametrize("m", SIZES)
def test_two_layer_step(lrb, m):
    h = torch.from_numpy(od.transfer_function(LAM, DX, Z, od.ANGULAR_SPECTRUM, m)).cuda()
    b = 3 if m <= 512 else 1
    for n in apertures(m):
        print(f"m {m} n {n}", flush=True)
        g = np.random.default_rng([m, n])
        det = wl.layout_grid(n, 4, max(2, n // 10))
        net = lrb.Network(LAM, DX, Z, lrb.LR_ANGULAR_SPECTRUM, n, m, 2, 0.9, lrb.Detector(det.size, det.y0, det.x0))
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).cuda()  # noqa: E731
        amp, phi = dev(g.random((b, n, n))), dev(g.random((2, n, n)) * 6.28)
        gs, gi = dev(g.standard_normal((b, 4))), dev(g.standard_normal((b, n, n)))
        skip = torch.complex(dev(g.random((b, n, n))), dev(g.random((b, n, n))))

        p = phi.double().requires_grad_()
        u = amp.double() + 0j
        for layer in range(2):
            u = hop(u, h, n, m) * (float(np.float32(0.9)) * torch.polar(torch.ones_like(p[layer]), p[layer]))
        ud = hop(u, h, n, m) + skip.to(torch.complex128)
        inten = ud.real ** 2 + ud.imag ** 2
        sums = torch.stack([inten[:, y:y + det.size, x:x + det.size].sum((1, 2)) for y, x in zip(det.y0, det.x0)], 1)
        ref_s, = torch.autograd.grad((sums * gs.double()).sum(), p, retain_graph=True)
        ref_i, = torch.autograd.grad((inten * gi.double()).sum(), p)

        saved = net.new_saved(b)
        out = lrb.lr_donn_forward(net, amp, phi, saved=saved, sums=True, intensity=True, field=True, skip=skip)
        assert rel(out["sums"], sums.detach()) < 3e-6
        assert rel(out["intensity"], inten.detach()) < 3e-6
        assert rel(out["field"], ud.detach()) < 3e-6
        assert rel(lrb.lr_donn_backward(net, phi, saved, grad_sums=gs, skip=skip)[0], ref_s) < 1e-5
        assert rel(lrb.lr_donn_backward(net, phi, saved, grad_intensity=gi, skip=skip)[0], ref_i) < 1e-5
        # sums alone skip the rows no region covers; accumulation adds
        alone = lrb.lr_donn_forward(net, amp, phi, sums=True, skip=skip)["sums"]
        assert rel(alone, sums.detach()) < 3e-6
        twice = lrb.lr_donn_forward(net, amp, phi, sums=True, intensity=True, skip=skip, accumulate=True,
                                    out_sums=alone.clone(), out_intensity=out["intensity"].clone())
        assert rel(twice["sums"], 2 * sums.detach()) < 3e-6
        assert rel(twice["intensity"], 2 * inten.detach()) < 3e-6


@pytest.mark.parametrize("m", SIZES)
def test_far_field_and_table_rows(lrb, m):
    """The far field (centred order, even table) and a sampled-kernel hop (a
    table that is not even: every row is read), both at half and full aperture."""
    z = 5.0
    dense = np.exp(-2j * np.pi / m * np.outer(np.arange(m) - m // 2, np.arange(m) - m // 2))
    f = torch.from_numpy(dense).cuda()
    for n in sorted({m, m // 2 - (m // 2 - m) % 2}):
        g = np.random.default_rng([m, n, 1])
        u = torch.from_numpy((g.standard_normal((2, n, n)) + 1j * g.standard_normal((2, n, n))).astype(np.complex64)).cuda()
        o = (m - n) // 2
        p = torch.zeros((2, m, m), dtype=torch.complex128, device="cuda")
        p[:, o:o + n, o:o + n] = u
        x = torch.from_numpy((np.arange(m) - m // 2) * LAM * z / (m * DX)).cuda()
        k = 2 * np.pi / LAM
        r2 = x.view(m, 1) ** 2 + x.view(1, m) ** 2
        base = 2 * np.pi * np.fmod(z / LAM, 1.0)
        q = torch.polar(torch.ones_like(r2), k * r2 / (2 * z) + base) * (DX * DX / (1j * LAM * z))
        ref = torch.stack([f @ p[i] @ f for i in range(2)]) * q
        net = lrb.Network(LAM, DX, z, lrb.LR_FRAUNHOFER, n, m, 1)
        assert rel(lrb.lr_propagate(net, u), ref) < 3e-6
        if m == 350:
            continue  # the sampled kernels take lengths of factors 2, 3 and 5 only
        net = lrb.Network(LAM, DX, Z, lrb.LR_RS_IR, n, m, 1)
        h = net.H.to(torch.complex128)
        for adjoint in (False, True):
            ref = hop(u.to(torch.complex128), h.conj() if adjoint else h, n, m)
            assert rel(lrb.lr_propagate(net, u, adjoint=adjoint), ref) < 3e-6
