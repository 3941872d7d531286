"""Values a caller may put into tables and arrays that the passes must honour.

The far-field table with a phase of the caller's own on every row, against
torch's complex128 transform of the same table.  Tolerance: 3e-6 in relative
2-norm, four times what float32 transforms of these lengths measure (7e-7).
A detector-plane field that is NaN or infinite where the loss does not look,
against the same step with those values finite: the gradients are equal.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LAM, DX = 1550e-9, 8e-6


@pytest.fixture(scope="module")
def lrb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_11268_amd import binding
    binding.load()
    return binding


def rel(a, b):
    return float(torch.linalg.vector_norm(a.to(b.dtype) - b) / torch.linalg.vector_norm(b))


@pytest.mark.parametrize("m,n", [(64, 64), (100, 50), (350, 350), (512, 256)])
def test_far_field_table_with_a_phase_of_its_own(lrb, m, n):
    print(f"m {m} n {n}", flush=True)
    g = np.random.default_rng([m, n, 2])
    net = lrb.Network(LAM, DX, 5.0, lrb.LR_FRAUNHOFER, n, m, 1)
    net.H *= torch.from_numpy(np.exp(6.28j * g.random((m, m))).astype(np.complex64)).cuda()
    u = torch.from_numpy((g.standard_normal((2, n, n)) + 1j * g.standard_normal((2, n, n))).astype(np.complex64)).cuda()
    o = (m - n) // 2
    p = torch.zeros((2, m, m), dtype=torch.complex128, device="cuda")
    p[:, o:o + n, o:o + n] = u
    # entry (dy, dx) of the table carries (-1)^(dy+dx), the shift of the input's origin
    ref = torch.fft.fftshift(torch.fft.fft2(p) * net.H.to(torch.complex128), dim=(1, 2))
    assert rel(lrb.lr_propagate(net, u), ref) < 3e-6


@pytest.mark.parametrize("m,n", [(64, 64), (128, 64), (200, 100), (350, 334), (1000, 500)])
@pytest.mark.parametrize("seed", ["map", "sums"])
def test_masked_loss_does_not_see_the_field_off_the_mask(lrb, m, n, seed):
    print(f"m {m} n {n} {seed}", flush=True)
    g = np.random.default_rng([m, n, 3])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).cuda()  # noqa: E731
    size = n // 4
    net = lrb.Network(LAM, DX, 0.05, lrb.LR_ANGULAR_SPECTRUM, n, m, 2, 1.0, lrb.Detector(size, [1, n // 2], [2, n // 2]))
    amp, phi = dev(g.random((3, n, n))), dev(g.random((2, n, n)) * 6.28)
    on = torch.zeros((n, n), dtype=torch.bool, device="cuda")
    for y, x in ((1, 2), (n // 2, n // 2)):
        on[y:y + size, x:x + size] = True
    gi = dev(g.standard_normal((3, n, n))) * on
    gs = dev(g.standard_normal((3, 2)))
    grads = []
    for off in (0.0, float("nan"), float("inf")):
        skip = torch.complex(dev(g.random((3, n, n))) * 0 + 0.25, torch.zeros((3, n, n), device="cuda"))
        skip.real[:, ~on] = off
        saved = net.new_saved(3)
        lrb.lr_donn_forward(net, amp, phi, saved=saved, sums=False, intensity=True, skip=skip)
        kw = {"grad_intensity": gi} if seed == "map" else {"grad_sums": gs}
        grads.append(lrb.lr_donn_backward(net, phi, saved, skip=skip, **kw)[0])
    assert bool(torch.isfinite(grads[0]).all())
    assert torch.equal(grads[1], grads[0]) and torch.equal(grads[2], grads[0])
