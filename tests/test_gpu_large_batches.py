"""Batches of millions of tiny apertures: more threads in all than one launch holds (2^32).

Region sums of more than 2^26 regions, each one pixel, against the intensity
map of the same call (equal), and an angular-spectrum hop of 2 x 2 pixels in
a 100 grid against the same hop of a few of its samples (equal).
"""

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


def gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def test_region_sums_of_a_million_samples(lrb):
    n, b = 8, (1 << 20) + 5
    ys, xs = [i // n for i in range(64)], [i % n for i in range(64)]
    net = lrb.Network(532e-9, 36e-6, 0.3, lrb.LR_FRESNEL, n, 64, 1, 1.0, lrb.Detector(1, ys, xs))
    amp = torch.rand((b, n, n), generator=gen(1), device="cuda")
    phi = torch.rand((1, n, n), generator=gen(2), device="cuda") * 6.28
    out = lrb.lr_donn_forward(net, amp, phi, sums=True, intensity=True)
    assert torch.equal(out["sums"].view(b, n, n), out["intensity"])


def test_hop_of_four_million_samples(lrb):
    n, m, b = 2, 100, (1 << 22) + 5
    net = lrb.Network(532e-9, 36e-6, 0.3, lrb.LR_ANGULAR_SPECTRUM, n, m)
    u = torch.view_as_complex(torch.rand((b, n, n, 2), generator=gen(3), device="cuda"))
    out = lrb.lr_propagate(net, u)
    for at in (slice(0, 7), slice(b // 2, b // 2 + 7), slice((1 << 22) - 20, b)):
        assert torch.equal(out[at], lrb.lr_propagate(net, u[at].contiguous()))
