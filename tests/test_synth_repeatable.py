"""The torch generator of lognormal boxes draws from its seed alone: the running
sum behind it has the same bits on every call and is the exact one to a few
roundings, and a large box drawn again and again is the same box."""
import numpy as np
import pytest

from paper_2301_12557_amd import synth


def _density(ngrid, device):
    import torch
    g = torch.Generator(device=device)
    g.manual_seed(3)
    return torch.exp(torch.randn(ngrid ** 3, generator=g, device=device, dtype=torch.float64) - 0.5)


def _check_sum(rho, ngrid, repeats):
    import torch
    first = synth._running_sum_torch(rho, ngrid)
    for _ in range(repeats):
        assert torch.equal(synth._running_sum_torch(rho, ngrid), first)
    # a row of ngrid adds up its values with at most ngrid roundings of the row's own
    # sum; the sum of the rows before it adds one rounding (those of their own sums
    # are far below it), and the addition of the two rounds once more
    # (the exact sums: multiples of 2^-30 in whole numbers, the rests below them in extended precision)
    r = rho.cpu().numpy()
    whole = np.floor(np.ldexp(r, 30))
    want = np.ldexp(np.cumsum(whole.astype(np.int64)).astype(np.longdouble), -30)
    want += np.cumsum((r - np.ldexp(whole, -30)).astype(np.longdouble))
    got = first.cpu().numpy()
    row = rho.reshape(-1, ngrid).sum(1).cpu().numpy().max()
    assert np.all(np.abs(got - want) <= 2.0 ** -53 * (2.0 * want + ngrid * row) * 1.01)
    assert np.all(np.diff(got) >= 0)


def test_running_sum():
    pytest.importorskip("torch")
    _check_sum(_density(32, "cpu"), 32, 3)


def test_box_repeats_on_the_cpu():
    torch = pytest.importorskip("torch")
    a, b = (synth.lognormal_box_torch(5000, 100.0, 9, device="cpu", ngrid=32) for _ in range(2))
    assert torch.equal(a, b)
    assert float(a.min()) >= 0.0 and float(a.max()) < 100.0


@pytest.mark.gpu
def test_running_sum_repeats_on_the_gpu():
    _check_sum(_density(256, "cuda"), 256, 40)


@pytest.mark.gpu
def test_large_box_repeats_on_the_gpu():
    import torch
    first = synth.lognormal_box_torch(10_000_000, 3000.0, 5)
    for _ in range(12):
        assert torch.equal(synth.lognormal_box_torch(10_000_000, 3000.0, 5), first)
