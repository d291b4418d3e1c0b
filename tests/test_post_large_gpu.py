"""Post-processing of volumes beyond 2^30 voxels, which are too many threads for one launch."""

import pytest
import torch

pytestmark = pytest.mark.gpu
V = (1 << 30) + 777


# decibels of at most 50 to 2e-5, as at other sizes; energies in float64 rounded to float32 once
def test_bmode_beyond_one_launch():
    from paper_2604_06257_amd import post
    g = torch.Generator(device="cuda").manual_seed(1)
    y = torch.empty(V, 1, dtype=torch.complex64, device="cuda")
    torch.view_as_real(y).normal_(generator=g)
    y[V - 5] = 100.0
    out = post.bmode(y, 50.0, out=torch.full((V, 1), 7.0, device="cuda"))
    for lo in range(0, V, 1 << 27):
        a = y[lo:lo + (1 << 27)].abs().double()
        want = (20 * torch.log10(a / 100.0)).clamp(min=-50.0)
        assert (out[lo:lo + (1 << 27)] - want).abs().max().item() <= 2e-5


def test_power_doppler_beyond_one_launch():
    from paper_2604_06257_amd import post
    g = torch.Generator(device="cuda").manual_seed(2)
    y = torch.empty(V, 2, dtype=torch.complex64, device="cuda")
    torch.view_as_real(y).normal_(generator=g)
    out = post.power_doppler(y, 0, out=torch.full((V,), 7.0, device="cuda"))
    for lo in range(0, V, 1 << 27):
        want = torch.view_as_real(y[lo:lo + (1 << 27)]).double().square().sum((1, 2))
        assert (out[lo:lo + (1 << 27)] - want).abs().max().item() <= 2.0 ** -23 * want.max().item()
