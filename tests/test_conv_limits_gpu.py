"""GPU convolution at the limits of the brick kernel: halos about 2 GiB long (32-bit offsets), weights that nearly fill the
LDS or do not fit it.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


# The farthest voxel that a lane of the first brick reads lies 5 slices, min(9, H) rows and min(17, W) voxels from the
# halo's first: with 5 x 4 x 4 voxels 100 voxels, 2^31 bytes at a stride of 10,737,418 channels.
@pytest.mark.parametrize("dims,stride", [((5, 4, 4), 10_737_416), ((5, 4, 4), 10_737_424), ((5, 4, 4), 11_000_000),
                                         ((6, 1, 3), 60_000_000), ((5, 2, 17), 7_000_000)])
def test_wide_rows_read_every_voxel(dims, stride):
    from paper_2604_06257_amd import learn as L
    g = torch.Generator(device=DEV).manual_seed(stride)
    V, cin, cout = dims[0] * dims[1] * dims[2], 16, 16
    x = torch.randn(V, cin, generator=g, device=DEV).bfloat16()
    w = (torch.randn(cout * 27 * cin, generator=g, device=DEV) / (27 * cin) ** 0.5).bfloat16()
    b = torch.randn(cout, generator=g, device=DEV)
    wide = torch.empty(V, stride, dtype=torch.bfloat16, device=DEV)
    wide[:, 8:8 + cin] = x
    got, want = (torch.full((V, cout), -5.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    L.conv3d(L.Slice(wide, 8, cin), w, b, got, dims)
    L.conv3d(x, w, b, want, dims)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("cin", [112, 120, 128, 136, 144, 160])
def test_many_input_channels_give_the_general_kernels_bits(cin):
    from paper_2604_06257_amd import learn as L
    g = torch.Generator(device=DEV).manual_seed(cin)
    dims, cout = (5, 9, 20), 32
    V = dims[0] * dims[1] * dims[2]
    x = torch.randn(V, cin, generator=g, device=DEV).bfloat16()
    w = (torch.randn(cout * 27 * cin, generator=g, device=DEV) / (27 * cin) ** 0.5).bfloat16()
    b = torch.randn(cout, generator=g, device=DEV)
    aligned = torch.full((V, cout), -5.0, dtype=torch.bfloat16, device=DEV)
    odd = torch.full((V, cout + 1), -5.0, dtype=torch.bfloat16, device=DEV)
    L.conv3d(x, w, b, aligned, dims, relu=True)
    L.conv3d(x, w, b, L.Slice(odd, 1, cout), dims, relu=True)
    assert torch.equal(aligned.view(torch.int16), odd[:, 1:].contiguous().view(torch.int16))


@pytest.mark.parametrize("dims,cin,cout", [((96, 96, 1), 120, 32), ((96, 96, 8), 96, 32), ((48, 48, 5), 72, 128),
                                           ((96, 96, 8), 64, 32), ((48, 48, 8), 72, 64)])
def test_short_rows_against_float64(dims, cin, cout):
    """Rows of up to 8 voxels with many channels, on either side of the rule that picks a kernel."""
    from paper_2604_06257_amd import learn as L
    g = torch.Generator(device=DEV).manual_seed(cin + cout)
    V = dims[0] * dims[1] * dims[2]
    x = torch.randn(V, cin, generator=g, device=DEV).bfloat16()
    w = (torch.randn(cout, 27, cin, generator=g, device=DEV) / (27 * cin) ** 0.5).bfloat16()
    got = L.conv3d(x, w.reshape(-1), None, torch.empty(V, cout, device=DEV), dims).double()
    pad = torch.nn.functional.pad(x.double().view(*dims, cin), (0, 0, 1, 1, 1, 1, 1, 1))
    want = torch.zeros(*dims, cout, dtype=torch.float64, device=DEV)
    for tap in range(27):
        z, y, u = tap // 9, tap // 3 % 3, tap % 3
        want += pad[z:z + dims[0], y:y + dims[1], u:u + dims[2]] @ w[:, tap].double().T
    # float32 sums of 27 cin products of unit scale in all: sqrt(27 cin) * 2^-24 < 4e-6 of it
    assert (got - want.view(V, cout)).abs().max().item() <= 2e-5
