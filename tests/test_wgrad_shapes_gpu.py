"""Weight gradient of volumes whose axes change places (few short rows, few parts), against float64."""

import pytest
import torch

from test_wgrad_blocks_gpu import check

pytestmark = pytest.mark.gpu


# tolerance as for the other volumes: rounding of at most sqrt(voxels) * 2^-24 of the terms' scale against 1e-5
@pytest.mark.parametrize("dims,cin,cout,chunk", [((64, 3, 3), 16, 16, 1024), ((31, 48, 1), 16, 16, 1504), ((2, 48, 4), 24, 32, 384), ((10, 5, 2), 48, 32, 128), ((5, 1, 90), 8, 16, 128), ((64, 3, 3), 112, 48, 320), ((63, 2, 5), 24, 32, 352),
                                                 ((200, 1, 1), 8, 16, 224), ((97, 2, 140), 16, 16, 32768), ((300, 3, 2), 128, 32, 96)])
def test_wgrad_of_narrow_volumes(dims, cin, cout, chunk):
    from paper_2604_06257_amd import learn
    g = torch.Generator(device="cuda").manual_seed(dims[0] + cin)
    v = dims[0] * dims[1] * dims[2]
    x = torch.randn((v, cin + 16), generator=g, device="cuda").bfloat16()
    dy = torch.randn((v, cout + 8), generator=g, device="cuda").bfloat16()
    check(learn.Slice(x, 8, cin), learn.Slice(dy, 8, cout), dims, cin, cout, chunk)


def test_wgrad_of_deep_volumes_beyond_32_bit_offsets():
    from paper_2604_06257_amd import learn
    dims, stride = (60, 1, 2), 1 << 24
    buf = torch.zeros((120, stride), dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    buf[:, 32:48] = torch.randn((120, 16), generator=g, device="cuda").bfloat16()
    dy = torch.randn((120, 16), generator=g, device="cuda").bfloat16()
    check(learn.Slice(buf, 32, 16), learn.Slice(dy), dims, 16, 16, 128)
