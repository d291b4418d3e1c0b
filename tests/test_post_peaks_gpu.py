"""The per-frame peaks that das_bmode leaves in the last F floats of its work buffer, with and without a kernel of their
own for the partial maxima.
"""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# a root of a float32 sum of two squares: within 2 units in the last place (2.4e-7 relative)
@pytest.mark.parametrize("V,F", [(1, 1), (1, 1024), (300, 32), (257, 7), (65536, 32), (65537, 32), (5000, 1000), (300000, 2),
                                 (300000, 1), (917504, 4), (917505, 4)])
def test_work_ends_with_the_peaks(V, F):
    from paper_2604_06257_amd import _lib
    lib = _lib.load()
    g = torch.Generator(device="cuda").manual_seed(V + F)
    y = torch.view_as_complex(torch.randn(V, F, 2, generator=g, device="cuda"))
    n = lib.das_bmode_work(V, F)
    work = torch.full((n,), float("nan"), device="cuda")
    out = torch.empty(V, F, device="cuda")
    p = [ctypes.c_void_p(t.data_ptr()) for t in (y, out, work)]
    _lib.check(lib.das_bmode(p[0], V, F, 60.0, p[1], p[2], n, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)),
               post=True)
    want = y.to(torch.complex128).abs().amax(0).cpu().numpy()
    np.testing.assert_allclose(work[n - F:].cpu().numpy(), want, rtol=3e-7)


# few frames on many voxels: 256 or 512 threads, one frame a thread up to 4 frames, workgroups that write up to 8192 voxels.
# The float32 logarithm of values down to -50 dB: root, quotient, log10 and product, each within 2 units in the last place
# of at most 50: 2e-5
@pytest.mark.parametrize("V,F", [(65537, 1), (262145, 2), (1048576, 1), (2097153, 2), (9000001, 1), (700001, 3), (524289, 4),
                                 (131073, 6), (70001, 9), (66000, 47), (66000, 48), (65793, 255)])
def test_decibels_of_few_frames(V, F):
    from paper_2604_06257_amd import post
    g = torch.Generator(device="cuda").manual_seed(V + F)
    y = torch.view_as_complex(torch.randn(V, F, 2, generator=g, device="cuda"))
    y *= torch.exp(torch.rand(V, 1, generator=g, device="cuda") * 5 - 4)
    got = post.bmode(y, 50.0, out=torch.full((V, F), 7.0, device="cuda"))
    a = y.to(torch.complex128).abs()
    want = (20 * torch.log10(a / a.amax(0))).clamp(min=-50.0)
    assert (got - want).abs().max().item() <= 2e-5 and bool((got.amax(0) == 0.0).all())
