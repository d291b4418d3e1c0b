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
                                 (300000, 1)])
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
