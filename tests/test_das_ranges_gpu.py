"""Plans at the edges of the beamforming kernels' ranges: which kernel serves them, and its results against the FP64 oracle.
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2604_06257_amd as das
from synth import linear_array
from synth.configs import random_iq

pytestmark = pytest.mark.gpu
C, FS, FD = 1540.0, 20e6, 5e6
GENERAL = (0, 0, 0)  # what das_plan_query reports for the general kernel


def column(n=64, z0=4e-3, step=5e-5):
    vox = np.zeros((n, 3), np.float32)
    vox[:, 2] = z0 + step * np.arange(n)
    return vox


def run(iq, elem, vox, tx, t0=0.0, fs=FS, fd=FD, per_tx=False):
    T, E, S, F = iq.shape
    p = das.Params(T, E, S, F, vox.shape[0], C, fs, fd, t0, 0.8, 0.5)
    with das.Plan(p, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (elem, vox, tx))) as plan:
        kernel = plan.info()["kernel"]
        x = torch.from_numpy(iq).cuda()
        y = (plan.execute_per_tx if per_tx else plan.execute)(x).cpu().numpy()
    o = dict(c=C, fs=fs, fd=fd, t0=t0, f_number=0.8, tukey_alpha=0.5)
    ref = (np.stack([oracle.das(iq[t:t + 1], elem, vox, tx[t:t + 1], **o) for t in range(T)]) if per_tx
           else oracle.das(iq, elem, vox, tx, **o))
    assert np.abs(ref).max() > 0
    return kernel, oracle.nrmse_db(y, ref)


@pytest.mark.parametrize("T,F", [(1, 1), (2, 3)])
def test_rows_too_far_apart_take_the_general_kernel(T, F):
    """A 600,000-row record, half of whose voxels use its beginning and half its end: more than 2^19 rows between them."""
    elem = linear_array(4, 0.3e-3)
    vox = column()
    tx = np.stack([vox[:, 2] / C + 1e-7 * t for t in range(T)]).astype(np.float32)
    tx[:, 32:] += np.float32(0.029)
    iq = random_iq((T, 4, 600_000, F), seed=1)
    kernel, db = run(iq, elem, vox, tx)
    assert kernel == GENERAL and db <= -100.0
