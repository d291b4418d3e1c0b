"""A beamforming call in several launches (plans of more workgroups than one launch holds), forced on a small plan: the same
bits as in one.
"""

import numpy as np
import pytest
import torch

import paper_2604_06257_amd as das
from conftest import small_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,per_tx", [(1, False), (2, True), (7, False), (33, False)])
def test_several_launches_give_the_same_bits(F, per_tx, monkeypatch):
    iq, elem, vox, tx, p = small_case(77 + F, T=2, E=12, S=60, F=F, V=1500)
    params = das.Params(n_tx=2, n_elem=12, n_samples=60, n_frames=F, n_vox=1500, sound_speed=p["c"], fs=p["fs"],
                        f_demod=p["fd"], t0=p["t0"], f_number=p["f_number"], tukey_alpha=p["tukey_alpha"])
    out = []
    for most in (None, "8", "3"):
        if most:
            monkeypatch.setenv("DAS_LAUNCH", most)
        with das.Plan(params, *(torch.from_numpy(a).cuda() for a in (elem, vox, tx))) as plan:
            x = torch.from_numpy(iq).cuda()
            y = torch.full((2, 1500, F) if per_tx else (1500, F), complex(7.0, 7.0), dtype=torch.complex64, device="cuda")
            out.append((plan.execute_per_tx if per_tx else plan.execute)(x, out=y).cpu().numpy())
    assert np.abs(out[0]).max() > 0
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
