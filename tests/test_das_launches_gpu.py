"""How a plan cuts its launch, forced on small plans: several launches (plans of more workgroups than one holds), element
groups and wave tiles of a workgroup.
"""

import numpy as np
import pytest
import torch

import oracle
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


SPLITS = ["1,1", "1,2", "1,4", "2,1", "2,4", "4,1", "4,4", "8,1", "8,2", "16,1"]  # groups, wave tiles (cut to fit a workgroup)


@pytest.mark.parametrize("kind", ["c64", "f16", "bf16"])
@pytest.mark.parametrize("variant,F,T", [("1,65,1", 1, 1), ("1,65,1", 2, 2), ("2,129,1", 3, 1), ("4,65,1", 6, 2), ("8,65,1", 11, 1),
                                         ("16,65,2", 23, 2), ("32,65,2", 40, 1)])
def test_groups_and_wave_tiles(variant, F, T, kind, monkeypatch):
    """Every number of groups (up to more than there are items) and of wave tiles a workgroup, for each wave size."""
    iq, elem, vox, tx, p = small_case(900 + F, T=T, E=19, S=96, F=F, V=700, depth=(0.3e-3, 2.0e-3))
    x = torch.from_numpy(iq)
    if kind != "c64":
        x = torch.view_as_real(x).to(torch.float16 if kind == "f16" else torch.bfloat16).contiguous()
        iq = x.float().numpy().view(np.complex64)[..., 0]
    ref = oracle.das(iq, elem, vox, tx, **p)
    params = das.Params(n_tx=T, n_elem=19, n_samples=96, n_frames=F, n_vox=700, sound_speed=p["c"], fs=p["fs"],
                        f_demod=p["fd"], t0=p["t0"], f_number=p["f_number"], tukey_alpha=p["tukey_alpha"])
    monkeypatch.setenv("DAS_VARIANT", variant)
    for split in SPLITS:
        monkeypatch.setenv("DAS_SPLIT", split)
        with das.Plan(params, *(torch.from_numpy(a).cuda() for a in (elem, vox, tx))) as plan:
            assert plan.info()["kernel"] == tuple(map(int, variant.split(",")))
            y = plan.execute(x.cuda()).cpu().numpy()
            db = [oracle.nrmse_db(y, ref)]
            if F <= 2:
                y = plan.execute_per_tx(x.cuda()).cpu().numpy()
                db += [oracle.nrmse_db(y[t], oracle.das(iq[t:t + 1], elem, vox, tx[t:t + 1], **p)) for t in range(T)]
        assert max(db) <= -100.0, (split, db)
