"""Plans whose windows hold many rows (scattered points, coarse grids): lanes gather their samples instead of staging the
windows.  Against the FP64 oracle; odd and even frame counts in chunks of 1 to 8, IQ types, several transmits, both ends of
the record, elements at several depths, per-transmit output.
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


def scattered(n, seed, depth=(5e-3, 45e-3)):
    r = np.random.default_rng(seed)
    return np.stack([r.uniform(-12e-3, 12e-3, n), r.uniform(-2e-3, 2e-3, n), r.uniform(*depth, n)], 1).astype(np.float32)


def run(iq, elem, vox, tx, kind="c64", t0=0.0, f_number=0.8, per_tx=False):
    x = torch.from_numpy(iq)
    if kind != "c64":
        x = torch.view_as_real(x).to(torch.float16 if kind == "f16" else torch.bfloat16).contiguous()
        iq = x.float().numpy().view(np.complex64)[..., 0]
    T, E, S, F = iq.shape
    p = das.Params(T, E, S, F, vox.shape[0], C, FS, FD, t0, f_number, 0.5)
    with das.Plan(p, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (elem, vox, tx))) as plan:
        assert plan.info()["kernel"][1] == -1
        y = (plan.execute_per_tx if per_tx else plan.execute)(x.cuda()).cpu().numpy()
    o = dict(c=C, fs=FS, fd=FD, t0=t0, f_number=f_number, tukey_alpha=0.5)
    if not per_tx:
        return oracle.nrmse_db(y, oracle.das(iq, elem, vox, tx, **o))
    return max(oracle.nrmse_db(y[t], oracle.das(iq[t:t + 1], elem, vox, tx[t:t + 1], **o)) for t in range(T))


@pytest.mark.parametrize("kind", ["c64", "f16", "bf16"])
@pytest.mark.parametrize("F,T", [(1, 1), (1, 5), (2, 1), (3, 2), (4, 1), (7, 1), (8, 2), (9, 1), (17, 3), (40, 1)])
def test_scattered_points(F, T, kind):
    vox = scattered(700, F)
    elem = linear_array(15, 0.6e-3)
    tx = np.stack([vox[:, 2] / C + 3e-7 * t for t in range(T)]).astype(np.float32)
    assert run(random_iq((T, 15, 1300, F), seed=F), elem, vox, tx, kind) <= -100.0


@pytest.mark.parametrize("F", [1, 3, 8, 13])
def test_both_record_ends_and_no_apodization(F):
    """A 300-row record inside the points' 1000 rows: rows -1 and 299, coordinates on either side."""
    vox = scattered(500, 50 + F)
    elem = linear_array(6, 0.6e-3)
    tx = (vox[None, :, 2] / C).astype(np.float32)
    u = (tx[0, :, None] + np.linalg.norm(vox[:, None].astype(np.float64) - elem[None], axis=-1) / C) * FS
    # the row before the record and its last row are both used
    t0 = next(b for b in range(300, 700) if (np.floor(u) == b - 1).any() and (np.floor(u) == b + 299).any()) / FS
    assert run(random_iq((1, 6, 300, F), seed=F), elem, vox, tx, t0=t0, f_number=0.0) <= -100.0


@pytest.mark.parametrize("F,T", [(1, 4), (2, 3), (1, 1)])
def test_per_transmit_output(F, T):
    vox = scattered(600, 90 + F)
    elem = linear_array(13, 0.6e-3)
    tx = np.stack([vox[:, 2] / C + 3e-7 * t for t in range(T)]).astype(np.float32)
    assert run(random_iq((T, 13, 1300, F), seed=F), elem, vox, tx, per_tx=True) <= -100.0


def test_per_transmit_output_of_small_launches_with_many_frames():
    """Small launches take 1 or 2 frames a chunk, for which per-transmit output is served: also where gathering takes 8."""
    vox = scattered(900, 7)
    elem = linear_array(9, 0.6e-3)
    tx = np.stack([vox[:, 2] / C, vox[:, 2] / C + 3e-7]).astype(np.float32)
    assert run(random_iq((2, 9, 1300, 21), seed=3), elem, vox, tx, per_tx=True) <= -100.0


def test_elements_at_several_depths():
    vox = scattered(700, 3)
    elem = linear_array(17, 0.6e-3)
    elem[:, 2] = (-elem[:, 0].astype(np.float64) ** 2 / 20e-3).astype(np.float32)
    tx = (vox[None, :, 2] / C).astype(np.float32)
    assert run(random_iq((1, 17, 1300, 5), seed=3), elem, vox, tx) <= -100.0


def test_unused_samples_and_unused_pairs_do_not_reach_the_output():
    """NaN in every sample that no active pair reads."""
    vox = scattered(300, 11)
    elem = linear_array(8, 0.6e-3)
    tx = (vox[None, :, 2] / C).astype(np.float32)
    iq = random_iq((1, 8, 1300, 3), seed=5)
    d = vox[:, None].astype(np.float64) - elem[None]
    u = (tx[0, :, None] + np.linalg.norm(d, axis=-1) / C) * FS
    active = 2 * 0.8 * np.hypot(d[..., 0], d[..., 1]) < 1.001 * d[..., 2]
    used = np.zeros((8, 1300), bool)
    for e in range(8):
        for k in np.floor(u[active[:, e], e]).astype(int):
            used[e, max(0, k - 1):k + 3] = True  # a row of margin
    iq[0][~used] = np.nan
    p = das.Params(1, 8, 1300, 3, 300, C, FS, FD, 0.0, 0.8, 0.5)
    with das.Plan(p, *(torch.from_numpy(a).cuda() for a in (elem, vox, tx))) as plan:
        assert plan.info()["kernel"][1] == -1
        y = plan.execute(torch.from_numpy(iq).cuda()).cpu().numpy()
    assert np.isfinite(y).all()
