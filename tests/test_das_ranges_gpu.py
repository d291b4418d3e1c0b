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


@pytest.mark.parametrize("late", [0.0625, 0.25, -0.25, 40.0])
@pytest.mark.parametrize("T,F,per_tx", [(1, 1, False), (2, 3, False), (3, 2, True)])
def test_any_time_base_keeps_the_staged_kernel(late, T, F, per_tx):
    """Arrival times and t0 on an absolute time base: millions of rows and carrier cycles, few of them between the two."""
    elem = linear_array(9, 0.3e-3)
    vox = column()
    tx = np.stack([np.float32(late) + (vox[:, 2] / C + 1e-7 * t).astype(np.float32) for t in range(T)]).astype(np.float32)
    kernel, db = run(random_iq((T, 9, 700, F), seed=11), elem, vox, tx, t0=late, per_tx=per_tx)
    assert kernel != GENERAL and db <= -100.0


@pytest.mark.parametrize("row,t0", [(0, 0.0), (150_000, 0.0), (598_700, 0.0), (598_700, 0.3), (-10, 0.0)])
@pytest.mark.parametrize("T,F", [(1, 1), (2, 7)])
def test_long_records_keep_the_staged_kernel(row, t0, T, F):
    """A 600,000-row record of which a plan uses some rows: at its beginning (partly before it), within it, at its end (partly
    past it)."""
    elem = linear_array(4, 0.3e-3)
    vox = column(step=3e-4)
    tx = np.stack([np.float32(t0) + (vox[:, 2] / C + 1e-7 * t + row / FS).astype(np.float32) for t in range(T)]).astype(np.float32)
    kernel, db = run(random_iq((T, 4, 600_000, F), seed=row + T + 20), elem, vox, tx, t0=t0)
    assert kernel != GENERAL and db <= -100.0


@pytest.mark.parametrize("f_number", [0.0, 0.8])
def test_points_far_outside_the_record_keep_the_staged_kernel(f_number):
    """Points and arrival times so far away that their sample coordinates leave the fixed point: exact zeros there, the
    others' sums as without them, in the same waves."""
    elem = linear_array(5, 0.3e-3)
    vox = column(128)
    tx = (vox[None, :, 2] / C).astype(np.float32)
    vox[3::8, 2] = 1e4                        # 1.3e8 rows
    vox[4::8, 0] = -3e7
    vox[5::16, 2] = 2e19                      # the square of the distance is infinite in float32
    tx[0, 6::16] = np.float32(3e38)
    tx[0, 7::16] = np.float32(-3e38)
    tx[0, 14::16] = 1.0
    tx[0, 15::16] = -0.05
    iq = random_iq((1, 5, 900, 3), seed=7)
    p = das.Params(1, 5, 900, 3, 128, C, FS, FD, 0.0, f_number, 0.5)
    with das.Plan(p, *(torch.from_numpy(a).cuda() for a in (elem, vox, tx))) as plan:
        kernel = plan.info()["kernel"]
        y = plan.execute(torch.from_numpy(iq).cuda()).cpu().numpy()
    near = np.ones(128, bool)
    for first, step in ((3, 8), (4, 8), (5, 16), (6, 16), (7, 16), (14, 16), (15, 16)):
        near[first::step] = False
    ref = oracle.das(iq, elem, vox[near], tx[:, near], c=C, fs=FS, fd=FD, t0=0.0, f_number=f_number, tukey_alpha=0.5)
    assert kernel != GENERAL and np.abs(ref).min() > 0
    assert np.all(y[~near] == 0) and oracle.nrmse_db(y[near], ref) <= -100.0


def test_high_carrier_in_a_slowly_sampled_record():
    """More carrier cycles than rows: 60 a row over 20,000 rows do not fit the fixed point, 20 do."""
    elem = linear_array(4, 0.3e-3)
    vox = column(step=1e-2, z0=0.1)
    tx = (vox[None, :, 2] / C).astype(np.float32)
    iq = random_iq((1, 4, 20_000, 2), seed=9)
    for cycles, general in ((20, False), (60, True)):
        kernel, db = run(iq, elem, vox, tx + np.float32(0.5), t0=0.5, fs=2e6, fd=2e6 * cycles)
        assert (kernel == GENERAL) == general and db <= -100.0


@pytest.mark.parametrize("T,F,per_tx", [(1, 1, False), (3, 2, True), (2, 9, False)])
def test_lists_of_too_many_items_take_the_general_kernel(T, F, per_tx, monkeypatch):
    """Three wave tiles of 33 elements and up to 3 transmits: at least 49 pairs of items, at most a few hundred."""
    elem = linear_array(33, 0.3e-3)
    vox = column(n=192, z0=9e-3, step=1e-5)
    tx = np.stack([(vox[:, 2] / C + 1e-7 * t).astype(np.float32) for t in range(T)])
    iq = random_iq((T, 33, 700, F), seed=12)
    for pairs, general in ((20, True), (10_000, False)):
        monkeypatch.setenv("DAS_ITEMS", str(pairs))
        kernel, db = run(iq, elem, vox, tx, per_tx=per_tx)
        assert (kernel == GENERAL) == general and db <= -100.0


def test_item_lists_beyond_32_bits_keep_the_staged_kernel():
    """2.4e9 work items (39 GB): 2,344 wave tiles that see every one of 16,384 x 64 (element, transmit) pairs."""
    T, E, S, V = 64, 16_384, 64, 150_000
    g = torch.Generator(device="cuda").manual_seed(5)
    elem = torch.rand((E, 3), generator=g, device="cuda") * 1e-3
    elem[:, 2] = 0
    vox = torch.rand((V, 3), generator=g, device="cuda") * 1e-3 + torch.tensor([0.0, 0.0, 1e-3], device="cuda")
    tx = (torch.rand((T, 1), generator=g, device="cuda") * 1e-7 + vox[None, :, 2] / C).float()
    iq = torch.randn((T, E, S, 1, 2), generator=g, device="cuda").half()
    p = das.Params(T, E, S, 1, V, C, FS, FD, 0.0, 0.0, 0.5)
    with das.Plan(p, elem, vox, tx) as plan:
        info = plan.info()
        y = plan.execute(iq).to(torch.complex128)[:, 0]
    assert info["kernel"] != GENERAL and info["active_triples"] == V * E * T
    idx = torch.randperm(V, generator=g, device="cuda")[:192].sort().values
    ref = torch.zeros(192, dtype=torch.complex128, device="cuda")
    q = torch.view_as_complex(iq[:, :, :, 0].double())
    for n, v in enumerate(idx):
        tau = tx[:, v].double()[:, None] + (vox[v].double() - elem.double()).norm(dim=1)[None] / C
        u = tau * FS
        i0 = u.floor().long()[..., None]
        beta = u - u.floor()
        s = torch.lerp(q.gather(2, i0)[..., 0], q.gather(2, i0 + 1)[..., 0], beta.to(torch.complex128))
        ref[n] = (s * torch.polar(torch.ones_like(tau), 2 * np.pi * FD * tau)).sum()
    # 65,536 float32 additions a group, sums growing with the root of their number: 2^-24 * 256 = -96 dB
    assert oracle.nrmse_db(y[idx].cpu().numpy(), ref.cpu().numpy()) <= -90.0


@pytest.mark.parametrize("T,E", [(4096, 3), (4097, 3), (16_384, 2), (1, 5000), (3, 16_385)])
def test_many_transmits_or_elements_keep_the_staged_kernel(T, E):
    elem = np.zeros((E, 3), np.float32)
    elem[:, 0] = np.linspace(-1e-3, 1e-3, E)
    vox = column(70)
    tx = (vox[None, :, 2] / C + 1e-7 * np.arange(T)[:, None] / T).astype(np.float32)
    kernel, db = run(random_iq((T, E, 220, 1), seed=T), elem, vox, tx)
    assert kernel != GENERAL and db <= -100.0
