"""Weight gradient of tensors with infinities and NaN: they reach the gradients that have them as terms, and no others."""

import pytest
import torch

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")


def reference(x, dy, dims):
    """dw [cout, 27, cin], db in float64, term by term; outside the volume the input is zero."""
    D, H, W = dims
    x = torch.nn.functional.pad(x.double().view(D, H, W, -1), (0, 0, 1, 1, 1, 1, 1, 1))
    g = dy.double().view(D, H, W, -1)
    dw = torch.empty((g.shape[3], 27, x.shape[3]), dtype=torch.float64, device="cuda")
    for tap in range(27):
        z, y, u = tap // 9, tap // 3 % 3, tap % 3
        dw[:, tap] = (g[..., :, None] * x[z:z + D, y:y + H, u:u + W, None, :]).sum((0, 1, 2))
    return dw, g.sum((0, 1, 2))


# (dims, non-finite inputs (z, y, x, channel, value), non-finite gradients): the volume's sides, its inside, and the places
# where rows longer than 128 voxels are cut; 64 x 2 x 2 takes its axes in another order
CASES = [((2, 3, 20), [(1, 1, 0, 3, INF)], []), ((2, 3, 20), [(0, 2, 19, 5, NAN), (1, 0, 0, 5, -INF)], []),
         ((3, 4, 9), [(1, 2, 4, 0, INF)], [(2, 3, 8, 7, -INF)]), ((1, 2, 300), [(0, 1, 0, 2, INF)], [(0, 0, 100, 4, INF), (0, 1, 200, 9, NAN)]),
         ((1, 3, 258), [], [(0, 1, 128, 1, INF), (0, 1, 129, 2, INF)]), ((64, 2, 2), [(5, 0, 1, 6, INF), (0, 1, 0, 8, NAN)], []),
         ((2, 2, 2), [], [])]


@pytest.mark.parametrize("dims,xs,gs", CASES)
def test_infinities_reach_their_own_terms_only(dims, xs, gs):
    from paper_2604_06257_amd import learn
    g = torch.Generator(device="cuda").manual_seed(dims[2])
    V = dims[0] * dims[1] * dims[2]
    x, dy = (torch.randn(V, 16, generator=g, device="cuda").bfloat16() for _ in range(2))
    for t, places in ((x, xs), (dy, gs)):
        for z, y, u, c, value in places:
            t.view(*dims, 16)[z, y, u, c] = value
    dw, db = torch.empty(16 * 27 * 16, device="cuda"), torch.empty(16, device="cuda")
    work = torch.empty(learn.wgrad_work_floats(dims, 16, 16, 1024), device="cuda")
    learn.conv3d_wgrad(x, dy, dw, db, work, dims, 1024)
    for got, want in zip((dw.view(16, 27, 16).double(), db.double()), reference(x, dy, dims)):
        assert torch.equal(got.isnan(), want.isnan())
        assert torch.equal(got == INF, want == INF) and torch.equal(got == -INF, want == -INF)
        ok = want.isfinite()
        # sums of up to 774 products of unit scale in float32: 1e-5 of the largest, as for finite tensors
        assert (got[ok] - want[ok]).abs().max() <= 1e-5 * max(1.0, want[ok].abs().max().item())


def check(dims, xs, gs, chunk):
    from paper_2604_06257_amd import learn
    g = torch.Generator(device="cuda").manual_seed(sum(dims) + chunk)
    V = dims[0] * dims[1] * dims[2]
    x, dy = (torch.randn(V, 16, generator=g, device="cuda").bfloat16() for _ in range(2))
    for t, places in ((x, xs), (dy, gs)):
        for z, y, u, c, value in places:
            t.view(*dims, 16)[z, y, u, c] = value
    dw, db = torch.empty(16 * 27 * 16, device="cuda"), torch.empty(16, device="cuda")
    work = torch.empty(learn.wgrad_work_floats(dims, 16, 16, chunk), device="cuda")
    learn.conv3d_wgrad(x, dy, dw, db, work, dims, chunk)
    for got, want in zip((dw.view(16, 27, 16).double(), db.double()), reference(x, dy, dims)):
        assert torch.equal(got.isnan(), want.isnan())
        assert torch.equal(got == INF, want == INF) and torch.equal(got == -INF, want == -INF)
        ok = want.isfinite()
        # float32 sums of V products of unit scale: sqrt(V) 2^-24 each a few times over, against a largest of about 3 sqrt(V)
        assert (got[ok] - want[ok]).abs().max() <= 1e-5 * max(1.0, want[ok].abs().max().item())


# (rows longer than 128 voxels are cut into blocks of columns; 64 x 2 x 2 takes its axes in another order)
@pytest.mark.parametrize("dims", [(2, 3, 5), (1, 9, 130), (64, 2, 2), (9, 30, 40)])
def test_gradients_at_the_volumes_sides(dims):
    """A gradient of the first or last column, in every row and slice: its outer taps meet the input's padding."""
    rows = [(z, y) for z in range(min(dims[0], 3)) for y in range(min(dims[1], 5))]
    for z, y in rows + [(dims[0] - 1, dims[1] - 1)]:
        for u in (0, dims[2] - 1):
            for chunk in (64, 1024):
                check(dims, [], [(z, y, u, 5, INF)], chunk)


@pytest.mark.parametrize("dims", [(9, 30, 40), (40, 17, 9), (3, 33, 260), (300, 2, 5)])
def test_inputs_whose_outer_taps_are_formed_again(dims):
    """Side columns of some blocks hold infinities, so that some parts' sums are formed again and the others kept."""
    D, H, W = dims
    check(dims, [(0, 0, 0, 3, INF), (D - 1, H - 1, W - 1, 7, -INF), (D // 2, H // 2, 0, 9, NAN), (D // 2, 1, W - 1, 9, INF),
                 (D // 3, 0, W // 2, 12, INF)], [], 64)
    check(dims, [(D // 2, H // 2, W - 1, 3, INF)], [(D // 3, 0, 0, 2, INF), (D // 3, 0, W // 2, 4, -INF)], 512)
