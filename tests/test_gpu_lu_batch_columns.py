"""The batched inverse with one, two and four blocks of 32 columns per workgroup: sizes around a block, parameters off a 16-byte border,
an infinite entry."""
import pytest
import torch

from paper_2602_17681_amd import binding as ae

pytestmark = pytest.mark.gpu


# matrices: 1 block (up to 256 workgroups), 2 and 4 (beyond), for 4, 3 and 2 blocks of columns in all; d = 97 and 33 leave a block nearly empty
@pytest.mark.parametrize("count,d", [(64, 128), (65, 128), (128, 97), (129, 128), (129, 101), (86, 96), (129, 96), (128, 64), (129, 64), (200, 33), (260, 30)])
@pytest.mark.parametrize("off", [0, 1])
def test_columns_per_workgroup(count, d, off):
    g = torch.Generator(device="cuda")
    g.manual_seed(count + d)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)      # noqa: E731
    lp, up = (torch.empty(count * d * d + 1, device="cuda")[off:off + count * d * d].view(count, d, d).copy_(rnd(count, d, d) * d ** -0.5) for _ in range(2))
    ls, sign = 0.3 * rnd(count, d), torch.where(rnd(count, d) < 0, -1.0, 1.0)
    perm = torch.argsort(torch.rand(count, d, device="cuda", generator=g), dim=1).to(torch.int32)
    ai = torch.empty(count, d, d, device="cuda")
    ae.model_lu_inverse_batch(lp, up, ls, sign, perm, count, d, ai)
    L = torch.tril(lp.double(), -1) + torch.eye(d, device="cuda", dtype=torch.float64)
    U = torch.triu(up.double(), 1) + torch.diag_embed(sign.double() * ls.double().exp())
    ref = torch.gather(torch.linalg.inv(L @ U), 2, perm.long()[:, None, :].expand(-1, d, -1))
    # substitution is backward stable: d roundings of 2^-24 at the size of |A^-1| |L| |U| |A^-1|
    bound = d * 2.0 ** -24 * (torch.linalg.inv(U).abs() @ (U.abs() @ (torch.linalg.inv(U).abs() @ torch.linalg.inv(L).abs())) +
                              torch.linalg.inv(U).abs() @ (torch.linalg.inv(L).abs() @ (L.abs() @ torch.linalg.inv(L).abs())))
    bound = torch.gather(bound, 2, perm.long()[:, None, :].expand(-1, d, -1))
    assert bool(((ai.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("count,d,i,j", [(65, 128, 100, 40), (65, 128, 39, 33), (129, 128, 100, 40), (129, 128, 127, 0), (129, 96, 39, 33)])
@pytest.mark.parametrize("which", ["L", "U"])
def test_an_infinity_stays_in_its_columns_and_rows(count, d, i, j, which):
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)      # noqa: E731
    lp, up, ls = rnd(count, d, d) * d ** -0.5, rnd(count, d, d) * d ** -0.5, 0.3 * rnd(count, d)
    sign, perm = torch.ones(count, d, device="cuda"), torch.randperm(d, device="cuda", generator=g).to(torch.int32).repeat(count, 1)
    out = []
    for value in (float("inf"), 0.0):
        (lp if which == "L" else up.transpose(1, 2))[:, i, j] = value
        ai = torch.empty(count, d, d, device="cuda")
        ae.model_lu_inverse_batch(lp, up, ls, sign, perm, count, d, ai)
        out.append(ai[:, :, perm[0].long() > j] if which == "L" else ai[:, j + 1:])
    assert ((out[0] - out[1]).norm() <= 1e-6 * out[1].norm()).item()


# the infinity sends whole columns through the sums that are taken again
@pytest.mark.parametrize("count,d", [(129, 128), (129, 97), (65, 128), (129, 64)])
@pytest.mark.parametrize("special", [0.0, float("inf")])
def test_a_matrix_does_not_depend_on_how_many_there_are(count, d, special):
    """Two and four blocks of columns per workgroup (a wavefront or two per 16 columns) against one (four): the same sums, the same bits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(count * d)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)      # noqa: E731
    lp, up, ls = rnd(count, d, d) * d ** -0.5, rnd(count, d, d) * d ** -0.5, 0.3 * rnd(count, d)
    if special:
        lp[:, d - 8, d // 3] = special
    sign, perm = torch.where(rnd(count, d) < 0, -1.0, 1.0), torch.argsort(torch.rand(count, d, device="cuda", generator=g), dim=1).to(torch.int32)
    many, few = torch.empty(count, d, d, device="cuda"), torch.empty(count, d, d, device="cuda")
    ae.model_lu_inverse_batch(lp, up, ls, sign, perm, count, d, many)
    for i in range(0, count, 32):
        n, s = min(32, count - i), slice(i, min(count, i + 32))
        ae.model_lu_inverse_batch(lp[s], up[s], ls[s], sign[s], perm[s], n, d, few[s])
    assert torch.equal(torch.nan_to_num(many, nan=123.0), torch.nan_to_num(few, nan=123.0))
    assert bool(torch.isfinite(many).all()) == (special == 0.0)
