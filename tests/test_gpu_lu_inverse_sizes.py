"""The full-size LU inverse at sizes around a merge of its recursion and a half of the last product's long sums, against float64."""
import pytest

pytestmark = pytest.mark.gpu


# one block; two; the last pair of a level partly or wholly inside the identity padding; an odd number of blocks in the last product; quarters and
# whole tiles in the merges; 4 096 and beyond: 256 x 128 tiles last
@pytest.mark.parametrize("d", [128, 256, 384, 640, 1024, 1152, 2048, 2176, 3200, 4096, 4224])
def test_lu_inverse(d):
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    lp, up, ls, sign = rand(d, d) * d ** -0.5, rand(d, d) * d ** -0.5, 0.3 * rand(d), torch.where(rand(d) < 0, -1.0, 1.0)
    perm = torch.randperm(d, device="cuda", generator=gen).to(torch.int32)
    lp.masked_fill_(torch.ones_like(lp, dtype=torch.bool).triu(), float("nan"))      # neither triangle reads the other
    up.masked_fill_(torch.ones_like(up, dtype=torch.bool).tril(), float("nan"))
    ai = torch.empty(d, d, device="cuda")
    ws = torch.full((ae.model_lu_inverse_workspace(d) // 4,), float("nan"), device="cuda")
    ae.model_lu_inverse(lp, up, ls, sign, perm, d, ai, ws)
    eye = torch.eye(d, device="cuda", dtype=torch.float64)
    L = torch.tril(torch.nan_to_num(lp.double()), -1) + eye
    U = torch.triu(torch.nan_to_num(up.double()), 1) + torch.diag(sign.double() * ls.double().exp())
    Li, Ui = torch.linalg.solve_triangular(L, eye, upper=False, unitriangular=True), torch.linalg.solve_triangular(U, eye, upper=True)
    ref = (Ui @ Li)[:, perm.long()]
    # the merges and the last product: a rounding of 2^-24 of every partial result for each of log2(d / 16) + 1 levels, amplified by the other factor
    amp = torch.linalg.matrix_norm(Ui.abs() @ Li.abs()) / torch.linalg.matrix_norm(ref)
    levels = (d - 1).bit_length() - 3
    assert ((ai.double() - ref).norm() / ref.norm()).item() <= 2.0 ** -24 * levels * max(1.0, amp.item())


@pytest.mark.parametrize("d", [128, 384, 2176])
def test_parameters_off_a_16_byte_border(d):
    """Both inverses read the parameters in place (dword-aligned buffer loads in the merges, single ones in the diagonal blocks): the same
    bits from any 4-byte border, with NaN behind the last entry and in the triangle that is not read."""
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    lp, up, ls, sign, g = rand(d, d) * d ** -0.5, rand(d, d) * d ** -0.5, 0.3 * rand(d), torch.where(rand(d) < 0, -1.0, 1.0), rand(d, d) * d ** -0.5
    perm = torch.randperm(d, device="cuda", generator=gen).to(torch.int32)
    lp.masked_fill_(torch.ones_like(lp, dtype=torch.bool).triu(), float("nan"))
    up.masked_fill_(torch.ones_like(up, dtype=torch.bool).tril(), float("nan"))
    ws = torch.empty(ae.model_lu_inverse_workspace(d), dtype=torch.uint8, device="cuda")
    wq = torch.empty(ae.model_qr_workspace(d, 3), dtype=torch.uint8, device="cuda")
    ae.model_qr_compose(g, up, ls, sign, d, torch.empty(d, d, device="cuda"), wq, 3)

    def moved(t, off):
        buf = torch.full((t.numel() + 8,), float("nan"), device="cuda")
        return buf[off:off + t.numel()].view(t.shape).copy_(t)

    out = []
    for off in range(4):
        ai, qi = torch.empty(d, d, device="cuda"), torch.empty(d, d, device="cuda")
        ae.model_lu_inverse(moved(lp, off), moved(up, off), ls, sign, perm, d, ai, ws)
        ae.model_qr_inverse(moved(up, off), ls, sign, d, wq, qi, ws, 3)
        out.append((ai, qi))
    assert all(bool(torch.isfinite(t).all()) for t in out[0])
    assert all(torch.equal(a, b) for o in out[1:] for a, b in zip(out[0], o))
