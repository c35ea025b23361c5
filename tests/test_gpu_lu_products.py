"""The full-size LU compose and backward pass at sizes of either product form, on one stream and two, with a permutation out of range."""
import pytest

pytestmark = pytest.mark.gpu


# d off 128: transposed operands, checked tiles (8 224: of 256 rows); 128 .. : operands as they lie, 128 x 128 tiles; 4 096: 256 x 128; 8 192:
# 256 x 256; a second stream from 2 048 (binary32: 1 024) on
@pytest.mark.parametrize("d,dtype", [(96, "bf16"), (128, "bf16"), (160, "bf16"), (640, "bf16"), (1024, "bf16"), (2048, "bf16"), (4096, "bf16"), (8192, "bf16"), (8224, "bf16"), (64, "f32"), (96, "f32"), (992, "f32"), (1024, "f32")])
def test_lu_step(d, dtype):
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    lp, up, ls, sign, g = rand(d, d) * d ** -0.5, rand(d, d) * d ** -0.5, 0.3 * rand(d), torch.where(rand(d) < 0, -1.0, 1.0), rand(d, d).to(td)
    perm = torch.randperm(d, device="cuda", generator=gen).to(torch.int32)
    i = int((perm == d - 1).nonzero())
    perm[[i, d - 1]] = perm[[d - 1, i]]
    perm[d - 1] = d + 7                            # out of range: read as d - 1, which no other entry names
    a, dlp, dup, dls = torch.empty(d, d, device="cuda", dtype=td), torch.empty(d, d, device="cuda"), torch.empty(d, d, device="cuda"), torch.empty(d, device="cuda")
    ws = torch.empty(ae.model_lu_workspace(d, ae.DTYPES[dtype]), dtype=torch.uint8, device="cuda")
    ae.model_lu_compose(lp, up, ls, sign, perm, d, a, ws)
    ae.model_lu_backward(g, lp, up, ls, sign, perm, d, dlp, dup, dls, ws)
    p = perm.long().clamp_max(d - 1)
    s = sign.double() * ls.double().exp()
    L, U = torch.tril(lp.double(), -1) + torch.eye(d, device="cuda", dtype=torch.float64), torch.triu(up.double(), 1) + torch.diag(s)
    B = torch.zeros_like(L)
    B[p] = g.double()
    dU, dL = L.t().contiguous() @ B, B @ U.t().contiguous()
    # operands and results rounded to the storage type (2^-9 each: three of them), the sums in binary32
    tol = 3 * 2.0 ** -9 if dtype == "bf16" else 2.0 ** -24 * d ** 0.5
    rel = lambda x, r: ((x.double() - r).norm() / r.norm()).item()      # noqa: E731
    assert rel(a, (L @ U)[p]) <= tol
    assert rel(dup, torch.triu(dU, 1)) <= tol and rel(dlp, torch.tril(dL, -1)) <= tol and rel(dls, torch.diagonal(dU) * s) <= tol
    assert torch.equal(dup, torch.triu(dup, 1)) and torch.equal(dlp, torch.tril(dlp, -1))


@pytest.mark.parametrize("d,dtype", [(96, "bf16"), (256, "bf16"), (2048, "bf16"), (256, "f32")])
def test_timed_products_are_those_of_untimed_calls(d, dtype):
    """While the products are timed the same kernels run on the same operands: the workspaces hold the same bits, operand for operand.  One
    product of the inverse is timed, the last."""
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    lp, up, ls, sign, g = rand(d, d) * d ** -0.5, rand(d, d) * d ** -0.5, 0.3 * rand(d), torch.ones(d, device="cuda"), rand(d, d).to(td)
    perm = torch.randperm(d, device="cuda", generator=gen).to(torch.int32)
    a, dlp, dup, dls = torch.empty(d, d, device="cuda", dtype=td), torch.empty(d, d, device="cuda"), torch.empty(d, d, device="cuda"), torch.empty(d, device="cuda")
    calls = [(1, ae.model_lu_workspace(d, ae.DTYPES[dtype]), lambda ws: ae.model_lu_compose(lp, up, ls, sign, perm, d, a, ws)),
             (2, ae.model_lu_workspace(d, ae.DTYPES[dtype]), lambda ws: ae.model_lu_backward(g, lp, up, ls, sign, perm, d, dlp, dup, dls, ws))]
    if d % 128 == 0:
        calls.append((1, ae.model_lu_inverse_workspace(d), lambda ws: ae.model_lu_inverse(lp, up, ls, sign, perm, d, a, ws)))
    for products, size, call in calls:
        plain, timed = torch.zeros(size, dtype=torch.uint8, device="cuda"), torch.zeros(size, dtype=torch.uint8, device="cuda")
        call(plain)
        ae.model_lu_timing(True)
        call(timed)
        ms, n = ae.model_lu_timing(False)
        assert n == products and ms > 0.0
        assert torch.equal(plain, timed)
