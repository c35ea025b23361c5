"""The batched small-matrix calls at sizes around a 32-wide tile, a 16-wide block of the inversion and the wide loads (d no
multiple of four, matrices that start off a 16-byte border), with a permutation that names a row twice and one out of range."""
import pytest
import torch

from paper_2602_17681_amd import binding as ae

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("count,d", [(1, 1), (3, 2), (2, 15), (2, 17), (3, 31), (2, 33), (2, 47), (5, 63), (2, 65), (3, 96), (2, 97), (300, 128)])
def test_sizes(count, d, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)      # noqa: E731
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    lp, up, ls = rnd(count, d, d) * d ** -0.5, rnd(count, d, d) * d ** -0.5, 0.3 * rnd(count, d)
    sign = torch.where(rnd(count, d) < 0, -1.0, 1.0)
    perm = torch.argsort(torch.rand(count, d, device="cuda", generator=g), dim=1).to(torch.int32)
    if d > 4:
        perm[-1, 3] = d                       # out of range: read as 3, which another entry names too
    gr = rnd(count, d, d).to(td)
    a, ai = torch.empty(count, d, d, device="cuda", dtype=td), torch.empty(count, d, d, device="cuda", dtype=td)
    dlp, dup, dls = torch.empty(count, d, d, device="cuda"), torch.empty(count, d, d, device="cuda"), torch.empty(count, d, device="cuda")
    ae.model_lu_compose_batch(lp, up, ls, sign, perm, count, d, a)
    ae.model_lu_backward_batch(gr, lp, up, ls, sign, perm, count, d, dlp, dup, dls)
    ae.model_lu_inverse_batch(lp, up, ls, sign, perm, count, d, ai)
    p = perm.long()
    p = torch.where(p < d, p, torch.arange(d, device="cuda"))
    s = sign.double() * ls.double().exp()
    L = torch.tril(lp.double(), -1) + torch.eye(d, device="cuda", dtype=torch.float64)
    U = torch.triu(up.double(), 1) + torch.diag_embed(s)
    A = torch.stack([(L[i] @ U[i])[p[i]] for i in range(count)])
    inv = torch.linalg.inv(L @ U)
    Ai = torch.stack([inv[i][:, p[i]] for i in range(count)])
    # K <= 128 terms in binary32, once rounded to the storage type; the inverse goes through the growth of two triangles
    tol = 3e-7 if dtype == "f32" else 3e-3
    rel = lambda x, r: ((x.double() - r).norm() / r.norm().clamp_min(1e-300)).item()      # noqa: E731
    assert rel(a, A) <= tol and rel(ai, Ai) <= 4 * tol, (rel(a, A), rel(ai, Ai))
    ok = count if d <= 4 else count - 1       # (which of two rows with the same name wins is not defined)
    B = torch.zeros_like(L)
    for i in range(ok):
        B[i][p[i]] = gr[i].double()
    dU, dL = L.transpose(1, 2).contiguous() @ B, B @ U.transpose(1, 2).contiguous()
    if ok:
        assert rel(dls[:ok], torch.diagonal(dU, dim1=1, dim2=2)[:ok] * s[:ok]) <= 5e-7
    if ok and d > 1:
        assert rel(dup[:ok], torch.triu(dU, 1)[:ok]) <= 5e-7 and rel(dlp[:ok], torch.tril(dL, -1)[:ok]) <= 5e-7
    assert torch.equal(dup, torch.triu(dup, 1)) and torch.equal(dlp, torch.tril(dlp, -1))


def test_full_size_inverse_takes_parameters_off_a_16_byte_border():
    d = 256
    torch.manual_seed(5)
    par = [torch.randn(d, d, device="cuda") * d ** -0.5, torch.randn(d, d, device="cuda") * d ** -0.5, 0.3 * torch.randn(d, device="cuda")]
    sign, perm = torch.ones(d, device="cuda"), torch.randperm(d, device="cuda").to(torch.int32)
    ws = torch.empty(ae.model_lu_inverse_workspace(d), dtype=torch.uint8, device="cuda")
    out = []
    for off in (0, 1):
        lp, up = (torch.empty(d * d + 1, device="cuda")[off:off + d * d].view(d, d).copy_(p) for p in par[:2])
        ai = torch.empty(d, d, device="cuda")
        ae.model_lu_inverse(lp, up, par[2], sign, perm, d, ai, ws)
        out.append(ai)
    assert torch.equal(*out)


def compose(lp, up, ls, sign, perm):
    """All matrices in one call, or each in a call of its own where they are too large for that."""
    n, d = ls.shape
    a = torch.empty(n, d, d, device="cuda")
    if d <= 128:
        ae.model_lu_compose_batch(lp, up, ls, sign, perm, n, d, a)
    else:
        ws = torch.empty(ae.model_lu_workspace(d, ae.DTYPES["f32"]), dtype=torch.uint8, device="cuda")
        for i in range(n):
            ae.model_lu_compose(lp[i], up[i], ls[i], sign[i], perm[i], d, a[i], ws)
    return a


@pytest.mark.parametrize("d", [33, 64, 97, 128, 160, 256, 1056])
def test_the_large_term_is_rounded_once(d):
    """Small off-diagonal entries beside a diagonal of ones: the results with the diagonal in them are off by their own rounding."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    n, eye = 64 if d <= 128 else 4, torch.eye(d, device="cuda", dtype=torch.float64)
    lp, up = (0.2 / d ** 0.5 * torch.randn(n, d, d, device="cuda", generator=g) for _ in range(2))
    perm = torch.arange(d, device="cuda", dtype=torch.int32).repeat(n, 1)
    a = compose(lp, up, torch.zeros(n, d, device="cuda"), torch.ones(n, d, device="cuda"), perm)
    ref = torch.diagonal((torch.tril(lp.double(), -1) + eye) @ (torch.triu(up.double(), 1) + eye).contiguous(), dim1=1, dim2=2)
    err = ((torch.diagonal(a, dim1=1, dim2=2).double() - ref).abs() / ref.abs()).max().item()
    assert err <= 1.1 * 2.0 ** -24, err * 2 ** 24        # half a last place; the other terms add up to 1e-2 of the result


@pytest.mark.parametrize("d,i,j", [(2, 1, 0), (40, 39, 20), (128, 70, 69), (160, 150, 3), (256, 255, 0), (256, 130, 129)])
@pytest.mark.parametrize("which", ["L", "U"])
def test_an_infinity_enters_one_row_or_column_of_the_product(d, i, j, which):
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    rnd = lambda *s: torch.randn(1, *s, device="cuda", generator=g)      # noqa: E731
    lp, up, ls = rnd(d, d) * d ** -0.5, rnd(d, d) * d ** -0.5, 0.3 * rnd(d)
    perm = torch.randperm(d, device="cuda", generator=g).to(torch.int32)[None]
    out = []
    for value in (float("inf"), 0.0):
        (lp[0] if which == "L" else up[0].t())[i, j] = value
        a = torch.empty(d, d, device="cuda")
        a[perm[0].long()] = compose(lp, up, ls, torch.ones(1, d, device="cuda"), perm)[0]         # rows as in L U
        bad = a[i, j:] if which == "L" else a[j:, i]       # L[i, j] U[j, j:], L[j:, j] U[j, i]
        out.append((bad.clone(), a))
        bad.zero_()
    assert not out[0][0].isfinite().any() and out[1][0].isfinite().all()
    assert (out[0][1] - out[1][1]).norm() <= 1e-6 * out[1][1].norm()


@pytest.mark.parametrize("which", ["L", "U"])
@pytest.mark.parametrize("d,i,j", [(2, 1, 0), (16, 15, 8), (24, 20, 3), (40, 39, 1), (64, 63, 32), (100, 99, 50), (128, 5, 2), (128, 127, 64), (128, 70, 20), (256, 5, 2), (256, 127, 64), (256, 250, 130)])
def test_an_infinity_stays_in_its_columns_and_rows(d, i, j, which):
    """An infinite entry (i, j) of L enters columns up to j of its inverse, one (j, i) of U rows up to j: the others are what
    they are with a zero in its place."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)      # noqa: E731
    lp, up, ls = rnd(d, d) * d ** -0.5, rnd(d, d) * d ** -0.5, 0.3 * rnd(d)
    sign, perm = torch.ones(d, device="cuda"), torch.randperm(d, device="cuda", generator=g).to(torch.int32)
    out = []
    for value in (float("inf"), 0.0):
        (lp if which == "L" else up.t())[i, j] = value
        ai = torch.empty(d, d, device="cuda")
        if d <= 128:
            ae.model_lu_inverse_batch(lp, up, ls, sign, perm, 1, d, ai)
        else:
            ae.model_lu_inverse(lp, up, ls, sign, perm, d, ai, torch.empty(ae.model_lu_inverse_workspace(d), dtype=torch.uint8, device="cuda"))
        out.append(ai[:, perm.long() > j] if which == "L" else ai[j + 1:])
    assert torch.equal(*out) or ((out[0] - out[1]).norm() <= 1e-6 * out[1].norm()).item()
