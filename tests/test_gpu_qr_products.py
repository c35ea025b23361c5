"""The QR calls at sizes with checked, 128-wide and 256 x 128 tiles in the products with a triangle, values and all gradients."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 96, 224, 512, 544, 1024, 1152, 1280])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_qr_against_float64(d, dtype):
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    g, rp, ls, sign, ga = rand(d, d) * d ** -0.5, rand(d, d) * d ** -0.5, 0.3 * rand(d), torch.where(rand(d) < 0, -1.0, 1.0), rand(d, d).to(td)
    a, dg, drp, dls = torch.empty(d, d, device="cuda", dtype=td), torch.empty(d, d, device="cuda"), torch.empty(d, d, device="cuda"), torch.empty(d, device="cuda")
    ws = torch.empty(ae.model_qr_workspace(d, 5), dtype=torch.uint8, device="cuda")
    ae.model_qr_compose(g, rp, ls, sign, d, a, ws, 5)
    ae.model_qr_backward(ga, rp, ls, sign, d, dg, drp, dls, ws, 5)
    g, rp, ls = (t.double().requires_grad_(True) for t in (g, rp, ls))
    x = (g - g.t()) / 64
    q = eye = torch.eye(d, device="cuda", dtype=torch.float64)
    for k in range(12, 0, -1):
        q = eye + x @ q / k
    for _ in range(5):
        q = q @ q
    ref = q @ (torch.triu(rp, 1) + torch.diag_embed(sign.double() * ls.exp()))
    ref.backward(ga.double())
    # the roundings of about six binary32 products at the size of the whole, doubled by every squaring; one rounding of the result to bfloat16
    tol = 6 * 2.0 ** 5 * 2.0 ** -24
    rel = lambda v, r: ((v.double() - r).norm() / r.norm()).item()      # noqa: E731
    assert rel(a, ref.detach()) <= (tol if dtype == "f32" else tol + 2.0 ** -9)
    assert max(rel(dg, g.grad), rel(drp, rp.grad), rel(dls, ls.grad)) <= tol
    assert torch.equal(drp, torch.triu(drp, 1)) and torch.equal(dg, -dg.t())


@pytest.mark.parametrize("d", [32, 96, 512])
def test_sums_of_the_polynomial_keep_their_order(d):
    """Q_0 = ((I + X) + X^2 / 2) + U Y, term by term in binary32: another order of the roundings at the size of the identity costs up to
    4 % of the accuracy at d = 32.  (From the matrices the call leaves in its workspace.)"""
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    squarings = 5
    ws = torch.empty(ae.model_qr_workspace(d, squarings), dtype=torch.uint8, device="cuda")
    ae.model_qr_compose(rand(d, d) * d ** -0.5, rand(d, d) * d ** -0.5, 0.3 * rand(d), torch.ones(d, device="cuda"), d, torch.empty(d, d, device="cuda"), ws, squarings)
    n = 8 + 2 * (squarings + 1) + 6
    slots = ws.view(torch.float32)[:n * d * d].view(n, d, d)
    x, neg_x2, q0, neg_uy = slots[0], slots[1], slots[8], slots[n - 5]
    assert torch.equal(q0, ((torch.eye(d, device="cuda") + x) - 0.5 * neg_x2) - neg_uy)
