"""Folding through products whose second operand lies [k][n]: groups of rows, one slab of K and more, every tile shape."""
import pytest

pytestmark = pytest.mark.gpu


# (out, in, p, q), 0 = that side absent: one and three groups of 128 and of 256 rows, K of 128 and more, 128 x 128 tiles (four stages of
# slabs; 384 tiles in three columns and 352 in eleven, three; K of 512 and more on few tiles in halves) and 256 x 256 (256 tiles); 192 rows
# of a group stay with the transposing form
@pytest.mark.parametrize("out,inn,p,q", [(128, 128, 128, 0), (256, 512, 0, 512), (512, 256, 512, 0), (128, 608, 0, 608), (128, 1152, 128, 1152), (384, 256, 128, 128), (768, 384, 256, 384), (4096, 1408, 128, 1408), (384, 768, 192, 256),
                                         (16384, 384, 128, 0), (4096, 4096, 4096, 256), (4096, 4096, 256, 4096), (65536, 256, 0, 256)])
def test_fold_bf16(out, inn, p, q):
    import torch
    from paper_2602_17681_amd import binding as ae
    gen = torch.Generator(device="cuda")
    gen.manual_seed(out + inn + p + q)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)      # noqa: E731
    w, b = (rand(out, inn) * inn ** -0.5).bfloat16(), rand(out)
    al, vl = ((rand(p, p) * p ** -0.5).bfloat16(), rand(p)) if p else (None, None)
    ar, vr = ((rand(q, q) * q ** -0.5).bfloat16(), rand(q)) if q else (None, None)
    guard = torch.full((out + 1, inn), 7.0, dtype=torch.bfloat16, device="cuda")
    w_out, b_out = guard[:out], torch.empty(out, device="cuda")
    ws = torch.empty(ae.model_fold_workspace(out, inn, p, q, ae.DTYPES["bf16"]), dtype=torch.uint8, device="cuda")
    ae.model_fold_linear(w, b, out, inn, al, vl, ar, vr, w_out, b_out, ws)
    # a product: one rounding to bfloat16 (2^-9, twice for the binary32 result between two of its values) and k + 1 binary32 ones of partial sums
    ref, err = w.double(), torch.zeros(out, inn, device="cuda", dtype=torch.double)
    if q:
        ref, mag = (ref.view(-1, q) @ ar.double()).view(out, inn), (ref.abs().view(-1, q) @ ar.double().abs()).view(out, inn)
        err = 2.0 ** -8 * ref.abs() + (q + 1) * 2.0 ** -24 * mag
    if p:
        a = al.double()
        left = lambda m, t: torch.matmul(m, t.view(out // p, p, inn)).view(out, inn)      # noqa: E731
        err, mag, ref = left(a.abs(), err), left(a.abs(), ref.abs() + err), left(a, ref)
        err = err + 2.0 ** -8 * (ref.abs() + err) + (p + 1) * 2.0 ** -24 * mag
    assert bool(((w_out.double() - ref).abs() <= err).all())
    assert bool((guard[out] == 7.0).all())
    bias = b.double() if not p else (b.double().view(-1, p) @ al.double().t()).view(-1) + vl.double().repeat(out // p)
    shift = torch.zeros_like(bias) if not q else w_out.double() @ vr.double().repeat(inn // q)
    mag = (w_out.double().abs().sum(1) * (0.0 if not q else vr.abs().max()) + bias.abs() + (0.0 if not p else al.double().abs().sum(1).max() * b.abs().max()))
    # chunks of eight terms in binary32, the rest in binary64
    assert bool(((b_out.double() - (bias - shift)).abs() <= 9 * 2.0 ** -24 * mag).all())
