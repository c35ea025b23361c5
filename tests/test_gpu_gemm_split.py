"""Dense binary32 products by bfloat16 parts: tile and K edges, and the operands that the parts cannot hold."""
import pytest
import torch

from paper_2602_17681_amd import binding as ae
from parity_util import run_case

pytestmark = pytest.mark.gpu


def product(e, a, v=None):
    out = torch.empty(e.shape[0], a.shape[0], device="cuda")
    ae.model_fold_embedding(e, e.shape[0], e.shape[1], a, v if v is not None else torch.zeros(a.shape[0], device="cuda"), out)
    return out


def rand(*shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(*shape, device="cuda", generator=g)


# rows around a 128-row tile and over 256 tiles of 256 rows; K of one odd slab, an odd and an even number of slabs
@pytest.mark.parametrize("rows,d", [(1, 80), (127, 528), (128, 512), (129, 1040), (300, 96), (16384, 1024), (16385, 1024), (700, 2000)])
def test_edges(rows, d):
    e, a, v = rand(rows, d, seed=1), rand(d, d, seed=2), rand(d, seed=3)
    r = e.double() @ a.double().t() + v.double()
    # a K of 16 rounds the sum once (2^-24 of a partial sum that grows like sqrt(k)): sqrt(d / 16) 2^-24 at most
    err = ((product(e, a, v).double() - r).norm() / r.norm()).item()
    assert err <= 2 * (d / 16) ** 0.5 * 2.0 ** -24 + 2.0 ** -23, err


@pytest.mark.parametrize("scale", [2.0 ** -120, 2.0 ** -100, 2.0 ** 100])
def test_rows_of_extreme_size(scale):
    e, a = rand(256, 512, seed=4), rand(512, 512, seed=5)
    e[7] *= scale
    if scale > 1:
        a[3] *= 2.0 ** -90
    r = e.double() @ a.double().t()
    err = ((product(e, a).double() - r).norm(dim=1) / r.norm(dim=1)).max().item()
    assert err <= 1e-6, err


@pytest.mark.parametrize("first,rest,w", [(0, -109, 60), (0, -112, 60), (0, -126, 60), (0, -140, 60), (-100, -130, 60), (-63, -63, -63)])
def test_every_output_to_its_own_terms(first, rest, w):
    """Rows whose large first element meets zeros: all there is of an output are products of their tiny elements."""
    e, a = rand(130, 256, seed=10), rand(256, 256, seed=11) * 2.0 ** w
    e[:, :1] *= 2.0 ** first
    e[:, 1:] *= 2.0 ** rest
    a[:, 0] = 0.0
    err = (product(e, a).double() - e.double() @ a.double().t()).abs() / (e.double().abs() @ a.double().abs().t())
    # 256 terms in binary32: sqrt(256) roundings of 2^-24
    assert err.max().item() <= 16 * 2.0 ** -24, err.max()


def test_infinities_nan_and_the_largest_values():
    e, a = rand(384, 512, seed=6).round() + 0.5, rand(512, 512, seed=7).round() + 0.5      # bf16 values: their lower parts are zero
    e[5, 17] = float("inf")
    e[140, 3] = float("nan")
    a[200, 40] = -float("inf")
    e[300, 9], a[:, 9] = 3.4e38, 0.5                                                      # rounds to a bfloat16 infinity
    e[300, :9], e[300, 10:] = 0.0, 0.0
    got, ref = product(e, a), e.double() @ a.double().t()
    assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isposinf(), ref.isposinf()) and torch.equal(got.isneginf(), ref.isneginf())
    ok = ref.isfinite()
    assert (got.double() - ref)[ok].abs().max() <= 1e-6 * ref[ok].abs().max()
    assert (got.double() - ref)[300][ok[300]].abs().max() <= 1e-6 * 1.7e38


def test_sums_beyond_the_range():
    e, a = rand(130, 512, seed=8).abs() * 2.0 ** 70, rand(512, 512, seed=9).abs() * 2.0 ** 70
    assert product(e, a).isposinf().all()
    e.zero_()
    e[:, 9], a[:, 9] = (1 + 2.0 ** -8 + 2.0 ** -20) * 2.0 ** 63, 1.98829 * 2.0 ** 64       # 1.996 x 2^127; both round up to 2.008 x 2^127
    ref = e.double() @ a.double().t()
    assert ((product(e, a).double() - ref).abs() <= 2.0 ** -23 * ref).all()


# few tiles and a long K (split K, ragged tiles); tiles that all lie inside; behind an upsample as four phases and with the
# stride-2 input gradient; behind an upsample with few tiles (no phases)
@pytest.mark.parametrize("wide,hw,up,cout", [(64, (6, 10), 0, 96), (32, (32, 64), 0, 128), (32, (64, 32), 1, 64), (48, (3, 5), 1, 64)])
def test_convolutions_of_operands_that_the_parts_cannot_hold(wide, hw, up, cout):
    """A sample of tiny inputs and one of tiny output gradients, then infinities: every sample's outputs and input gradients and
    the tiny sample's own weight gradients to their size.  The first layer's weight gradients of input channel n are those
    of sample n, the only one with something in that channel."""
    B, (h, w) = 4, hw
    m = ae.Model("in:%dx%dx%d,conv1:%d,%sconv3:%d" % (B, h, w, wide, "up2," if up else "", cout), B, ae.DTYPES["f32"])
    torch.manual_seed(13)
    w1, w2 = torch.randn(wide, B, 1, 1), torch.randn(cout, wide, 3, 3)
    p = torch.cat([w1.flatten(), torch.zeros(wide), w2.flatten(), torch.zeros(cout)]).cuda()
    x = torch.eye(B).view(B, B, 1, 1) * torch.rand(B, B, h, w)
    dy = torch.randn(B, cout, h << up, w << up)
    x[1] *= 2.0 ** -120
    dy[2] *= 2.0 ** -120
    dy[[0, 2, 3], 5] = 0.0
    rel = lambda a, r: ((a - r).norm() / r.norm()).item()      # noqa: E731
    # sums of at most 32,768 terms in binary32: sqrt(32768 / 16) roundings of 2^-24 of the growing sum, 2.7e-6
    tol = 3e-6
    for infinite in ("", "x", "dy"):
        xi, dyi = x.clone(), dy.clone()
        if infinite == "x":
            xi[3, 3, 0, 0] = float("inf")
        if infinite == "dy":
            dyi[0, 7, 0, 0] = float("inf")
        r1, r2 = w1.double().requires_grad_(), w2.double().requires_grad_()
        z = torch.nn.functional.conv2d(xi.double(), r1)
        ry = torch.nn.functional.conv2d(torch.nn.functional.interpolate(z, scale_factor=2) if up else z, r2, padding=1)
        ry.backward(dyi.double())
        y, g = torch.empty(dy.shape, device="cuda"), torch.empty(m.n_params, device="cuda")
        m.model_timing_enable(True)
        m.model_forward(p, xi.cuda(), 10.0, 1, y)
        m.model_backward(p, xi.cuda(), dyi.cuda(), g)
        names = [r["name"] for r in m.model_timing_read()]
        y, g1, g2 = y.cpu().double(), g[:w1.numel()].view(w1.shape).cpu().double(), g[w1.numel() + wide:-cout].view(w2.shape).cpu().double()
        sound = [n for n in range(B) if infinite != "x" or n != 3]
        err = [rel(y[n], ry[n]) for n in sound]
        if infinite != "dy":
            err += [rel(g1[:, n], r1.grad[:, n]) for n in sound]
        if infinite == "":
            err += [rel(g2[5], r2.grad[5]), rel(g2, r2.grad)]
        if infinite == "x":
            assert torch.equal(y[3].isfinite(), ry[3].isfinite()) and torch.equal(g1[:, 3].isfinite(), r1.grad[:, 3].isfinite())
        if infinite == "dy":
            rows = [c for c in range(cout) if c != 7]
            err += [rel(g2[rows], r2.grad[rows]), rel(g2[5], r2.grad[5])]
            assert not g2[7].isfinite().all()
        assert max(err) <= tol and all(e == e for e in err), (infinite, err)
    assert any("fwd.conv_mfma" in n for n in names) and any("bwd.dgrad_mfma" in n for n in names) and any("bwd.wgrad_chunks" in n for n in names)


def test_column_sums_of_a_launch_of_many_tiles():
    """Batch statistics behind a dense product large enough for the 256-row tiles: the sums stay one block per 128 rows."""
    run_case("in:1024x16x16,conv1:512,bn,relu,conv1:2", 33, dtype="f32", seed=440, flips=True, backward=False)
