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


def test_column_sums_of_a_launch_of_many_tiles():
    """Batch statistics behind a dense product large enough for the 256-row tiles: the sums stay one block per 128 rows."""
    run_case("in:1024x16x16,conv1:512,bn,relu,conv1:2", 33, dtype="f32", seed=440, flips=True, backward=False)
