"""Short passes between the layers: the channel step of a sample by several workgroups, layout changes by pieces and by
thin matrices, and the gradients that leave few partial sums, at lengths that divide by nothing."""
import pytest

from parity_util import run_case

pytestmark = pytest.mark.gpu


# latents of 1 365 and 2 079 values (no whole quads: the last one is cut) and of 1 372 and 2 604 (whole quads, short last share), by
# one workgroup per sample from 257 samples on
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("spec,batch", [("in:7x15x13,conv1:7,pnorm,awgn,conv1:5", 3), ("in:5x9x11,conv1:21,pnorm,awgn,conv1:3", 24),
                                        ("in:7x14x14,conv1:7,pnorm,awgn,conv1:5", 2), ("in:3x14x31,conv1:6,pnorm,awgn,conv1:2", 1),
                                        ("in:2x15x13,conv1:7,pnorm,awgn,conv1:2", 256), ("in:2x15x13,conv1:7,pnorm,awgn,conv1:2", 257)])
def test_channel_step_in_shares(spec, batch, dtype):
    run_case(spec, batch, dtype=dtype, seed=500 + batch, flips=(dtype == "bf16"))


# channels x pixels: whole tiles of 64 x 64, 64 x 16, 16 x 64, the general tile, up to four rows or columns
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c,h,w,batch", [(64, 16, 8, 3), (128, 4, 4, 2), (192, 4, 12, 1), (16, 8, 8, 5), (48, 16, 8, 2), (33, 9, 5, 2),
                                         (2, 7, 300, 3), (3, 16, 16, 2), (4, 1, 1025, 2), (40, 1, 3, 7), (520, 2, 2, 2), (64, 7, 9, 2)])
def test_layout_changes(c, h, w, batch, dtype, off):
    """An identity 1x1 layer: what comes out is the input, bit for bit (a product with 1 and zeros is exact), through the
    layout change on either side; the gradient comes back the same way."""
    import torch
    from paper_2602_17681_amd import binding as ae
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    m = ae.Model("in:%dx%dx%d,conv1:%d" % (c, h, w, c), batch, ae.DTYPES[dtype])
    p = torch.zeros(m.n_params, device="cuda")
    p[:c * c].view(c, c).fill_diagonal_(1.0)
    torch.manual_seed(c)
    n = batch * c * h * w
    x = torch.empty(n + 1, device="cuda", dtype=td)[off:off + n].view(batch, c, h, w)
    y = torch.full((n + 9,), 7.0, device="cuda", dtype=td)
    x.copy_(torch.randn(batch, c, h, w, device="cuda"))
    m.model_forward(p, x, 10.0, 1, y[off:off + n].view(batch, c, h, w))
    assert torch.equal(y[off:off + n].view(batch, c, h, w), x)
    assert bool((y[:off] == 7.0).all()) and bool((y[off + n:] == 7.0).all())


@pytest.mark.parametrize("c,rows", [(2048, 5), (2049, 120), (40, 16), (4096, 2100)])
def test_bias_gradients_of_few_partial_sums(c, rows):
    """Column sums of a few rows of many columns and of many of a few, against float64: a binary32 sum of blocks of at most
    256 rows, combined in double and rounded once."""
    import torch
    from paper_2602_17681_amd import binding as ae
    m = ae.Model("in:8x1x1,fc:%d" % c, rows, ae.DTYPES["f32"])
    torch.manual_seed(c)
    p, x, dy = torch.zeros(m.n_params, device="cuda"), torch.randn(rows, 8, device="cuda"), torch.randn(rows, c, device="cuda")
    y, g = torch.empty_like(dy), torch.empty(m.n_params, device="cuda")
    m.model_forward(p, x, 10.0, 1, y)
    m.model_backward(p, x, dy, g)
    bound = 257 * 2.0 ** -24 * dy.double().abs().sum(0)
    assert bool(((g[8 * c:].double() - dy.double().sum(0)).abs() <= bound).all())
