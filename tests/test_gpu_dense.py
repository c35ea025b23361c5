"""Dense bf16 products in check-free tiles: row lengths from one slab of the load pipeline up, every tile shape."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = 65536


# columns: 256 x 256 tiles (eight wavefronts), 256 x 128, 128 x 128; K: 1 .. 5 slabs of 32 and a longer run
@pytest.mark.parametrize("cols", [256, 384, 128])
@pytest.mark.parametrize("k", [32, 64, 96, 128, 160, 448])
def test_dense_bf16(cols, k):
    import torch
    from paper_2602_17681_amd import binding as ae
    m = ae.Model("in:%dx1x1,fc:%d" % (k, cols), ROWS, ae.DTYPES["bf16"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k + cols)
    p = torch.randn(m.n_params, device="cuda", generator=gen)
    x = torch.randn(ROWS, k, device="cuda", generator=gen).bfloat16()
    y = torch.empty(ROWS, cols, dtype=torch.bfloat16, device="cuda")
    m.model_set_inference(True)
    m.model_forward(p, x, 10.0, 1, y)
    w, b = p[:cols * k].view(cols, k).bfloat16().double(), p[cols * k:].double()
    ref = x.double() @ w.t() + b
    # one rounding to bfloat16 (2^-9, twice for the binary32 result between two of its values), k + 1 binary32 roundings of partial sums
    mag = x.double().abs() @ w.abs().t() + b.abs()
    assert bool(((y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + (k + 1) * 2.0 ** -24 * mag).all())


# 128 x 128: 256, 784 and 1 008 tiles and 384 in one column (four stages of slabs), 352, 576 in one column and 729 (three);
# 256 x 128: 576 tiles in nine columns, up to K = 96 in the one kernel and beyond in the other
@pytest.mark.parametrize("rows,cols", [(2048, 2048), (2816, 2048), (3456, 3456), (3584, 3584), (8064, 2048), (49152, 128), (73728, 128), (16384, 1152)])
@pytest.mark.parametrize("k", [32, 64, 96, 128, 160, 448])
def test_dense_bf16_tile_counts(rows, cols, k, monkeypatch):
    monkeypatch.setitem(globals(), "ROWS", rows)
    test_dense_bf16(cols, k)
