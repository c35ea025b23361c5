"""Column sums (bias gradients and the shift's gradient of a batch-norm) against float64: what rounding they may have."""
import math

import pytest

pytestmark = pytest.mark.gpu


# rows of a block and row lanes of the kernels: 64 and 64, 64 and 21, 32 and 2 (three blocks per compute unit would be 64)
@pytest.mark.parametrize("c,batch,h,w,chain", [(16, 1, 256, 256, 1), (48, 24, 30, 72, 4), (512, 1, 256, 256, 16)])
@pytest.mark.parametrize("layer", ["", ",relu", ",bn,relu"])
def test_rounding_of_column_sums(c, batch, h, w, chain, layer):
    import torch
    from paper_2602_17681_amd import binding as ae
    import workloads as wl
    spec = "in:%dx%dx%d,conv1:%d%s" % (c, h, w, c, layer)
    m = ae.Model(spec, batch, ae.DTYPES["f32"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c)
    p = torch.randn(m.n_params, device="cuda", generator=gen) * 0.01
    ent = {e["kind"]: e for e in wl.param_layout(spec)[0]}
    part = lambda t, kind: t[ent[kind]["offset"]:ent[kind]["offset"] + c]     # noqa: E731
    part(p, "b").fill_(1.0)
    if "bn" in layer:                              # every output above zero: the sums are those of dy
        part(p, "gamma").fill_(0.1)
        part(p, "beta").fill_(10.0)
    x = torch.rand(batch, c, h, w, device="cuda", generator=gen)
    if not layer:
        p.zero_()
    elif "bn" not in layer:
        p[:c * c].zero_()
    dy = torch.randn(batch, c, h, w, device="cuda", generator=gen)
    y, g = torch.empty_like(dy), torch.empty_like(p)
    m.model_forward(p, x, 10.0, 1, y)
    assert not layer or bool((y > 0).all())
    m.model_backward(p, x, dy, g)
    rows = batch * h * w
    err = part(g, "beta" if "bn" in layer else "b").double() - dy.double().sum(dim=(0, 2, 3))
    # Terms of variance 1.  An addition with a result of variance i rounds by 2^-24 sqrt(i) / sqrt(3) at most (root of the mean
    # square): i = 2 .. chain in a thread, (chain + 1) / 2 a row on average; the block's sum and the whole one are rounded
    # once each, 1 a row: sqrt(((chain + 1) / 2 + 2) / 3) 2^-24 sqrt(rows).
    bound = math.sqrt(((chain + 1) / 2 * (chain > 1) + 2) / 3) * 2.0 ** -24 * math.sqrt(rows)
    rms = float(err.square().mean().sqrt())
    print("%s: %.2e of %.2e" % (spec, rms / math.sqrt(rows), bound / math.sqrt(rows)))
    assert rms <= bound
