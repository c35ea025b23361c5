"""Big fully-connected layers of bf16 models, multiplied straight from the binary32 parameters: row counts around the
tiles, splits of K, parameters off 16-byte borders, against float64 and against the packed copies."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["", ",relu"])
@pytest.mark.parametrize("batch,k,n,off", [(1, 1024, 1024, 0), (3, 8192, 128, 1), (31, 128, 8192, 0), (129, 1152, 1024, 3),
                                           (300, 4096, 384, 0), (512, 1024, 1280, 2), (513, 1024, 1024, 0)])
def test_forward(batch, k, n, off, act):
    import torch
    from paper_2602_17681_amd import binding as ae
    m = ae.Model("in:%dx1x1,fc:%d%s" % (k, n, act), batch, ae.DTYPES["bf16"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    p = torch.randn(m.n_params + off, device="cuda", generator=gen)[off:]
    x = torch.randn(batch, k, device="cuda", generator=gen).bfloat16()
    y = torch.full((batch + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")      # (a row behind the output)
    m.model_forward(p, x, 10.0, 1, y[:batch])
    w, b = p[:k * n].view(n, k).bfloat16().double(), p[k * n:].double()
    ref = x.double() @ w.t() + b
    if act:
        ref = ref.clamp(min=0.0)
    # one rounding to bfloat16 (2^-9, twice for the binary32 sum between two of its values), k + 1 binary32 roundings of partial sums
    mag = x.double().abs() @ w.abs().t() + b.abs()
    assert bool(((y[:batch].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + (k + 1) * 2.0 ** -24 * mag).all())
    assert bool((y[batch:] == 7.0).all())


@pytest.mark.parametrize("batch,k,latent", [(1, 8192, 128), (37, 8192, 256), (130, 2048, 640)])
def test_input_gradient(batch, k, latent):
    """The second layer's input gradient shows in the first layer's gradients: against the packed weights, which hold the
    same values (both sum in binary32 and round to bfloat16 once)."""
    import torch
    from paper_2602_17681_amd import binding as ae
    spec = "in:%dx1x1,fc:%d,pnorm,awgn,fc:%d" % (k, latent, k)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(latent)
    x = torch.randn(batch, k, device="cuda", generator=gen).bfloat16()
    dy = torch.randn(batch, k, device="cuda", generator=gen).bfloat16()
    out = []
    for packed in (False, True):
        m = ae.Model(spec, batch, ae.DTYPES["bf16"])
        m.model_set_params_static(packed)
        gen.manual_seed(1)
        p = torch.randn(m.n_params, device="cuda", generator=gen) * k ** -0.5
        y, g = torch.empty_like(x), torch.empty(m.n_params, device="cuda")
        m.model_forward(p, x, 10.0, 1, y)
        m.model_backward(p, x, dy, g)
        out.append((y.double(), g[:k * latent].double(), g[k * latent:].double()))
    # a binary32 sum in another order moves a stored bfloat16 value by one place (2^-8) now and then: far below one place in the 2-norm
    for a, b in zip(*out):
        assert float((a - b).norm()) <= 2.0 ** -9 * float(b.norm())


@pytest.mark.parametrize("batch,k,latent", [(1, 8192, 128), (37, 8192, 256), (130, 2048, 640), (512, 1024, 1024)])
def test_input_gradient_itself(batch, k, latent):
    """Noise hands the second layer's input gradient on unchanged, and with unit vectors as inputs the first layer's weight
    gradient holds it column by column: against float64; and that it was the kernels for the parameters themselves, which
    static parameters do not take."""
    import torch
    from paper_2602_17681_amd import binding as ae
    spec = "in:%dx1x1,fc:%d,awgn,fc:%d" % (k, latent, k)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(latent)
    x = torch.eye(batch, k, device="cuda").bfloat16()
    dy = torch.randn(batch, k, device="cuda", generator=gen).bfloat16()
    for static in (False, True):
        m = ae.Model(spec, batch, ae.DTYPES["bf16"])
        m.model_set_params_static(static)
        gen.manual_seed(1)
        p = torch.randn(m.n_params, device="cuda", generator=gen)
        y, g = torch.empty_like(x), torch.empty(m.n_params, device="cuda")
        m.model_timing_enable(True)
        m.model_forward(p, x, 10.0, 1, y)
        m.model_backward(p, x, dy, g)
        names = [t["name"].split(".", 1)[1] for t in m.model_timing_read() if t["launches"]]
        assert (names.count("fwd.fc"), names.count("bwd.fc_dgrad")) == ((0, 0) if static else (2, 1)), names
        w2 = p[k * latent + latent:][:k * latent].view(k, latent).bfloat16().double()
        ref = dy.double() @ w2
        dz = g[:k * latent].view(latent, k)[:, :batch].t().double()
        # one rounding to bfloat16 (2^-9, twice for the binary32 sum between two of its values), k + 1 binary32 roundings of partial sums
        mag = dy.double().abs() @ w2.abs()
        assert bool(((dz - ref).abs() <= 2.0 ** -8 * ref.abs() + (k + 1) * 2.0 ** -24 * mag).all())
        assert bool((g[:k * latent].view(latent, k)[:, batch:] == 0).all())
