"""The backward pass as it schedules itself, on two streams and on one: the same gradients, below and above the line between them."""
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("net,side,batch,dtype", [("cfg2", 16, 8, "f32"), ("cfg2", 32, 96, "f32"), ("cfg5", 64, 2, "bf16"), ("cfg5", 128, 10, "bf16")])
def test_same_gradients(net, side, batch, dtype):
    import torch
    from paper_2602_17681_amd import binding as ae
    spec, td = wl.scaled_spec(net, side), {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    out = []
    for overlap in (None, True, False):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(side)
        m = ae.Model(spec, batch, ae.DTYPES[dtype])
        if overlap is not None:
            m.model_set_overlap(overlap)
        p = 0.05 * torch.randn(m.n_params, device="cuda", generator=gen)
        x = torch.rand(batch, *m.in_shape, device="cuda", generator=gen).to(td)
        y, dy, loss = torch.empty(batch, *m.out_shape, device="cuda", dtype=td), torch.empty(batch, *m.out_shape, device="cuda", dtype=td), torch.empty(1, device="cuda")
        grads = torch.full((m.n_params,), float("nan"), device="cuda")
        for step in range(3):                      # (steps that follow one another share the buffers and the second stream)
            m.model_forward(p, x, 10.0, step, y)
            ae.model_loss_mse(y, x, loss, dy)
            m.model_backward(p, x, dy, grads)
        out.append((y.clone(), grads.clone()))
    assert bool(torch.isfinite(out[0][1]).all())
    assert all(torch.equal(a, b) for o in out[1:] for a, b in zip(out[0], o))


@pytest.mark.parametrize("net,side,batch,dtype,two", [("cfg2", 16, 8, "f32", False), ("cfg2", 32, 96, "f32", True), ("cfg5", 64, 2, "bf16", False), ("cfg5", 128, 10, "bf16", True)])
def test_streams(net, side, batch, dtype, two):
    """One stream or two by default, whatever is asked for with 0 and 1, and the default again with -1."""
    import torch
    from paper_2602_17681_amd import binding as ae
    import parity_util as pu
    spec, td = wl.scaled_spec(net, side), {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    m = ae.Model(spec, batch, ae.DTYPES[dtype])
    p, x = 0.05 * torch.randn(m.n_params, device="cuda"), torch.rand(batch, *m.in_shape, device="cuda").to(td)
    y, dy, grads = torch.empty(batch, *m.out_shape, device="cuda", dtype=td), torch.rand(batch, *m.out_shape, device="cuda").to(td), torch.empty(m.n_params, device="cuda")
    m.model_forward(p, x, 10.0, 1, y)
    for on, expected in ((None, two), (True, True), (False, False), (-1, two), (1, True), (-1, two)):
        if on is not None:
            m.model_set_overlap(on)
        m.model_backward(p, x, dy, grads)
        assert pu.captured_branches(lambda: m.model_backward(p, x, dy, grads)) == expected, on
    m.close()
