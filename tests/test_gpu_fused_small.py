"""The three-launch forward pass of small-image networks: images whose pixels do not fill tiles of 16, channel counts off
multiples of 4, latents with and without 16-byte rows, both workgroup sizes."""
import pytest

import oracle.ae_oracle as orc
import workloads as wl
from parity_util import assert_close, to_dev

pytestmark = pytest.mark.gpu


def _spec(c0, h, w, c1, c2, n, cr, c3, c4):
    return ("in:%dx%dx%d,conv3:%d,bn,relu,pool2,conv3:%d,bn,relu,pool2,flatten,fc:%d,pnorm,awgn,fc:%d,reshape:%dx%dx%d,"
            "up2,conv3:%d,relu,up2,conv3:%d,sigmoid" % (c0, h, w, c1, c2, n, cr * (h // 4) * (w // 4), cr, h // 4, w // 4, c3, c4))


@pytest.mark.parametrize("dims,batch", [((1, 8, 8, 16, 16, 4, 5, 16, 1), 40), ((3, 12, 20, 32, 48, 10, 7, 32, 3), 50),
                                        ((3, 20, 12, 16, 32, 64, 38, 32, 1), 3), ((1, 28, 28, 16, 32, 132, 32, 16, 1), 257),
                                        ((1, 28, 28, 16, 32, 64, 32, 16, 1), 256), ((4, 32, 32, 32, 16, 3, 16, 32, 4), 2)])
def test_small_image_forward(dims, batch):
    import torch
    from paper_2602_17681_amd import binding as ae
    spec = _spec(*dims)
    params = wl.make_params(spec, batch, perturb=True)
    x = wl.make_input(spec, batch, batch)
    y_ref = orc.Net(spec, batch).forward(params, x, snr_db=7.0, seed=batch, first_sample=3)
    m = ae.Model(spec, batch, ae.DTYPES["f32"])
    m.model_set_inference(True)
    m.model_set_sample_offset(3)
    m.model_timing_enable(True)
    y = torch.empty((batch,) + tuple(m.out_shape), device="cuda")
    m.model_forward(to_dev(params, "f32", torch), to_dev(x, "f32", torch), 7.0, batch, y)
    assert [t["name"] for t in m.model_timing_read() if t["launches"]] == ["step00.fwd.fused_small"]
    assert_close(y.cpu().numpy(), y_ref, 1e-4, "y")          # the binary32 tolerance of the whole-network tests


@pytest.mark.parametrize("dims,batch", [((1, 16, 32, 16, 16, 64, 37, 64, 1), 2), ((1, 16, 28, 16, 48, 64, 38, 64, 1), 300),
                                        ((3, 12, 32, 32, 128, 64, 33, 64, 4), 2), ((1, 20, 12, 16, 16, 8, 3, 16, 1), 5),
                                        ((1, 8, 8, 16, 16, 4, 2, 16, 1), 20), ((1, 8, 4, 16, 16, 4, 7, 16, 1), 33)])
def test_small_image_forward_any_reshape(dims, batch):
    """Channels after the reshape off multiples of 4, up to networks that just fit the LDS of the third launch."""
    test_small_image_forward(dims, batch)


@pytest.mark.parametrize("dims,batch", [((1, 28, 28, 16, 32, 64, 32, 16, 1), 1), ((1, 28, 28, 16, 32, 64, 32, 16, 1), 64), ((1, 28, 28, 16, 32, 62, 32, 16, 1), 85),
                                        ((2, 32, 20, 32, 64, 64, 9, 32, 2), 30), ((1, 8, 4, 16, 16, 4, 3, 16, 1), 7), ((1, 12, 24, 16, 128, 8, 4, 16, 1), 128),
                                        # the decoder's fc in whole passes of eight outputs: one of 1 024 threads, four of 512
                                        ((1, 16, 16, 16, 32, 64, 32, 16, 1), 200), ((1, 32, 32, 16, 32, 64, 16, 16, 1), 257)])
def test_small_image_forward_bands(dims, batch):
    """Several workgroups per sample: one to eight bands of rows, of the first two launches up to four (never three)."""
    test_small_image_forward(dims, batch)
