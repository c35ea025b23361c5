"""Message bits and error counts over row lengths around the words, units and lane groups of their kernels."""
import numpy as np
import pytest

import oracle.ae_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])            # a buffer on a 16-byte border, and one off it
@pytest.mark.parametrize("batch,k", [(1, 1), (65, 1), (130, 3), (63, 4), (64, 30), (1, 64), (8193, 64), (65, 127), (64, 128),
                                     (33, 129), (7, 260), (300, 1028), (3, 8197), (2, 65532)])
def test_bits_and_counts(batch, k, off):
    import torch
    from paper_2602_17681_amd import binding as ae
    seed, first = 5, (1 << 32) - 3
    buf = torch.full((batch * k + off + 8,), 7.0, device="cuda")
    x = buf[off:off + batch * k].view(batch, k)
    ae.model_gen_bits(seed, first, batch, k, x)
    ref = orc.gen_bits(seed, first, batch, k)
    assert np.array_equal(x.cpu().numpy(), ref)
    assert bool((buf[:off] == 7.0).all()) and bool((buf[off + batch * k:] == 7.0).all())
    rng = np.random.default_rng(k)
    y = (ref > 0).astype(np.float32) * 0.8 + 0.1
    wrong = rng.random((batch, k)) < 1.5 / k       # some rows without an error, some with several
    y[wrong] = 1.0 - y[wrong]
    y[rng.random((batch, k)) < 0.5 / k] = np.nan   # not above the threshold: a 0
    yb = torch.full((batch * k + off,), 7.0, device="cuda")
    yd = yb[off:].view(batch, k)
    yd.copy_(torch.from_numpy(y))
    be = torch.full((1,), 5, dtype=torch.int64, device="cuda")
    ke = torch.full((1,), 6, dtype=torch.int64, device="cuda")
    ae.model_count_errors(yd, x, batch, k, be, ke)
    bad = (y > 0.5) != (ref > 0)
    assert (int(be.item()) - 5, int(ke.item()) - 6) == (int(bad.sum()), int(bad.any(axis=1).sum()))


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("batch,k", [(257, 1), (300, 2), (513, 4), (255, 5), (256, 8), (515, 31), (257, 32), (65, 33)])
def test_bits_of_short_rows(batch, k, off):
    """Row lengths around the kernels for few bits, batches around their workgroups."""
    test_bits_and_counts(batch, k, off)
