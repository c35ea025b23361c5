"""The matrix-core kernels for any channel counts (16-byte chunks of K walked across tap borders) against the oracle, at
the sizes where they can go wrong: channel counts around a chunk, a slab, a column tile; row counts around a row tile;
images narrower than a slab of pixels; the summed-weight forms behind a x2 upsample; split K."""
import pytest

from parity_util import run_case

pytestmark = pytest.mark.gpu

# The tail turns the compared layer's gradient into one that is not constant; conv1:2 keeps its own gradients small.
CASES = [
    # channel counts around a chunk (8 or 4 elements), a slab (32 or 16), the column tiles (32, 64, 128)
    ("in:5x6x7,conv3:33,relu,conv3:1", 3),
    ("in:8x5x9,conv3:31,relu,conv3:17,relu,conv1:3", 2),
    ("in:24x8x8,conv3:65,relu,conv3:129,relu,conv1:2", 2),
    ("in:12x7x5,conv1:40,relu,conv1:130,relu,conv1:7", 4),
    ("in:36x4x4,conv3:96,relu,conv3:12", 3),
    # 127, 128 and 129 rows; one row of one pixel
    ("in:20x1x127,conv3:24,relu,conv1:20", 1),
    ("in:20x8x16,conv3:24,relu,conv1:20", 1),
    ("in:20x3x43,conv3:24,relu,conv1:20", 1),
    ("in:7x1x1,fc:9,relu,fc:5", 1),
    # batch-norm statistics, pooling, the channel in the middle, the summed-weight forms of an upsampled layer
    ("in:3x12x20,conv3:12,bn,relu,pool2,conv3:24,bn,relu,pool2,conv1:6,pnorm,awgn,conv1:24,up2,conv3:12,relu,up2,conv3:3,sigmoid", 3),
    ("in:6x3x5,up2,conv3:20,bn,relu,up2,conv1:9,sigmoid", 2),
    ("in:72x6x6,up2,conv3:56,relu,conv3:64,relu,conv3:40", 2),
    # a long K over few rows (split), and an unaligned fully-connected pair
    ("in:5x9x21,flatten,fc:33,relu,fc:945,relu,reshape:5x9x21,conv3:2", 3),
    # one side aligned to the tiled kernels, the other not
    ("in:64x8x8,conv3:48,relu,conv3:64,relu,conv1:20,relu,conv1:128", 2),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_any_channel_counts(case, dtype):
    spec, batch = CASES[case]
    run_case(spec, batch, dtype=dtype, seed=400 + case, flips=(dtype == "bf16"))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tall_tiles_and_many_splits(dtype):
    # 33,024 rows: the 256-row tiles with a ragged last one; a weight gradient in over a hundred pieces
    run_case("in:12x64x43,conv3:20,relu,conv3:12,relu,conv1:3", 12, dtype=dtype, seed=431, flips=(dtype == "bf16"))


# rows of no whole 16 bytes: more and less than half of a wavefront's columns, a ragged last row tile (of 128 and of 256
# rows), statistics of a batch-norm, the four phases behind an upsample, a sigmoid and its binary32 copy
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("spec,batch", [("in:9x11x13,conv3:99,relu,conv3:101,bn,relu,conv1:57,relu,conv1:35,relu,conv1:27,relu,conv1:3", 3),
                                        ("in:5x64x43,conv3:33,relu,conv1:61,bn,relu,conv1:21,conv1:2", 12),
                                        ("in:6x5x7,up2,conv3:99,relu,up2,conv3:51,sigmoid", 2), ("in:12x7x5,conv1:99,sigmoid,conv1:2", 4),
                                        ("in:64x9x11,conv3:99,relu,conv1:64,relu,conv3:70,bn,relu,conv1:2", 3), ("in:32x64x64,conv1:101,relu,conv1:3", 33)])
def test_stores_of_odd_rows(spec, batch, dtype):
    run_case(spec, batch, dtype=dtype, seed=440 + batch, flips=(dtype == "bf16"))


@pytest.mark.parametrize("tail", ["", ",awgn"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tensors_of_the_caller_off_a_16_byte_border(dtype, tail):
    """x and dy one element into a buffer: the same results, bit for bit, as from aligned copies."""
    import torch
    from paper_2602_17681_amd import binding as ae
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    torch.manual_seed(7)
    B = 200
    m = ae.Model("in:24x1x1,fc:144,relu,fc:40" + tail, B, ae.DTYPES[dtype])
    p = torch.randn(m.n_params, device="cuda") * 0.1
    out = []
    for off in (0, 1):
        x, dy = (torch.empty(B * c + 1, device="cuda", dtype=td)[off:off + B * c] for c in (24, 40))
        torch.manual_seed(8)
        x.copy_(torch.randn(B * 24, device="cuda"))
        dy.copy_(torch.randn(B * 40, device="cuda"))
        y, g = torch.empty(B, 40, device="cuda", dtype=td), torch.empty(m.n_params, device="cuda")
        m.model_forward(p, x, 10.0, 1, y)
        m.model_backward(p, x, dy, g)
        out.append((y.clone(), g.clone()))
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("cin,cout,batch,side", [(64, 64, 4, 8), (68, 132, 3, 7), (128, 96, 28, 16), (128, 96, 29, 16), (256, 256, 16, 16)])
def test_weight_gradient_tiles(cin, cout, batch, side):
    """Binary32 weight gradients of 3x3 layers on tiles of 64 (fewer than 256 workgroups: up to 28 x 16 x 16 pixels of 128 -> 96) and 128."""
    import torch
    from paper_2602_17681_amd import binding as ae
    torch.manual_seed(15)
    m = ae.Model("in:%dx%dx%d,conv3:%d" % (cin, side, side, cout), batch, ae.DTYPES["f32"])
    p, x, dy = torch.zeros(m.n_params, device="cuda"), torch.randn(batch, cin, side, side), torch.randn(batch, cout, side, side)
    y, g = torch.empty(dy.shape, device="cuda"), torch.empty(m.n_params, device="cuda")
    m.model_forward(p, x.cuda(), 10.0, 1, y)
    m.model_backward(p, x.cuda(), dy.cuda(), g)
    ref = torch.nn.grad.conv2d_weight(x.double(), (cout, cin, 3, 3), dy.double(), padding=1)
    # at most 7,424 terms in binary32: sqrt(7424 / 16) roundings of 2^-24 of the growing sum
    assert ((g[:ref.numel()].cpu().double().view_as(ref) - ref).norm() / ref.norm()).item() <= 1.3e-6


@pytest.mark.parametrize("spec,pads", [("in:10x1x1,fc:12", 0), ("in:10x1x1,fc:1200", 1), ("in:8x1x1,fc:10,relu,fc:12", 1)])
def test_no_copy_that_nothing_reads(spec, pads):
    """Inputs with rows that are no whole chunks: copied in the forward pass where its kernel or, for a layer behind the first, the weight gradient reads the copy."""
    import torch
    from paper_2602_17681_amd import binding as ae
    m = ae.Model(spec, 200, ae.DTYPES["f32"])
    p, x, dy = torch.rand(m.n_params, device="cuda"), torch.rand(200, *m.in_shape, device="cuda"), torch.rand(200, *m.out_shape, device="cuda")
    y, g = torch.empty_like(dy), torch.empty(m.n_params, device="cuda")
    m.model_timing_enable(True)
    m.model_forward(p, x, 10.0, 1, y)
    assert sum(r["launches"] for r in m.model_timing_read() if r["name"].endswith("fwd.pad_channels")) == pads
    m.model_backward(p, x, dy, g)
    if ",relu" not in spec:
        ref = dy.flatten(1).double().t() @ x.flatten(1).double()
        assert ((g[:ref.numel()].view_as(ref).double() - ref).norm() / ref.norm()).item() <= 1e-6      # 200 terms in binary32


@pytest.mark.parametrize("c,batch,kernel", [(256, 8, "direct"), (1024, 1, "direct"), (1024, 2, "chunks"), (2048, 8, "chunks"), (192, 9, "chunks")])
def test_weight_gradient_over_a_few_rows(c, batch, kernel):
    import torch
    from paper_2602_17681_amd import binding as ae
    torch.manual_seed(12)
    m = ae.Model("in:%dx1x1,fc:%d" % (c, c), batch, ae.DTYPES["f32"])
    p, x, dy = torch.zeros(m.n_params, device="cuda"), torch.randn(batch, c, device="cuda"), torch.randn(batch, c, device="cuda")
    y, g = torch.empty(batch, c, device="cuda"), torch.empty(m.n_params, device="cuda")
    m.model_timing_enable(True)
    m.model_forward(p, x, 10.0, 1, y)
    m.model_backward(p, x, dy, g)
    assert any(r["name"].endswith("bwd.wgrad_" + kernel) for r in m.model_timing_read())
    ref = dy.double().t() @ x.double()
    assert ((g[:c * c].view(c, c).double() - ref).norm() / ref.norm()).item() <= 2e-7      # at most nine terms in binary32


def test_gradients_by_parts_of_extreme_size():
    """Binary32: a channel whose gradients are all tiny, and an infinity among the activations."""
    import torch
    from paper_2602_17681_amd import binding as ae
    torch.manual_seed(9)
    B, cin, cout = 600, 64, 96
    m = ae.Model("in:%dx1x1,fc:%d" % (cin, cout), B, ae.DTYPES["f32"])
    p = torch.randn(m.n_params, device="cuda") * 0.1
    x, dy = torch.randn(B, cin, device="cuda"), torch.randn(B, cout, device="cuda")
    dy[:, 70] *= 2.0 ** -110
    y, g = torch.empty(B, cout, device="cuda"), torch.empty(m.n_params, device="cuda")
    for bad in (False, True):
        if bad:
            x[5, 3] = float("inf")
            dy[:, 4] = 0.0
        m.model_forward(p, x, 10.0, 1, y)
        m.model_backward(p, x, dy, g)
        got, ref = g[:cin * cout].view(cout, cin).double(), dy.double().t() @ x.double()
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf())
        ok = ref.isfinite()
        err = torch.where(ok, got - ref, 0.0).norm(dim=1) / torch.where(ok, ref, 0.0).norm(dim=1).clamp_min(1e-300)
        # 600 terms in binary32: about sqrt(600 / 16) roundings of 2^-24
        assert err.max().item() <= 1e-6, err.max()


@pytest.mark.parametrize("rest", [-109, -112, -130])
def test_every_weight_gradient_to_its_own_terms(rest):
    """Binary32: a large output gradient meets zero inputs; all there is of a weight's are products of its tiny ones."""
    import torch
    from paper_2602_17681_amd import binding as ae
    B, cin, cout = 256, 64, 96
    m = ae.Model("in:%dx1x1,fc:%d" % (cin, cout), B, ae.DTYPES["f32"])
    p, y, g = torch.zeros(m.n_params, device="cuda"), torch.empty(B, cout, device="cuda"), torch.empty(m.n_params, device="cuda")
    torch.manual_seed(11)
    x, dy = torch.randn(B, cin, device="cuda") * 2.0 ** 60, torch.randn(B, cout, device="cuda")
    dy[1:] *= 2.0 ** rest
    x[0] = 0.0
    m.model_forward(p, x, 10.0, 1, y)
    m.model_backward(p, x, dy, g)
    err = (g[:cin * cout].view(cout, cin).double() - dy.double().t() @ x.double()).abs() / (dy.double().abs().t() @ x.double().abs())
    assert err.max().item() <= 16 * 2.0 ** -24, err.max()          # 256 terms in binary32: sqrt(256) roundings of 2^-24


def test_weight_gradients_beyond_the_range():
    import torch
    from paper_2602_17681_amd import binding as ae
    B, cin, cout = 600, 64, 96
    m = ae.Model("in:%dx1x1,fc:%d" % (cin, cout), B, ae.DTYPES["f32"])
    p, y, g = torch.zeros(m.n_params, device="cuda"), torch.empty(B, cout, device="cuda"), torch.empty(m.n_params, device="cuda")
    torch.manual_seed(10)
    x, dy = torch.randn(B, cin, device="cuda").abs() * 2.0 ** 70, torch.randn(B, cout, device="cuda").abs() * 2.0 ** 70
    for one in (False, True):
        if one:
            dy.zero_()
            # 1.996 x 2^127; the leading parts of both round up, to 2.008 x 2^127
            x[9], dy[9] = (1 + 2.0 ** -8 + 2.0 ** -20) * 2.0 ** 63, 1.98829 * 2.0 ** 64
        m.model_forward(p, x, 10.0, 1, y)
        m.model_backward(p, x, dy, g)
        got, ref = g[:cin * cout].view(cout, cin).double(), dy.double().t() @ x.double()
        assert ((got - ref).abs() <= 2.0 ** -23 * ref).all() if one else got.isposinf().all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["first weight", "second weight", "dy", "x"])
@pytest.mark.parametrize("spec", ["in:12x5x9,conv3:20,conv3:7", "in:12x1x70,conv3:36,conv3:150", "in:20x3x4,up2,conv3:24,up2,conv3:9", "in:168x4x3,conv3:40,conv3:10", "in:60x5x6,conv3:100,conv3:68"])
def test_infinities_at_the_border(spec, where, dtype):
    """Nothing but positive numbers and one infinity: no sum is NaN, and the ones that are infinite are those in which 1e30
    in its place makes itself felt.  The infinite weights are corner taps, the infinite values lie in an image's corner."""
    import torch
    from paper_2602_17681_amd import binding as ae
    import workloads as wl
    td, B = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype], 2
    m = ae.Model(spec, B, ae.DTYPES[dtype])
    weights = [e for e in wl.param_layout(spec)[0] if e["kind"] == "w"]
    torch.manual_seed(14)
    p = 0.1 * torch.rand(m.n_params, device="cuda") + 0.01
    x, dy = (torch.rand(B, *c, device="cuda") + 0.5 for c in (m.in_shape, m.out_shape))
    out = []
    for big in (float("inf"), 1e30):
        v = dict(p=p.clone(), x=x.to(td), dy=dy.to(td))
        if "weight" in where:
            v["p"][weights[where == "second weight"]["offset"]] = big          # channels 0 -> 0, tap (0, 0)
        else:
            v[where].view(-1)[0] = big
        y, g = torch.empty(B, *m.out_shape, device="cuda", dtype=td), torch.empty(m.n_params, device="cuda")
        m.model_forward(v["p"], v["x"], 10.0, 1, y)
        m.model_backward(v["p"], v["x"], v["dy"], g)
        out.append((y.double(), g.double()))
    for got, ref in zip(*out):
        assert not got.isnan().any() and torch.equal(got.isinf(), ref > 1e20), (int(got.isnan().sum()), int(got.isinf().sum()), int((ref > 1e20).sum()))
        ok = got.isfinite()
        # the re-summed outputs add their terms one by one: at most 1512 in binary32, then a rounding to the format per layer
        assert ((got - ref)[ok].abs() <= (1e-4 if dtype == "f32" else 2.0 ** -6) * ref[ok]).all()
