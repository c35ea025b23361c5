"""A 1-4-channel first layer with a sigmoid and nothing else behind it, in bfloat16: the sigmoid's backward pass reads a
binary32 copy of its output, which the thin-layer kernels do not write."""
import pytest

from parity_util import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_first_layer_with_a_sigmoid(dtype):
    run_case("in:2x8x8,conv3:16,sigmoid,conv1:8,relu,conv3:2", 3, dtype=dtype, seed=310, flips=(dtype == "bf16"))
