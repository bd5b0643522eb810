"""Hidden widths that end inside a 128-byte slice of the matrix mainloop (64 bfloat16 or 32
float32 values): the last slice of the logits reads zeros past d instead of the next row's
values.  Compared with the float64 oracle at the bars of helpers.py."""
import pytest

import workloads as wl
from helpers import compare_all, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


# 8: one chunk is all there is; 56, 120: one (bf16) chunk short of whole slices; 72: one chunk
# past a slice; 1000: many slices and a tail of five (bf16) or two (f32) chunks.
@pytest.mark.parametrize("d", [8, 56, 72, 120, 1000])
@pytest.mark.parametrize("name", ["tiny_f32_T256_d256_V2048_P8", "bf16_T4096_d2880_V201088_P8"])
def test_width_inside_a_slice(name, d):
    inp = wl.make_inputs(name, T=270, d=d, V=900, P=1, seed=47)
    inp = wl.resplit(inp, [300, 77, 523], order=[1, 2, 0])
    g = wl.random_grad_loss(inp.T, 47, "random")
    compare_all(inp, run_gpu(inp, g), run_oracle(inp, g), f"{inp.dtype} d={d}")
