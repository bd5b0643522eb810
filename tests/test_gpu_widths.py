"""Hidden widths that end inside a 128-byte slice of the matrix mainloop (64 bfloat16 or 32
float32 values): the last slice of the logits reads zeros past d instead of the next row's
values.  Compared with the float64 oracle at the bars of helpers.py.  (The shards of the first
test run on the streamed 128 x 64 tiles; test_gpu_tiles.py has part slices on every other.)"""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_grad_close, assert_loss_close, compare_all, run_gpu, run_oracle, to_device

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


# What lies behind a row is not read into its products, though zeros of the other operand would
# meet it: beside NaN or infinite tokens, and with NaN behind the last row of H and of a shard,
# the other tokens' results are as they are without them.  The tiles of few tokens (64 and 128
# wide), the large ones, and the residual's on 128 x 64, 128 x 128 and 256 x 256.
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("T,d,rows", [(40, 72, [700, 200]), (230, 2672, [21915]), (1333, 456, [9000, 4000]),
                                      (1333, 360, [9000, 4000])])
@pytest.mark.parametrize("name", ["tiny_f32_T256_d256_V2048_P8", "bf16_T4096_d2880_V201088_P8"])
def test_neighbours_stay_out_of_a_part_slice(name, T, d, rows, value):
    import torch

    import paper_2609_14306_amd as vp

    inp = wl.resplit(wl.make_inputs(name, T=T, d=d, V=sum(rows), P=1, seed=97), rows)
    g = wl.random_grad_loss(T, 97, "random")
    ref = run_oracle(inp, g)
    H, Ws, t = to_device(inp)
    H[1::4] = value

    def in_a_buffer(x):  # the same rows with NaN behind the last one
        buf = torch.full((x.shape[0] + 1, d), float("nan"), dtype=x.dtype, device="cuda")
        buf[:-1] = x
        return buf[:-1]

    H, Ws = in_a_buffer(H), [in_a_buffer(w) for w in Ws]
    loss, lse = vp.forward(H, Ws, t, inp.ignore_index)
    dH, _ = vp.backward(H, Ws, t, lse, torch.from_numpy(g).cuda(), inp.ignore_index)
    ok = np.arange(T) % 4 != 1
    what = f"{name} T={T} d={d} {value}"
    assert_loss_close(inp.dtype, lse.cpu().numpy()[ok], ref["lse"][ok], what + " lse")
    assert_loss_close(inp.dtype, loss.cpu().numpy()[ok], ref["loss"][ok], what + " loss")
    assert_grad_close(inp.dtype, dH.cpu().numpy()[ok], ref["dH"][ok], what + " dH")
    assert bool(torch.isnan(lse).cpu().numpy()[~ok].all())
