"""How the backward is cut: token counts and widths around its tiles, several shards in one
strip (ragged, and next to ones that keep a strip of their own), shards cut into pieces and
tokens into chunks by a small strip budget, dH sums in one and in many jobs, and dW added to.
Whole gradients against the float64 oracle at the bars of helpers.py."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_grad_close, compare_all, run_gpu, run_oracle, to_device

pytestmark = pytest.mark.gpu

F32, BF16 = "tiny_f32_T256_d256_V2048_P8", "bf16_T4096_d2880_V201088_P8"

CASES = [
    # T, d, shard rows, order, strip_elems
    (63, 72, [300, 256, 257, 255, 700], [4, 1, 0, 3, 2], 0),       # joined and lone shards
    (129, 136, [256] * 20, list(range(20)), 0),                    # more shards than a strip takes
    (200, 264, [30000], [0], 0),                                   # one segment in many jobs
    (200, 320, [2600, 900, 1100], [2, 0, 1], 256 * 1024),          # shards cut into pieces
    (257, 1000, [700, 3001], [1, 0], 0),                           # few shards in several jobs
    (1100, 520, [9000, 300, 5000], [0, 1, 2], 0),                  # large tiles (bfloat16)
    (2048, 264, [6000, 7000], [1, 0], 0),
    (700, 136, [300, 260], [1, 0], 256 * 2048),                    # joined shards, two token chunks
]


@pytest.mark.parametrize("T,d,rows,order,strip", CASES)
@pytest.mark.parametrize("name", [F32, BF16])
def test_few_token_gradients(name, T, d, rows, order, strip):
    inp = wl.make_inputs(name, T=T, d=d, V=sum(rows), P=1, seed=59)
    inp = wl.resplit(inp, rows, order=order)
    g = wl.random_grad_loss(T, 59, "random")
    compare_all(inp, run_gpu(inp, g, strip_elems=strip), run_oracle(inp, g), f"{inp.dtype} T={T} d={d}")


# Many tokens on transposed copies of W and H, with several shards in a strip: in float32 each
# shard's sum is added to dH by itself.
@pytest.mark.parametrize("name,T,d,rows", [(BF16, 20480, 512, [5120, 5119, 5110, 5000]),
                                           (F32, 10240, 4096, [2560, 2500, 2559, 2560])])
def test_many_tokens_on_joined_shards(name, T, d, rows):
    inp = wl.make_inputs(name, T=T, d=d, V=sum(rows), P=1, seed=67)
    inp = wl.resplit(inp, rows, order=[2, 0, 3, 1])
    g = wl.random_grad_loss(T, 67, "random")
    compare_all(inp, run_gpu(inp, g), run_oracle(inp, g), f"{inp.dtype} T={T} d={d}")


@pytest.mark.parametrize("name", [F32, BF16])
def test_few_token_dw_is_added_to(name):
    import torch

    import oracle
    import paper_2609_14306_amd as vp
    from helpers import oracle_inputs

    rows = [600, 1500, 260]
    inp = wl.resplit(wl.make_inputs(name, T=150, d=96, V=sum(rows), P=1, seed=61), rows)
    g = wl.random_grad_loss(inp.T, 61, "random")
    H, Ws, t = to_device(inp)
    _, lse = vp.forward(H, Ws, t)
    base = [torch.randn(r, inp.d, device="cuda") for r in rows]
    dH, dW = vp.backward(H, Ws, t, lse, torch.from_numpy(g).cuda(), dW_shards=[b.clone() for b in base],
                         accumulate=True)
    H64, W64 = oracle_inputs(inp)
    ref = oracle.forward_backward(H64, W64, inp.targets, g)
    got = np.concatenate([(a.double() - b.double()).cpu().numpy() for a, b in zip(dW, base)])
    # the sum is rounded once more, at the size of base + dW: 2^-24 relative per element
    noise = 2.0 ** -24 * float(torch.cat(dW).norm()) / np.linalg.norm(ref["dW"])
    assert_grad_close(inp.dtype, dH.cpu().numpy(), ref["dH"], "dH")
    err = np.linalg.norm(got - ref["dW"]) / np.linalg.norm(ref["dW"])
    assert err <= (1e-2 if inp.dtype == "bf16" else 1e-5) + noise, err
