"""Every tile class of the backward and every tile of the forward, with the ways a tile may end
(tile_cases.py): whole gradients, losses, normalisers and fold states against the float64
oracle at the bars of helpers.py."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_loss_close, compare_all, oracle_inputs, run_gpu, run_oracle, to_device
from tile_cases import BACKWARD, FORWARD

pytestmark = pytest.mark.gpu

NAMES = {"f32": "tiny_f32_T256_d256_V2048_P8", "bf16": "bf16_T4096_d2880_V201088_P8"}


def _inputs(dtype, T, d, rows):
    inp = wl.make_inputs(NAMES[dtype], T=T, d=d, V=sum(rows), P=1, seed=89)
    return wl.resplit(inp, rows, order=list(range(len(rows)))[::-1])


@pytest.mark.parametrize("cls,dtype,T,d,rows,strip", BACKWARD)
def test_backward_tile(cls, dtype, T, d, rows, strip):
    inp = _inputs(dtype, T, d, rows)
    g = wl.random_grad_loss(T, 89, "random")
    errs = compare_all(inp, run_gpu(inp, g, strip_elems=strip), run_oracle(inp, g), f"class {cls} {dtype} T={T} d={d}")
    print(f"class {cls} {dtype} T={T} d={d}:", errs, flush=True)


@pytest.mark.parametrize("kind,folds,dtype,T,d,rows", FORWARD)
def test_forward_tile(kind, folds, dtype, T, d, rows):
    import oracle
    import paper_2609_14306_amd as vp

    inp = _inputs(dtype, T, d, rows)
    H, Ws, t = to_device(inp)
    H64, W64 = oracle_inputs(inp)
    ref_loss, ref_lse = oracle.forward(H64, np.concatenate(W64), inp.targets, inp.ignore_index)
    loss, lse = vp.forward(H, Ws, t, inp.ignore_index, inp.order)
    state = vp.new_state(T, "cuda")
    start = np.cumsum([0] + rows)
    for q in inp.order:
        vp.fold_shard(H, Ws[q], int(start[q]), t, state)
    f_loss, f_lse = vp.fold_finalize(t, state, rows, inp.ignore_index)
    for got, ref, what in ((loss, ref_loss, "loss"), (lse, ref_lse, "lse"), (f_loss, ref_loss, "fold loss"),
                           (f_lse, ref_lse, "fold lse")):
        assert_loss_close(dtype, got.cpu().numpy(), ref, f"kind {kind} {dtype} T={T} d={d} {what}")
