"""Vocabulary rows that a program has switched off: with a last hidden feature of one, a row
of zeros whose last weight is minus infinity, or the type's lowest value, has that logit for
every token (the rows that pad a vocabulary to a round size).  Such rows have probability zero,
wherever they lie: the loss, the normaliser and the gradients are those of the other rows
alone, from the float64 oracle at the bars of helpers.py."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_grad_close, assert_loss_close, to_device

pytestmark = pytest.mark.gpu

F32, BF16 = "tiny_f32_T256_d256_V2048_P8", "bf16_T4096_d2880_V201088_P8"


def _masked(name, T, d, rows, dead, value):
    """Inputs with the global rows of `dead` (half-open ranges) switched off, and the oracle's
    view of the rest: (inp, H, shards, targets, live rows)."""
    import torch

    inp = wl.resplit(wl.make_inputs(name, T=T, d=d, V=sum(rows), P=1, seed=83), rows,
                     order=list(range(len(rows)))[::-1])
    off = np.zeros(sum(rows), bool)
    for lo, hi in dead:
        off[lo:hi] = True
    live = np.flatnonzero(~off)
    ok = inp.targets != inp.ignore_index
    inp.targets[ok] = live[inp.targets[ok] % live.size]
    H, Ws, t = to_device(inp)
    H[:, -1] = 1.0
    low = -float("inf") if value == "inf" else torch.finfo(H.dtype).min
    start = np.cumsum([0] + rows)
    for p, w in enumerate(Ws):
        m = torch.from_numpy(off[start[p]:start[p + 1]]).cuda()
        w[m] = 0.0
        w[m, -1] = low
    return inp, H, Ws, t, live


def _live_oracle(inp, H, Ws, live, g=None):
    import torch

    import oracle

    W64 = torch.cat([w.double() for w in Ws]).cpu().numpy()[live]
    to_live = np.full(inp.V, -1)
    to_live[live] = np.arange(live.size)
    tg = np.where(inp.targets == inp.ignore_index, inp.ignore_index, to_live[inp.targets])
    H64 = H.double().cpu().numpy()
    if g is None:
        return oracle.forward(H64, W64, tg, inp.ignore_index)
    return oracle.forward_backward(H64, [W64], tg, g, inp.ignore_index)


# A vocabulary of 16321 padded to a multiple of 64 in one shard, as programs do it.
@pytest.mark.parametrize("T", [1, 40, 100, 300])
@pytest.mark.parametrize("name", [F32, BF16])
def test_padded_vocabulary(name, T):
    import paper_2609_14306_amd as vp

    inp, H, Ws, t, live = _masked(name, T, 128, [16384], [(16321, 16384)], "lowest")
    ref_loss, ref_lse = _live_oracle(inp, H, Ws, live)
    loss, lse = vp.forward(H, Ws, t, inp.ignore_index, inp.order)
    assert_loss_close(inp.dtype, lse.cpu().numpy(), ref_lse, f"{name} T={T} lse")
    assert_loss_close(inp.dtype, loss.cpu().numpy(), ref_loss, f"{name} T={T} loss")


# The tail of the vocabulary, rows that start a shard, and whole shards; the tiles of few
# tokens, of many, and one tile per workgroup.
SHARDS = [2048, 1100, 512, 300]
DEAD = [(0, 64), (1984, 2048), (3148, 3660), (3900, 3960)]


@pytest.mark.parametrize("T", [1, 40, 100, 300, 2048, 2500])
@pytest.mark.parametrize("value", ["inf", "lowest"])
@pytest.mark.parametrize("name", [F32, BF16])
def test_forward_and_fold_ignore_masked_rows(name, value, T):
    import paper_2609_14306_amd as vp

    for d in (64, 520):
        inp, H, Ws, t, live = _masked(name, T, d, SHARDS, DEAD, value)
        ref_loss, ref_lse = _live_oracle(inp, H, Ws, live)
        loss, lse = vp.forward(H, Ws, t, inp.ignore_index, inp.order)
        assert_loss_close(inp.dtype, lse.cpu().numpy(), ref_lse, f"{name} {value} T={T} d={d} lse")
        assert_loss_close(inp.dtype, loss.cpu().numpy(), ref_loss, f"{name} {value} T={T} d={d} loss")
        state = vp.new_state(T, "cuda")
        start = np.cumsum([0] + SHARDS)
        for q in (2, 0, 3, 1):  # the switched-off shard first
            vp.fold_shard(H, Ws[q], int(start[q]), t, state)
            if q == 2:
                assert bool((state[:T] == -float("inf")).all()) and bool((state[T:2 * T] == 0).all())
        loss, lse = vp.fold_finalize(t, state, SHARDS, inp.ignore_index)
        assert_loss_close(inp.dtype, lse.cpu().numpy(), ref_lse, f"{name} {value} T={T} d={d} fold lse")
        assert_loss_close(inp.dtype, loss.cpu().numpy(), ref_loss, f"{name} {value} T={T} d={d} fold loss")


# (the lowest value only: a gradient multiplies the probability, zero, by the row's weight)
@pytest.mark.parametrize("T", [40, 700])
@pytest.mark.parametrize("name", [F32, BF16])
def test_backward_ignores_masked_rows(name, T):
    import torch

    import paper_2609_14306_amd as vp

    inp, H, Ws, t, live = _masked(name, T, 264, SHARDS, DEAD, "lowest")
    g = wl.random_grad_loss(T, 83, "random")
    ref = _live_oracle(inp, H, Ws, live, g)
    _, lse = vp.forward(H, Ws, t, inp.ignore_index, inp.order)
    dH, dW = vp.backward(H, Ws, t, lse, torch.from_numpy(g).cuda(), inp.ignore_index, inp.order)
    dW = torch.cat(dW).cpu().numpy()
    assert_grad_close(inp.dtype, dH.cpu().numpy(), ref["dH"], f"{name} T={T} dH")
    assert_grad_close(inp.dtype, dW[live], ref["dW"], f"{name} T={T} dW")
    assert not np.delete(dW, live, axis=0).any()
