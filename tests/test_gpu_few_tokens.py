"""The forward's tiles for few tokens (at most 2048): token counts around the 64-, 128- and
256-token tiles, shards around the 128- and 256-row tiles, widths with and without a part
slice, one and many turns per workgroup, and both workspace sizes the call accepts.  Losses,
normalisers and fold states against the float64 oracle at the bars of helpers.py."""
import ctypes

import numpy as np
import pytest

import workloads as wl
from helpers import assert_loss_close, oracle_inputs, to_device

pytestmark = pytest.mark.gpu

F32, BF16 = "tiny_f32_T256_d256_V2048_P8", "bf16_T4096_d2880_V201088_P8"


def _inputs(name, T, d, rows, order):
    inp = wl.make_inputs(name, T=T, d=d, V=sum(rows), P=1, seed=53)
    inp = wl.resplit(inp, rows, order=order)
    edge = [0, sum(rows) - 1, rows[0], wl.IGNORE_INDEX]  # targets at the ends and a shard's start
    n = min(T, len(edge))
    inp.targets[:n] = edge[:n]
    return inp


def _oracle_forward(inp):
    import oracle

    H, Ws = oracle_inputs(inp)
    return oracle.forward(H, np.concatenate(Ws), inp.targets, inp.ignore_index)


# 72 and 320: a part slice in bfloat16 or none in either type.  The small vocabulary has one
# tile per workgroup, the large one up to fifteen.
@pytest.mark.parametrize("T", [1, 64, 65, 129, 257, 1000, 2048])
@pytest.mark.parametrize("d,rows", [(72, [1, 127, 128, 129, 0, 2615]), (320, [20000, 1, 300])])
@pytest.mark.parametrize("name", [F32, BF16])
def test_forward_few_tokens(name, d, rows, T):
    import paper_2609_14306_amd as vp

    inp = _inputs(name, T, d, rows, list(range(len(rows)))[::-1])
    H, Ws, t = to_device(inp)
    loss, lse = vp.forward(H, Ws, t, inp.ignore_index, inp.order)
    ref_loss, ref_lse = _oracle_forward(inp)
    assert_loss_close(inp.dtype, loss.cpu().numpy(), ref_loss, f"{name} T={T} d={d} loss")
    assert_loss_close(inp.dtype, lse.cpu().numpy(), ref_lse, f"{name} T={T} d={d} lse")


# A wide hidden state, where 65..128 tokens take the 128-token tile for the large shard in
# float32 (bfloat16 shards run on it in test_gpu_tiles.py).
@pytest.mark.parametrize("T", [65, 128])
@pytest.mark.parametrize("name", [F32, BF16])
def test_fold_128_token_tile(name, T):
    import paper_2609_14306_amd as vp

    rows = [50000, 1, 300]
    inp = _inputs(name, T, 2056, rows, [1, 2, 0])
    H, Ws, t = to_device(inp)
    state = vp.new_state(T, "cuda")
    offs = np.cumsum([0] + rows)
    for q in inp.order:
        vp.fold_shard(H, Ws[q], int(offs[q]), t, state)
    loss, lse = vp.fold_finalize(t, state, rows, inp.ignore_index)
    ref_loss, ref_lse = _oracle_forward(inp)
    assert_loss_close(inp.dtype, loss.cpu().numpy(), ref_loss, f"{name} T={T} loss")
    assert_loss_close(inp.dtype, lse.cpu().numpy(), ref_lse, f"{name} T={T} lse")


def test_workspace_of_32_splits_is_enough():
    # The partial states of 32 splits have always been enough; vp_ce_workspace_size asks for
    # more at few tokens, and the call uses what it is given.
    import torch

    import paper_2609_14306_amd as vp

    T, d, rows = 40, 512, [9000, 4000]
    inp = _inputs(BF16, T, d, rows, [0, 1])
    H, Ws, t = to_device(inp)
    prob = vp.problem_for(H, Ws, inp.ignore_index, inp.order)
    a256 = lambda n: (n + 255) // 256 * 256
    small = 256 + 2 * a256(32 * T * 4) + a256(T * 4)
    assert small < vp.vp_ce_workspace_size(prob)[0]
    ws = torch.full((small + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    loss = torch.empty(T, device="cuda")
    lse = torch.empty(T, device="cuda")
    lib = vp.load_library()
    ptrs = (ctypes.c_void_p * 2)(*[w.data_ptr() for w in Ws])

    def call(nbytes):
        return lib.vp_ce_forward(ctypes.byref(prob.c), H.data_ptr(), ptrs, t.data_ptr(), loss.data_ptr(),
                                 lse.data_ptr(), ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream)

    assert call(small - 1) == vp.VP_ERR_WORKSPACE
    assert call(small) == vp.VP_OK
    torch.cuda.synchronize()
    assert bool((ws[small:] == 0x5A).all()), "wrote past the workspace"
    ref_loss, ref_lse = _oracle_forward(inp)
    assert_loss_close("bf16", loss.cpu().numpy(), ref_loss, "32 splits loss")
    assert_loss_close("bf16", lse.cpu().numpy(), ref_lse, "32 splits lse")


def test_fold_keeps_a_workspace_of_32_splits():
    # fold_shard allocates only where the workspace it is given is too small for the call.
    import torch

    import paper_2609_14306_amd as vp

    T, rows = 40, [9000, 4000]
    inp = _inputs(BF16, T, 512, rows, [0, 1])
    H, Ws, t = to_device(inp)
    a256 = lambda n: (n + 255) // 256 * 256
    small = 256 + 2 * a256(32 * T * 4) + a256(T * 4)
    assert small < vp.vp_ce_workspace_size(vp.problem_for(H, Ws[:1]))[0]
    for nbytes, allocations in ((small, 0), (small - 1, 2)):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        state = vp.new_state(T, "cuda")
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        vp.fold_shard(H, Ws[0], 0, t, state, ws)
        vp.fold_shard(H, Ws[1], rows[0], t, state, ws)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] - before == allocations
        loss, lse = vp.fold_finalize(t, state, rows, inp.ignore_index)
        ref_loss, ref_lse = _oracle_forward(inp)
        assert_loss_close("bf16", loss.cpu().numpy(), ref_loss, f"{nbytes} bytes loss")
        assert_loss_close("bf16", lse.cpu().numpy(), ref_lse, f"{nbytes} bytes lse")


# More than 2048 tokens, where a full last round takes fewer splits than the workspace has
# room for, and more splits than tiles.
@pytest.mark.parametrize("T,rows", [(2304, [9000, 4000]), (5000, [100, 3000]), (9000, [500])])
@pytest.mark.parametrize("name", [F32, BF16])
def test_forward_many_tokens(name, T, rows):
    import paper_2609_14306_amd as vp

    inp = _inputs(name, T, 64, rows, list(range(len(rows))))
    H, Ws, t = to_device(inp)
    loss, lse = vp.forward(H, Ws, t, inp.ignore_index, inp.order)
    ref_loss, ref_lse = _oracle_forward(inp)
    assert_loss_close(inp.dtype, loss.cpu().numpy(), ref_loss, f"{name} T={T} loss")
    assert_loss_close(inp.dtype, lse.cpu().numpy(), ref_lse, f"{name} T={T} lse")
