"""Host-side tests of the Python binding's tensor checks (no GPU).

The C ABI takes bare pointers, so the binding checks every tensor against the
problem before taking its pointer: dtype, shape (including each shard's width d),
contiguity, and one GPU device for all of them.  Each refusal below is raised on
the host; the library is never called with these tensors."""
import os

import pytest
import torch

import paper_2609_14306_amd as vp

pytestmark = pytest.mark.skipif(not os.path.exists(vp.LIB_PATH),
                                reason="libvpce.so not built (run __graft_entry__.build())")

T, D, ROWS = 6, 16, [5, 0, 7]


def _inputs(dtype=torch.bfloat16):
    H = torch.zeros(T, D, dtype=dtype)
    Ws = [torch.zeros(r, D, dtype=dtype) for r in ROWS]
    t = torch.zeros(T, dtype=torch.int64)
    return H, Ws, t


def _prob(dtype=torch.bfloat16):
    return vp.Problem(T, D, ROWS, vp.VP_BF16 if dtype == torch.bfloat16 else vp.VP_F32)


def _fwd_args(**over):
    H, Ws, t = _inputs()
    a = dict(prob=_prob(), H=H, W_shards=Ws, targets=t, loss=torch.zeros(T), lse=torch.zeros(T),
             ws=torch.zeros(vp.vp_ce_workspace_size(_prob())[0], dtype=torch.uint8))
    a.update(over)
    return a


def _bwd_args(**over):
    H, Ws, t = _inputs()
    a = dict(prob=_prob(), H=H, W_shards=Ws, targets=t, lse=torch.zeros(T), grad_loss=torch.zeros(T),
             dH=torch.zeros(T, D), dW_shards=[torch.zeros(r, D) for r in ROWS],
             ws=torch.zeros(vp.vp_ce_workspace_size(_prob())[1], dtype=torch.uint8))
    a.update(over)
    return a


def _refused(fn, args, match):
    with pytest.raises(ValueError, match=match):
        fn(**args)


FWD_CASES = {
    "H float32 with bf16 problem": (dict(H=torch.zeros(T, D)), "H: dtype"),
    "H wrong width": (dict(H=torch.zeros(T, D + 8, dtype=torch.bfloat16)), "H: shape"),
    "H not contiguous": (dict(H=torch.zeros(D, T, dtype=torch.bfloat16).t()), "H: must be contiguous"),
    "shard wrong width": (dict(W_shards=[torch.zeros(5, D + 8, dtype=torch.bfloat16),
                                         torch.zeros(0, D, dtype=torch.bfloat16),
                                         torch.zeros(7, D, dtype=torch.bfloat16)]), r"W_shards\[0\]: shape"),
    "shard wrong dtype": (dict(W_shards=[torch.zeros(5, D, dtype=torch.bfloat16),
                                         torch.zeros(0, D, dtype=torch.bfloat16),
                                         torch.zeros(7, D)]), r"W_shards\[2\]: dtype"),
    "shard count": (dict(W_shards=[torch.zeros(5, D, dtype=torch.bfloat16)]), "W_shards: 1 shards"),
    "int32 targets": (dict(targets=torch.zeros(T, dtype=torch.int32)), "targets: dtype"),
    "short targets": (dict(targets=torch.zeros(T - 1, dtype=torch.int64)), "targets: shape"),
    "bf16 loss": (dict(loss=torch.zeros(T, dtype=torch.bfloat16)), "loss: dtype"),
    "strided lse": (dict(lse=torch.zeros(2 * T)[::2]), "lse: must be contiguous"),
    "small workspace": (dict(ws=torch.zeros(8, dtype=torch.uint8)), "ws:"),
    "host tensors": ({}, "must be on a GPU device"),
}


@pytest.mark.parametrize("case", sorted(FWD_CASES))
def test_forward_refuses(case):
    over, match = FWD_CASES[case]
    _refused(vp.vp_ce_forward, _fwd_args(**over), match)


BWD_CASES = {
    "float64 grad_loss": (dict(grad_loss=torch.zeros(T, dtype=torch.float64)), "grad_loss: dtype"),
    "bf16 lse": (dict(lse=torch.zeros(T, dtype=torch.bfloat16)), "lse: dtype"),
    "dH bf16": (dict(dH=torch.zeros(T, D, dtype=torch.bfloat16)), "dH: dtype"),
    "dH transposed": (dict(dH=torch.zeros(D, T).t()), "dH: must be contiguous"),
    "dW bf16": (dict(dW_shards=[torch.zeros(5, D, dtype=torch.bfloat16), torch.zeros(0, D),
                                torch.zeros(7, D)]), r"dW_shards\[0\]: dtype"),
    "dW wrong rows": (dict(dW_shards=[torch.zeros(5, D), torch.zeros(0, D), torch.zeros(6, D)]),
                      r"dW_shards\[2\]: shape"),
    "dW count": (dict(dW_shards=[torch.zeros(5, D)]), "dW_shards: 1 shards"),
    "small workspace": (dict(ws=torch.zeros(64, dtype=torch.uint8)), "ws:"),
    "host tensors": ({}, "must be on a GPU device"),
}


@pytest.mark.parametrize("case", sorted(BWD_CASES))
def test_backward_refuses(case):
    over, match = BWD_CASES[case]
    _refused(vp.vp_ce_backward, _bwd_args(**over), match)


# On GPU tensors the checks are one pass that takes the pointers (_call_pointers); what it
# answers None for goes to the checks above.  CPU tensors whose H says it is on a GPU take
# that pass here (their device index is -1 like H's own).
class _GpuLike(torch.Tensor):
    is_cuda = property(lambda self: True)


class _OtherGpu(torch.Tensor):
    def get_device(self):
        return 1


def _pass(a):
    H = a["H"]
    per_token = (a["loss"], a["lse"]) if "loss" in a else (a["lse"], a["grad_loss"])
    return vp._call_pointers(a["prob"], H.as_subclass(_GpuLike), a["W_shards"], a["targets"], per_token,
                             a.get("dH"), a.get("dW_shards"), a["ws"])


def test_one_pass_takes_the_pointers():
    for a in (_fwd_args(), _bwd_args()):
        h, w, t, v, g, gw, ws, n = _pass(a)
        assert h == a["H"].data_ptr() and t == a["targets"].data_ptr()
        assert list(w) == [x.data_ptr() or None for x in a["W_shards"]]
        assert v == [x.data_ptr() for x in ((a["loss"], a["lse"]) if "loss" in a else (a["lse"], a["grad_loss"]))]
        assert (ws, n) == (a["ws"].data_ptr(), a["ws"].numel())
        if "dH" in a:
            assert g == a["dH"].data_ptr() and list(gw) == [x.data_ptr() or None for x in a["dW_shards"]]
        else:
            assert g is None and gw is None


@pytest.mark.parametrize("case", sorted(set(FWD_CASES) - {"small workspace", "host tensors"}))
def test_one_pass_refuses_forward(case):  # (the library checks the workspace's size)
    assert _pass(_fwd_args(**FWD_CASES[case][0])) is None


@pytest.mark.parametrize("case", sorted(set(BWD_CASES) - {"small workspace", "host tensors"}))
def test_one_pass_refuses_backward(case):
    assert _pass(_bwd_args(**BWD_CASES[case][0])) is None


def test_one_pass_refuses_other_forms():
    bf = torch.bfloat16
    z = torch.zeros
    for over in (dict(H=z(T, D, dtype=bf).unsqueeze(0)), dict(targets=z(2 * T, dtype=torch.int64)[::2]),
                 dict(W_shards=[z(D, 5, dtype=bf).t(), z(0, D, dtype=bf), z(7, D, dtype=bf)]),
                 dict(W_shards=[z(5, D, dtype=bf), None, z(7, D, dtype=bf)]), dict(loss=z(T + 1)), dict(lse=None),
                 dict(ws=_fwd_args()["ws"].as_subclass(_OtherGpu)), dict(loss=z(T).as_subclass(_OtherGpu)),
                 dict(targets=[0] * T), dict(ws=z(1 << 20, dtype=torch.uint8)[::2]), dict(ws=7)):
        assert _pass(_fwd_args(**over)) is None, over
    for over in (dict(dH=z(T, D + 1)), dict(dW_shards=[z(D, 5).t(), z(0, D), z(7, D)]), dict(dW_shards=None),
                 dict(dW_shards=[z(5, D), z(0, D), z(7, D + 1)])):
        assert _pass(_bwd_args(**over)) is None, over
    assert _pass(_fwd_args(H=z(T, D, dtype=bf))) is not None
    x = z(T)
    assert vp._pointers((x,), torch.float32, (T,), -1) == [x.data_ptr()]
    assert vp._pointers((x,), torch.float32, (T,), 0) is None  # another device
    assert vp._shard_pointers(_prob(), [z(5, D, dtype=bf), z(0, D, dtype=bf), z(7, D, dtype=bf)], bf, 1) is None
    a = _fwd_args()
    assert vp._call_pointers(a["prob"], a["H"], a["W_shards"], a["targets"], (a["loss"], a["lse"])) is None  # a CPU H


def test_fold_calls_refuse():
    H, Ws, t = _inputs()
    shard = vp.Problem(T, D, [7], vp.VP_BF16)
    ws = torch.zeros(vp.vp_ce_workspace_size(shard)[0], dtype=torch.uint8)
    with pytest.raises(ValueError, match="state: shape"):
        vp.vp_ce_fold_shard(shard, 0, H, Ws[2], t, torch.zeros(T), ws)
    with pytest.raises(ValueError, match="W_shards\\[0\\]: shape"):
        vp.vp_ce_fold_shard(shard, 0, H, Ws[0], t, torch.zeros(3 * T), ws)
    with pytest.raises(ValueError, match="must be on a GPU device"):
        vp.vp_ce_fold_shard(shard, 0, H, Ws[2], t, torch.zeros(3 * T), ws)
    with pytest.raises(ValueError, match="state: dtype"):
        vp.vp_ce_state_init(torch.zeros(3 * T, dtype=torch.float64), T)
    full = vp.Problem(T, D, ROWS, vp.VP_BF16)
    with pytest.raises(ValueError, match="targets: dtype"):
        vp.vp_ce_fold_finalize(full, t.int(), torch.zeros(3 * T), torch.zeros(T), torch.zeros(T),
                               torch.zeros(256, dtype=torch.uint8))


def test_fold_refuses_a_state_that_is_no_tensor(monkeypatch):
    # On a GPU the state's pointer is taken after the other tensors passed the one-pass
    # checks: here they are made to pass.
    H, Ws, t = _inputs()
    shard = vp.Problem(T, D, [7], vp.VP_BF16)
    ws = torch.zeros(vp.vp_ce_workspace_size(shard)[0], dtype=torch.uint8)
    monkeypatch.setattr(vp, "_call_pointers", lambda *a, **k: (0, [None], 0, [], None, None, 0, 0))
    for state in (None, 3, [0.0] * (3 * T)):
        with pytest.raises(ValueError, match="state: expected a torch.Tensor"):
            vp.vp_ce_fold_shard(shard, 0, H, Ws[2], t, state, ws)
