"""The package's functions marshal the usual arguments in native code and all others by themselves: the same calls either way, and the same errors."""
import ctypes
import types

import numpy as np
import pytest
import torch

import paper_2605_22718_amd as wk
from wkt import dev

pytestmark = pytest.mark.gpu
H, T, F, M, R = 3, 40, 3, 6, 2


def _calls():
    """(name, function of fresh outputs that makes the call and returns them) of every entry point with a native form."""
    d, g = dev(), torch.Generator(device=dev()).manual_seed(1)
    rn = lambda *s, dt=torch.bfloat16: torch.randn(s, generator=g, device=d).to(dt)
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32, device=d)
    desc = wk.make_compress_desc(H, T, F, wk.WK_BF16, 0.5)
    n_out, _ = wk.wk_keep_count(0.5, wk.WK_RATIO_CHUNK, wk.WK_ANCHOR_FIRST_FRAME, F, T)
    K, V, Q = rn(H, F * T, 128), rn(H, F * T, 128), rn(H, 50, 128)
    store = wk.Store([rn(H, n_out, 128) for _ in range(M)], [rn(H, n_out, 128) for _ in range(M)])
    ids, n_ids, poses = i32(4, 1), i32(2), rn(M, 5, dt=torch.float32)
    cap = 30 + R * n_out

    def compress():
        kept, Ko, Vo = i32(*range(n_out)).view(1, n_out), rn(H, n_out, 128), rn(H, n_out, 128)
        n = wk.wk_compress_chunk(desc, K, V, None, kept, Ko, Vo, torch.empty(wk.wk_compress_workspace_bytes(desc), dtype=torch.uint8, device=d))
        assert n == n_out
        return kept, Ko, Vo

    def poses_call(cur=(0.5, 1.0, -2.0, 0.25, 0.1)):
        out = i32(0, 0), torch.zeros(R, dtype=torch.float64, device=d), i32(0)
        wk.wk_score_chunks(poses, M, cur, wk.WK_NORM_MAX, R, *out)
        return out

    def gather():
        Kw, Vw, n = torch.zeros(H, cap, 128, dtype=K.dtype, device=d), torch.zeros(H, cap, 128, dtype=K.dtype, device=d), i32(0)
        wk.wk_gather_window(store.desc, ids, n_ids, R, K[:, :30].contiguous(), V[:, :30].contiguous(), 30, Kw, Vw, cap, n)
        return Kw, Vw, n

    def attention(**kw):
        O, lse = torch.zeros_like(Q), torch.zeros(H, 50, device=d)
        wk.wk_attention(Q, K, V, O, lse, **kw)
        return O, lse

    def in_place():
        O, lse = torch.zeros_like(Q), torch.zeros(H, 50, device=d)
        wk.wk_attention_in_place(Q, K, V, 100, store.desc, ids, n_ids, R, O, lse)
        wk.wk_attention_in_place(Q, None, None, 0, store.desc, ids, n_ids, R, O2 := torch.zeros_like(Q))
        return O, lse, O2

    def chunk_lse():
        lse = torch.zeros(M, H, 50, device=d)
        return (wk.wk_chunk_lse(store.desc, Q, lse),)

    def update():
        Kw, Vw = torch.zeros(H, cap, 128, dtype=K.dtype, device=d), torch.zeros(H, cap, 128, dtype=K.dtype, device=d)
        slots, n, nf = i32(-1, -1), i32(0), i32(0)
        wk.wk_window_update(store.desc, ids, None, R, n_out, slots, 30, Kw, Vw, cap, n, nf,
                            torch.empty(wk.wk_window_update_workspace_bytes(R), dtype=torch.uint8, device=d))
        return Kw, Vw, slots, n, nf

    length = i32(77)
    return {"compress": compress, "poses": poses_call, "gather": gather, "attention": attention, "in_place": in_place, "chunk_lse": chunk_lse, "update": update,
            "attention_length": lambda: attention(N_kv=90, n_kv_dev=length, scale=0.05),
            "attention_lse_only": lambda: (wk.wk_attention(Q, K, None, None, lse := torch.zeros(H, 50, device=d)), lse)[1:],
            # not the usual arguments: numbers of other kinds, a pose of mixed ones, tensors that are subclasses
            "numpy": lambda: attention(N_kv=np.int64(90), scale=np.float32(0.05)), "whole_scale": lambda: attention(scale=0),
            "pose_of_numbers": lambda: poses_call(np.array([1, 2, 3, 0, 0])), "pose_of_ints": lambda: poses_call([1, 2, 3, 0, 0])}


NAMES = ["compress", "poses", "gather", "attention", "in_place", "chunk_lse", "update", "attention_length", "attention_lse_only", "numpy", "whole_scale",
         "pose_of_numbers", "pose_of_ints"]


@pytest.mark.parametrize("name", NAMES)
def test_native_and_python_marshalling_make_the_same_call(name, monkeypatch):
    assert isinstance(wk._native, types.ModuleType), "the binding is not built"
    wk.lib()
    call, answers = _calls()[name], []

    class Watched:
        def __getattr__(self, function):
            def run(*args):
                answers.append(getattr(native, function)(*args))
                return answers[-1]
            return run

    native = wk._native
    monkeypatch.setattr(wk, "_native", Watched())
    got = call()
    assert len(answers) >= 1 and all((a is None) == (name in NAMES[-4:]) for a in answers)
    monkeypatch.setattr(wk, "_native", type("Absent", (), {"__getattr__": lambda self, f: lambda *a: None})())
    for a, b in zip(got, call()):
        assert torch.equal(a, b)


def test_errors_are_those_of_the_functions():
    d = dev()
    Q, K = torch.zeros(2, 8, 128, dtype=torch.bfloat16, device=d), torch.zeros(2, 64, 128, dtype=torch.bfloat16, device=d)
    O = torch.empty_like(Q)
    with pytest.raises(ValueError, match="K_win: must be contiguous"):
        wk.wk_attention(Q, K.transpose(0, 1), K, O)
    with pytest.raises(TypeError, match="V_win"):
        wk.wk_attention(Q, K, K.float(), O)
    with pytest.raises(TypeError, match="lse"):
        wk.wk_attention(Q, K, K, O, torch.empty(2, 8, dtype=torch.float64, device=d))
    with pytest.raises(TypeError):
        wk.wk_attention(Q.half(), K.half(), K.half(), O.half())
    with pytest.raises(ValueError, match="Q: must live"):
        wk.wk_attention(Q.cpu(), K, K, O)
    with pytest.raises(wk.WkError) as e:
        wk.wk_attention(Q, K, K, O, N_kv=65)
    assert e.value.status == wk.WK_ERR_SHAPE or e.value.status == wk.WK_ERR_INVALID_ARG
    with pytest.raises(ctypes.ArgumentError):   # a structure of another type is not taken for one
        wk.wk_chunk_lse(wk.make_compress_desc(2, 8, 3, wk.WK_BF16, 0.5), Q, torch.empty(1, 2, 8, device=d))
