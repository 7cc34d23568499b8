"""The log-sum-exp alone over windows long enough for its own workgroup layout (64 queries a wave, every score against a reference
that seldom moves): every count of left-over tiles, rows and queries, and scores far above the first tile's."""
import glob
import importlib.util
import os
import re
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import dev

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_22718_amd", "csrc")


def test_loop_is_what_its_generator_writes():
    spec = importlib.util.spec_from_file_location("gen_lse_loop", os.path.join(CSRC, "gen_lse_loop.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    assert gen.render() == open(os.path.join(CSRC, gen.NAME)).read()
    lines = gen.generate()
    # two steps of 32 matrix instructions, the first LEAD once more in front of the loop, what either last step keeps back behind it
    assert sum(ln.startswith("v_mfma") for ln in lines) == 2 * 32 + gen.LEAD + 2 * gen.BACK
    assert sum(ln == "s_barrier" for ln in lines) == 2
    # a trip leaves for code behind the loop where a sum has grown or the loop ends, and branches nowhere else
    trip = lines[lines.index("L_trip_%=:"):lines.index("s_cbranch_scc0 L_trip_%=")]
    assert [re.sub(r"\d.*", "", ln) for ln in trip if "branch" in ln] == ["s_cbranch_scc"] * 5
    assert all(ln.startswith(("s_cbranch_scc1 L_grown", "s_cbranch_scc1 L_odd")) for ln in trip if "branch" in ln)


def test_no_register_waits_in_scratch(tmp_path):
    tools = "/opt/rocm/llvm/bin"
    if not os.path.exists(os.path.join(tools, "llvm-readelf")):
        pytest.skip("no llvm-readelf")
    shutil.copy(os.path.join(os.path.dirname(CSRC), "libwk.so"), tmp_path)
    subprocess.run([os.path.join(tools, "llvm-objdump"), "--offloading", "libwk.so"], cwd=tmp_path, check=True, capture_output=True)
    notes = "".join(subprocess.run([os.path.join(tools, "llvm-readelf"), "--notes", f], check=True, capture_output=True, text=True).stdout
                    for f in glob.glob(str(tmp_path / "*gfx950*")))
    kernels = [k for k in notes.split(".args:") if "k_lse_wide_bf16" in k]
    assert len(kernels) == 1 and re.search(r"\.private_segment_fixed_size: *0\b", kernels[0])


def _inputs(H, N_q, N_kv, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(H, n, 128, generator=g).to(torch.bfloat16) for n in (N_q, N_kv)]


def _lse(Q, K):
    out = torch.full(Q.shape[:2], float("nan"), device=dev())
    wk.wk_attention(Q.to(dev()), K.to(dev()), None, None, out)
    return out.cpu().numpy().astype(np.float64)


def _reference(Q, K):
    return oracle.attention(Q, K, K, want_lse=True)[1]


def _close(got, Q, K):
    """Every weight is rounded to bf16 (8 significant bits: by at most 2^-8 of itself, uniformly: 2^-8 / sqrt(3) rms), independently:
    six standard deviations of the sum, and 1e-5 for its fp32 terms and their logarithm."""
    p = torch.softmax(torch.matmul(Q.double(), K.double().transpose(1, 2).contiguous()) / 128 ** 0.5, -1)
    bound = 6 * 2.0 ** -8 / 3 ** 0.5 * p.pow(2).sum(-1).sqrt().numpy() + 1e-5
    return (np.abs(got - _reference(Q, K)) <= bound).all()


@pytest.mark.gpu
@pytest.mark.parametrize("N_q", [193, 256, 257, 321])
@pytest.mark.parametrize("N_kv", [641, 703, 704, 705, 768, 769, 833, 961, 1560])
def test_against_the_oracle(N_q, N_kv):
    Q, K = _inputs(2, N_q, N_kv, N_q * 10000 + N_kv)
    only = _lse(Q, K)
    assert _close(only, Q, K)
    d = dev()
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), K.to(d), O, lse)
    assert np.array_equal(lse.cpu().numpy(), only)   # no maximum grows by more than 2^8 behind the first tile


# Scores far above the first tile's: within the exponent's range (20) and beyond it (120, and a first tile without weight).  One
# weight can be all of a sum: half a unit in the last of bf16's 8 places, 2^-8 of it; fp32 scores of that size add their own
# rounding, 2^-23 of |score| <= 2000 in each of few steps.
@pytest.mark.gpu
@pytest.mark.parametrize("N_kv", [650, 704, 1000])
@pytest.mark.parametrize("factor", [20, 120, float("inf")])
def test_scores_above_the_first_tile(N_kv, factor):
    Q, K = _inputs(2, 300, N_kv, N_kv)
    if factor == float("inf"):
        Q[..., 0] = 1
        K[:, :64, 0] = -factor
        ref = _reference(Q, K[:, 64:].contiguous())
    else:
        K[:, 64:] *= factor
        ref = _reference(Q, K)
    assert np.abs(_lse(Q, K) - ref).max() <= 2.0 ** -8 + 2e-3


# one key far above the rest, in either key block of tiles of either parity, in the loop and behind it: its weight is not rounded (fp32
# sums of 704 terms)
@pytest.mark.gpu
@pytest.mark.parametrize("key", [64, 100, 128, 191, 640, 690, 703])
@pytest.mark.parametrize("log2_weight", [9.3, 14.7, 50.1, 200.3])
def test_a_dominating_weight_is_exact(key, log2_weight):
    Q, K = torch.zeros(1, 256, 128), torch.zeros(1, 704, 128)
    Q[..., 0] = 1
    K[0, key, 0] = log2_weight * 128 ** 0.5 * np.log(2)
    Q, K = Q.to(torch.bfloat16), K.to(torch.bfloat16)
    assert np.abs(_lse(Q, K) - _reference(Q, K)).max() <= 704 * 2.0 ** -24 + 2.0 ** -23 * log2_weight


@pytest.mark.gpu
def test_chunks_of_all_lengths_in_one_launch():
    d, lens = dev(), [700, 1, 64, 0, 385, 129, 192, 65, 1201]
    Q, K = _inputs(3, 333, max(lens), 5)
    keys = [K[:, :max(n, 1)].contiguous().to(d) for n in lens]
    store = wk.Store(keys, keys, d)
    store.n_tok[3] = 0
    out = torch.full((len(lens), 3, 333), float("nan"), device=d)
    wk.wk_chunk_lse(store.desc, Q.to(d), out)
    for n, got in zip(lens, out.cpu().numpy().astype(np.float64)):
        if n == 0:
            assert np.isneginf(got).all()
        else:
            assert _close(got, Q, K[:, :n].contiguous())
