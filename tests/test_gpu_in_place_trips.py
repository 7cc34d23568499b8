"""Attention in place where the host's bounds promise long segments: whole trips of the hand-scheduled loop inside a segment, compiled
steps across its boundaries.  Lengths around the trips' edges, and chunks that turn out shorter than the bound."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import K128_PAIR, K256, assert_attention_close_bf16, attention_plan, dev

pytestmark = pytest.mark.gpu


# workgroups of 256 queries, and of 128 with tiles in pairs, in less than a round and in more; 9 tiles of native rows beside 26 of a chunk are
# just short of the share that takes the loop, 10 have it
@pytest.mark.parametrize("H,layout", [(2, K128_PAIR), (100, K256), (130, K128_PAIR)])
@pytest.mark.parametrize("n_native,lens", [(64 * 30, []), (64 * 29 + 1, [64]), (64 * 40, [63, 130]), (0, [64 * 24, 64 * 23 + 63, 64 * 25 + 1]), (64 * 9, [64 * 26]), (64 * 10, [64 * 26]),
                                           (64 * 21 - 1, [64 * 22, 1, 64 * 21, 700]), (100, [64 * 27 - 1, 64 * 13, 64 * 12, 64 * 11 + 5])])
def test_against_oracle(H, layout, n_native, lens):
    N_q, d = 270, dev()
    assert attention_plan(H, N_q, n_native + len(lens) * max(lens, default=0))[0] == layout
    assert wk.lib().wk_internal_in_place_trips(n_native, len(lens), max(lens, default=1)) == (n_native != 64 * 9)
    g = torch.Generator().manual_seed(n_native + len(lens))
    rn = lambda n: torch.randn(H, n, 128, generator=g).to(torch.bfloat16)
    Q, Kn, Vn = rn(N_q), rn(n_native), rn(n_native)
    ks, vs = [rn(n) for n in lens], [rn(n) for n in lens]
    K, V = torch.cat([Kn, *ks], 1), torch.cat([Vn, *vs], 1)
    store = wk.Store([x.to(d) for x in ks or [rn(1)]], [x.to(d) for x in vs or [rn(1)]])
    R = len(lens)
    ids, n_ids = torch.arange(max(R, 1), dtype=torch.int32, device=d), torch.full((1,), R, dtype=torch.int32, device=d)
    O, lse = torch.empty_like(Q, device=d), torch.empty((H, N_q), device=d)
    wk.wk_attention_in_place(Q.to(d), Kn.to(d) if n_native else None, Vn.to(d) if n_native else None, n_native, store.desc, ids, n_ids, R, O, lse)
    rows = np.array([0, 1, 31, 32, 127, 128, 200, 255, 256, 269]) if H > 2 else np.arange(N_q)
    ref, ref_lse = oracle.attention(Q, K, V, rows=rows, want_lse=True)
    assert_attention_close_bf16(O.cpu()[:, rows], ref, lse.cpu()[:, rows], ref_lse)
