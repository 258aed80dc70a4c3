"""The claiming form of the one-launch decode step (257 to 512 attention units of at least 64 KiB of K rows, unsplit):
every variant of its kernel against the two calls, bit for bit, and the attention against the oracle. Each case states
that the dispatch takes this form, so that a change of its rule cannot leave the kernel untested.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_out_close, bits_to_torch, random_sel, say, step_form, torch_to_bits

pytestmark = pytest.mark.gpu

TD = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}

# layers, first layer, sequences, query heads, kv heads, head dim, type, tokens per cluster, fan-out, clusters selected,
# tail rows, sharing period, similarity, group rule
CASES = [
    (16, 0, 1, 32, 32, 128, "bf16", 32, 8, 8, 0, 4, "linear", "sum"),    # the shortest list: 256 rows of 256 B
    (16, 3, 1, 32, 32, 128, "bf16", 32, 8, 12, 0, 4, "linear", "sum"),   # layers 3-5 owned before the block
    (256, 5, 1, 2, 2, 64, "fp16", 16, 4, 32, 0, 2, "linear", "sum"),     # the most layers; layer 5 owned before
    (24, 0, 1, 12, 12, 64, "fp32", 16, 4, 16, 0, 2, "linear", "sum"),    # fp32, 288 units
    (5, 1, 2, 32, 32, 128, "fp32", 8, 2, 16, 0, 2, "mean", "sum"),       # 320 units, two sequences
    (40, 0, 1, 32, 8, 128, "bf16", 64, 8, 4, 0, 4, "linear", "max"),     # four query heads a row, the largest counts
    (40, 2, 1, 16, 8, 64, "fp16", 64, 8, 8, 0, 4, "maxprod", "max"),     # two
    (33, 0, 1, 64, 8, 128, "fp16", 16, 4, 16, 0, 2, "maxprod", "sum"),   # eight, 264 units
    (16, 0, 1, 32, 32, 128, "fp16", 32, 8, 12, 19, 4, "maxprod", "sum"),  # a tail
    (33, 1, 1, 32, 8, 128, "bf16", 16, 4, 20, 5, 4, "mean", "max"),      # a tail, owners before the block
]


@pytest.mark.parametrize("case", CASES)
def test_claiming_step_equals_two_calls_and_oracle(case):
    import paper_2501_06807_amd as M
    L, layer0, B, Hq, Hkv, d, dtype, s, f, k_sel, n_tail, period, sim, group = case
    say(f"[claim] {case}")
    rng = np.random.default_rng(L * 1000 + Hq + k_sel)
    C = k_sel + 5
    S = -(-C // f)
    Ts, sm = C * s, 1.0 / math.sqrt(d)
    draw = lambda *x: torch_to_bits(torch.from_numpy(rng.standard_normal(x).astype(np.float32)).to(TD[dtype]), dtype)  # noqa: E731
    k, v = draw(L, B, Hkv, Ts + n_tail, d), draw(L, B, Hkv, Ts + n_tail, d)
    kt, vt = bits_to_torch(k, dtype), bits_to_torch(v, dtype)
    cfg = M.select_cfg(s, f, S, k_sel, share_period=period, similarity=sim, group=group)
    dims = M.dims_of(torch.empty((L, B, Hq, d), dtype=TD[dtype]), kt, layer0)
    assert step_form(dims, Ts, cfg, n_tail) == ("claiming", 1, 8)
    R = 2 if sim == "maxprod" else 1
    n_c = -(-(Ts + n_tail) // s)
    cent = torch.zeros(L, B, Hkv, n_c, *([R, d] if R > 1 else [d]), device="cuda")
    scent = torch.zeros(L, B, Hkv, -(-n_c // f), *cent.shape[4:], device="cuda")
    M.mpc_build_clusters(kt, cent, scent, cfg, Ts=Ts, layer0=layer0)
    # layers owned before the block come with a selection
    sel_in = torch.from_numpy(random_sel(rng, L * B * Hkv, C, k_sel).reshape(L, B, Hkv, k_sel)).cuda()
    before = [l for l in range(L) if oracle.owner_layer(layer0 + l, period, 2) < layer0]
    ws = M.workspace(M.workspace_bytes(M.MPC_OP_DECODE_STEP, dims, Ts, cfg))
    ws_attn = M.workspace(M.workspace_bytes(M.MPC_OP_DECODE_ATTN, dims, Ts))
    for step in range(2):  # the second on the words that the first left
        q = draw(L, B, Hq, d)
        qt = bits_to_torch(q, dtype)
        got = []
        for one in (False, True):
            sel = torch.full((L, B, Hkv, k_sel), -7, dtype=torch.int32, device="cuda")
            sel[before] = sel_in[before]
            sc = torch.zeros(sel.shape, device="cuda")
            out = torch.full((L, B, Hq, d), 3.0, dtype=TD[dtype], device="cuda")
            lse = torch.zeros((L, B, Hq), device="cuda")
            if one:
                M.mpc_decode_step(qt, cent, scent, kt, vt, sel, out, cfg, sm_scale=sm, Ts=Ts, n_tail=n_tail, sel_score=sc,
                                  lse=lse, ws=ws, layer0=layer0)
            else:
                M.mpc_select_clusters(qt, cent, scent, sel, cfg, Ts=Ts, sel_score=sc, layer0=layer0)
                M.mpc_sparse_decode_attn(qt, kt, vt, sel, out, cluster_size=s, sm_scale=sm, Ts=Ts, n_tail=n_tail, lse=lse,
                                         ws=ws_attn, layer0=layer0)
            torch.cuda.synchronize()
            got.append((sel, sc, out, lse))
        for name, a, b in zip(("sel", "sel_score", "out", "lse"), *got):
            assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8)), (step, name)
        assert M.mpc_decode_step_status(ws) == 0 and not ws[256:].any()  # every head's words back at zero
        sel, _, out, lse = got[1]
        ref, ref_lse = oracle.sparse_decode_attn(q, k, v, sel.cpu().numpy(), dtype, cluster=s, sm_scale=sm, n_tail=n_tail)
        assert_out_close(out.double().cpu().numpy(), ref, dtype, case)
        # fp32 sums of fp32 exponentials: a few units in the last place of scores up to about 10
        np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, rtol=0, atol=2e-5)
