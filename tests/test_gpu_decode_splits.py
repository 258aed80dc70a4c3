"""Sparse decode attention where the split rule changes its mind: token lists just below and above one, two and
the most splits, for each group size and row width, against the oracle; and the one-call decode step on the same
blocks against the two calls, bit for bit.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_out_close, bits_to_torch, random_sel, say, step_form, torch_to_bits

pytestmark = pytest.mark.gpu

TD = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}

# layers, sequences, query heads, kv heads, head dim, type, tokens per cluster, clusters selected, tail rows, splits. A
# workgroup takes 128 rows of 256 B a step, and up to three steps stay whole
SHAPES = [
    (1, 1, 4, 4, 128, "bf16", 16, 24, 0, 1),    # 384 rows: three steps
    (1, 1, 4, 4, 128, "bf16", 16, 24, 1, 4),    # 400 slots with one token in the last cluster: a fourth step
    (1, 1, 4, 4, 128, "bf16", 16, 31, 0, 4),
    (1, 1, 4, 4, 128, "bf16", 16, 32, 0, 4),    # 512: four whole steps
    (1, 1, 4, 4, 128, "bf16", 16, 31, 3, 4),
    (1, 2, 3, 3, 128, "fp32", 24, 8, 0, 1),     # 192 rows of 512 B: three steps of 64
    (1, 2, 3, 3, 128, "fp32", 24, 11, 0, 5),
    (1, 1, 2, 2, 64, "fp16", 32, 31, 1, 4),     # 1024 slots of 128 B, one token in the last cluster
    (1, 1, 8, 2, 128, "bf16", 16, 16, 0, 1),    # four query heads a row on the matrix cores: 128 rows a step
    (1, 1, 8, 2, 64, "fp16", 16, 24, 0, 1),     # of either width: three steps
    (1, 1, 8, 2, 64, "fp16", 16, 25, 0, 4),
    (1, 1, 16, 2, 128, "fp16", 8, 15, 5, 1),    # eight
    (1, 1, 16, 2, 128, "fp16", 8, 48, 5, 4),
    (1, 1, 1, 1, 128, "bf16", 64, 64, 7, 11),   # one unit, splits of three steps
    (1, 1, 1, 1, 128, "bf16", 64, 32, 0, 16),   # the most
    (2, 1, 127, 127, 64, "bf16", 4, 9, 0, 1),   # 254 units, short lists
    (1, 1, 128, 128, 64, "bf16", 32, 32, 0, 2),  # 256 workgroups
    (4, 1, 36, 36, 128, "fp32", 64, 50, 0, 3),  # 144 units, two splits to a compute unit: the step takes two kernels
    (4, 1, 64, 64, 64, "bf16", 8, 200, 0, 1),   # 256 units: never split
]


@pytest.mark.parametrize("shape", SHAPES)
def test_splits_match_oracle(shape, waves=8):
    import paper_2501_06807_amd as M
    L, B, Hq, Hkv, d, dtype, s, k_sel, n_tail, splits = shape
    say(f"[decode splits] {shape}")
    rng = np.random.default_rng(sum(map(hash, (L, B, Hq, Hkv, d, s, k_sel, n_tail))) % 2**32)
    Ts, sm = (k_sel + 4) * s, 1.0 / math.sqrt(d)
    draw = lambda *x: torch_to_bits(torch.from_numpy(rng.standard_normal(x).astype(np.float32)).to(TD[dtype]), dtype)  # noqa: E731
    q, k, v = draw(L, B, Hq, d), draw(L, B, Hkv, Ts + n_tail, d), draw(L, B, Hkv, Ts + n_tail, d)
    sel = random_sel(rng, L * B * Hkv, Ts // s, k_sel).reshape(L, B, Hkv, k_sel)
    qt, kt, vt = (bits_to_torch(x, dtype) for x in (q, k, v))
    out, lse = torch.empty_like(qt), torch.empty((L, B, Hq), dtype=torch.float32, device="cuda")
    need = M.workspace_bytes(M.MPC_OP_DECODE_ATTN, M.dims_of(qt, kt), Ts)
    ws = M.workspace(need)
    for _ in range(2):  # the arrival counters are back at zero after each call
        M.mpc_sparse_decode_attn(qt, kt, vt, torch.from_numpy(sel).cuda(), out, cluster_size=s, sm_scale=sm, Ts=Ts,
                                 n_tail=n_tail, lse=lse, ws=ws)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.sparse_decode_attn(q, k, v, sel, dtype, cluster=s, sm_scale=sm, n_tail=n_tail)
    assert_out_close(out.double().cpu().numpy(), ref, dtype, shape)
    # fp32 sums of fp32 exponentials: a few units in the last place of scores up to about 10
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, rtol=0, atol=2e-5)

    f = 4
    C = Ts // s
    cfg = M.select_cfg(s, f, -(-C // f), k_sel, share_period=1)
    assert step_form(M.dims_of(qt, kt), Ts, cfg, n_tail)[1:] == (splits, waves)
    cap = Ts + n_tail
    cent = torch.zeros(L, B, Hkv, -(-cap // s), d, device="cuda")
    scent = torch.zeros(L, B, Hkv, -(-cent.shape[3] // f), d, device="cuda")
    M.mpc_build_clusters(kt, cent, scent, cfg, Ts=Ts)
    sels = [torch.zeros((L, B, Hkv, k_sel), dtype=torch.int32, device="cuda") for _ in range(2)]
    outs = [torch.empty_like(qt) for _ in range(2)]
    M.mpc_select_clusters(qt, cent, scent, sels[0], cfg, Ts=Ts)
    M.mpc_sparse_decode_attn(qt, kt, vt, sels[0], outs[0], cluster_size=s, sm_scale=sm, Ts=Ts, n_tail=n_tail, ws=ws)
    step_ws = M.workspace(M.workspace_bytes(M.MPC_OP_DECODE_STEP, M.dims_of(qt, kt), Ts, cfg))
    for _ in range(2):
        M.mpc_decode_step(qt, cent, scent, kt, vt, sels[1], outs[1], cfg, sm_scale=sm, Ts=Ts, n_tail=n_tail, ws=step_ws)
    torch.cuda.synchronize()
    assert torch.equal(sels[0], sels[1])
    assert torch.equal(outs[0].view(torch.uint8), outs[1].view(torch.uint8))


# many units with lists of at most 16 KiB of K rows (a wave each), and the first ones past that rule: layers,
# sequences, query heads, kv heads, head dim, type, tokens per cluster, clusters selected, tail rows, waves a unit
WAVE_SHAPES = [
    (32, 1, 32, 32, 128, "bf16", 4, 16, 0, 1),   # 64 rows of 256 B, the longest list of rows
    (32, 1, 32, 32, 128, "bf16", 4, 15, 3, 1),   # with a tail in a cluster of its own
    (32, 1, 32, 32, 128, "bf16", 1, 63, 1, 1),   # 64 entries
    (32, 1, 32, 32, 128, "bf16", 1, 64, 1, 8),   # 65: a workgroup
    (32, 1, 32, 32, 128, "bf16", 5, 13, 0, 8),   # 65 rows: a workgroup
    (32, 2, 16, 16, 64, "fp16", 7, 18, 0, 1),    # 126 rows of 128 B, clusters that no load step divides
    (32, 1, 64, 32, 64, "bf16", 16, 2, 0, 1),    # two query heads a row
    (33, 1, 32, 32, 128, "fp32", 3, 10, 2, 8),   # 33 slots of 512 B, the tail's among them: a workgroup
    (33, 1, 33, 33, 128, "fp32", 3, 9, 2, 1),    # 30, a last workgroup of one unit
    (32, 1, 64, 32, 128, "fp32", 32, 1, 0, 1),
]


@pytest.mark.parametrize("shape", WAVE_SHAPES)
def test_short_lists_match_oracle(shape):
    test_splits_match_oracle((*shape[:-1], 1), shape[-1])
