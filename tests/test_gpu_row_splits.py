"""GPU parity of the eviction's scoring passes where keys (row pass) or window rows (column pass) are split over
several workgroups, and where the row offsets have to move: log-sum-exps and token scores against the oracle.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import bits_to_torch, say, torch_to_bits

pytestmark = pytest.mark.gpu


def _evict(q, k, v, dtype, keep, causal, sm):
    import paper_2501_06807_amd as M
    L, B, Hkv, T, d = k.shape
    Hq, W = q.shape[2:4]
    qt, kt, vt = (bits_to_torch(x, dtype) for x in (q, k, v))
    kept = torch.zeros((L, B, Hkv, keep), dtype=torch.int32, device="cuda")
    k_out = torch.empty((L, B, Hkv, keep, d), dtype=kt.dtype, device="cuda")
    v_out = torch.empty_like(k_out)
    score = torch.zeros((L, B, Hkv, T), dtype=torch.float32, device="cuda")
    lse = torch.zeros((L, B, Hq, W), dtype=torch.float32, device="cuda")
    cfg = M.MpcEvictCfg(window=W, keep=keep, local_keep=8, sm_scale=sm, causal=int(causal), share_period=1, share_start=2)
    need = M.workspace_bytes(M.MPC_OP_STATIC_EVICT, M.dims_of(qt, kt), T, cfg)
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")  # no initial contents needed
    M.mpc_static_evict(qt, kt, vt, kept, k_out, v_out, keep=keep, local_keep=8, sm_scale=sm, causal=causal,
                       token_score=score, row_lse=lse, ws=ws)
    torch.cuda.synchronize()
    return need, kept.cpu().numpy(), torch_to_bits(k_out, dtype), score.cpu().numpy(), lse.cpu().numpy()


def _bits(x, dtype):
    td = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    return torch_to_bits(torch.from_numpy(x).to(td), dtype)


# T, W, query heads, kv heads, head dim, type, causal, kind. Splits run out of tiles (T below 16 tiles of
# 64 keys), a last split of masked tiles only or of none, ragged tiles, a window of one row and of every
# row, column splits that begin inside a query head's rows, fp32 column workgroups of two waves and of eight, groups of
# several column units with a last one of fewer;
# "rising": each 64-key tile scores about eight binary orders above the one before, so the offsets of
# most tiles have to move; "falling": the first tile holds the maximum.
CASES = [
    (64, 64, 1, 1, 64, "bf16", True, "random"),
    (65, 1, 2, 1, 128, "fp16", True, "random"),
    (300, 300, 2, 2, 128, "bf16", True, "random"),
    (1025, 257, 4, 2, 128, "bf16", True, "random"),
    (1025, 257, 4, 1, 64, "fp16", False, "random"),
    (2111, 130, 2, 2, 64, "fp32", True, "random"),
    (513, 200, 1, 1, 128, "fp32", False, "random"),
    (2111, 400, 4, 4, 64, "fp32", True, "random"),
    (1100, 64, 16, 16, 128, "fp32", False, "random"),
    (257, 130, 8, 1, 128, "bf16", True, "random"),
    (700, 513, 8, 2, 64, "fp16", True, "random"),
    (2000, 20, 100, 100, 64, "bf16", True, "random"),
    (900, 700, 203, 203, 64, "fp16", True, "random"),
    (1025, 1025, 160, 160, 64, "bf16", True, "random"),
    (600, 90, 2, 1, 128, "bf16", True, "rising"),
    (600, 90, 2, 2, 64, "fp16", False, "rising"),
    (500, 300, 1, 1, 64, "fp32", True, "rising"),
    (600, 90, 2, 1, 128, "bf16", True, "falling"),
]


@pytest.mark.parametrize("T,W,Hq,Hkv,d,dtype,causal,kind", CASES)
def test_row_splits_match_oracle(T, W, Hq, Hkv, d, dtype, causal, kind):
    rng = np.random.default_rng(T * 1000 + W)
    q = rng.standard_normal((1, 1, Hq, W, d))
    k = rng.standard_normal((1, 1, Hkv, T, d))
    v = rng.standard_normal((1, 1, Hkv, T, d))
    sm = 1.0 / math.sqrt(d)
    if kind != "random":
        u = np.ones(d) / math.sqrt(d)
        step = (np.arange(T) // 64 - T // 128) * (1.0 if kind == "rising" else -1.0)  # scores on both sides of 0
        q = 0.2 * q + 4.0 * u                                   # q . u close to 4
        k = 0.2 * k + (step * 8 * math.log(2.0) / (4.0 * sm))[:, None] * u
    q, k, v = (_bits(x.astype(np.float32), dtype) for x in (q, k, v))
    keep = max(8, T // 2)
    _, _, _, ref = oracle.static_evict(q, k, v, dtype, keep=keep, local_keep=8, sm_scale=sm, causal=causal,
                                       share_period=1, share_start=2, with_scores=True)
    need, kept, ko, score, lse = _evict(q, k, v, dtype, keep, causal, sm)
    say(f"[row splits] T={T} W={W} Hq={Hq} Hkv={Hkv} d={d} {dtype} causal={causal} {kind}: "
        f"workspace {need}")
    top = float(ref.max())
    # the bound of the eviction tests (scaled scores up to 28 here, so a 32-bit q . k is off by up to
    # about 4e-6 of them); scores far below the largest may underflow in fp32
    np.testing.assert_allclose(score, ref, rtol=2e-5, atol=1e-6 * top if kind != "random" else 0.0)
    for hq in range(Hq):
        for t in sorted({0, 1, W // 2, W - 1} & set(range(W))):
            want = oracle.row_lse(q[0, 0, hq, t], t, W, k[0, 0, hq // (Hq // Hkv)], dtype, sm, causal)
            # the eviction tests' bound, with the 4e-6 above for the large scores
            assert abs(lse[0, 0, hq, t] - want) <= 2e-6 * max(3.0, abs(want)), (hq, t, lse[0, 0, hq, t], want)
    np.testing.assert_array_equal(ko[0, 0, 0], k[0, 0, 0, kept[0, 0, 0]])
