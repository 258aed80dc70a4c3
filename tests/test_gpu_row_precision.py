"""Rounding of the 16-bit row pass where it can be told apart: how many terms are summed in fp32, and how far a term's
exponent may lie from the row's offset. Log-sum-exps near zero, so that their own rounding does not hide it. Then scores
that are not finite, in every form of the row pass.
"""
import math

import numpy as np
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu

# heads enough that no row block's keys are split over workgroups
B, H, D = 16, 64, 64
SM = 0.6931  # about ln 2: scores are exponents of two
C = float(np.float32(np.float64(np.float32(SM)) * 1.4426950408889634))  # the kernels' exponent scale


def _row_lse(q, k, dtype):
    """Row log-sum-exps of the non-zero leading channels q [B][H][W][c] and k [T][c] (the same keys for every head)."""
    import paper_2501_06807_amd as M
    W, T, c = q.shape[2], k.shape[0], k.shape[1]
    qt = torch.zeros((1, B, H, W, D), dtype=dtype, device="cuda")
    kt = torch.zeros((1, B, H, T, D), dtype=dtype, device="cuda")
    qt[..., :c] = q.cuda()
    kt[..., :c] = k.cuda()
    assert torch.equal(qt[0, ..., :c].cpu().double(), q.double()) and torch.equal(kt[0, 0, 0, :, :c].cpu().double(), k.double())
    kept = torch.zeros((1, B, H, 1), dtype=torch.int32, device="cuda")
    out = torch.empty((1, B, H, 1, D), dtype=dtype, device="cuda")
    lse = torch.zeros((1, B, H, W), dtype=torch.float32, device="cuda")
    M.mpc_static_evict(qt, kt, kt, kept, out, torch.empty_like(out), keep=1, local_keep=0, sm_scale=SM, causal=True,
                       row_lse=lse)
    torch.cuda.synchronize()
    return lse[0].double().cpu().numpy()


def _exact(q, k):
    """The same in fp64, every key visible to every row."""
    x = (q.double().numpy() @ k.double().numpy().T) * C  # exponents of two
    return np.log(np.exp2(x).sum(-1))


@pytest.mark.parametrize("T", [63, 64, 128])  # a masked tile, a full one, two
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16], ids=str)
def test_fp32_sums_hold_at_most_16_terms(T, dtype):
    """One term of 1 and T - 1 of 2^-24.5, which fp32 drops beside the 1: a sum of n terms loses n - 1 of them. At most
    16 terms to a sum lose 15; the rounding of the log-sum-exp itself is far below that here."""
    say(f"[fp32 sums] T={T} {dtype}")
    k = torch.full((T, 1), -24.5)
    k[0] = 0.0
    k = k.to(dtype).float()
    q = torch.ones((B, H, 1, 1))
    err = np.abs(_row_lse(q, k, dtype) - _exact(q, k))
    assert err.max() <= 16 * 2.0**-24.5, err.max()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16], ids=str)
def test_exponents_stay_at_most_one(dtype):
    """A key of the first 64 scores about six binary orders below one further on, which then holds nearly all of the
    row's sum. With its exponent in (-1, 1], as an offset at the maximum gives, the exponent's rounding is 1.2e-8 rms of
    the sum (half of 2^-24, uniform, times ln 2); the hardware exponential is off by one unit in the last place
    at most, about 3.4e-8 rms, and the stored log-sum-exp by 1.3e-8: 4e-8 together. An exponent between 4 and 5 would be
    rounded to 2^-22, 9.5e-8 rms."""
    say(f"[exponents] {dtype}")
    rng = np.random.default_rng(3)
    W, T = 40, 128
    a = torch.from_numpy(rng.integers(129, 256, (B, H, W, 1)) / 256.0).float()  # in (1/2, 1), eight bits
    q = torch.cat([a, torch.ones_like(a)], -1)
    k = torch.zeros((T, 2))
    k[:, 1] = -48.0                       # below fp32's reach beside the others
    k[3, 1] = -6.0625
    k[70] = torch.tensor([-0.9, 0.0]).to(dtype).float()  # scores in (-0.9, -0.45)
    err = _row_lse(q, k, dtype) - _exact(q, k)
    rms = float(np.sqrt((err**2).mean()))
    say(f"  rms error {rms:.2e}, largest {np.abs(err).max():.2e}")
    assert rms <= 5.5e-8


@pytest.mark.parametrize("heads,T,W", [(2, 1025, 150), (512, 200, 40)], ids=["split", "whole"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32], ids=str)
def test_rows_that_see_a_nan_are_nan_and_minus_infinity_adds_nothing(heads, T, W, dtype):
    """A NaN key makes every row that sees it NaN, wherever its tile, lane or workgroup, and leaves the others alone; a
    score of -infinity, at the start of a row or later, has weight zero."""
    import paper_2501_06807_amd as M
    say(f"[not finite] heads={heads} T={T} W={W} {dtype}")
    gen = torch.Generator().manual_seed(5)
    q = torch.randn((1, 1, heads, W, D), generator=gen).to(dtype)
    q[..., 0] = q[..., 0].abs() + 0.5
    k = torch.randn((1, 1, heads, T, D), generator=gen).to(dtype)
    sm = 1 / math.sqrt(D)
    for kind, keys in (("nan", [T - W // 2]), ("nan", [T - W // 2 + 7]), ("nan", [T - 1]), ("nan", [3]), ("-inf", [0]),
                       ("-inf", list(range(40)) + [T - W, T - 2])):
        kk = k.clone()
        kk[..., keys, 0] = float(kind)
        s = (q[0, 0].double() @ kk[0, 0].double().transpose(1, 2)) * float(np.float32(sm))
        seen = torch.arange(T)[None, :] <= torch.arange(W)[:, None] + T - W
        want = torch.logsumexp(s.masked_fill(~seen, -math.inf), -1)
        qt, kt = q.cuda(), kk.cuda()
        kept = torch.zeros((1, 1, heads, 1), dtype=torch.int32, device="cuda")
        out = torch.empty((1, 1, heads, 1, D), dtype=dtype, device="cuda")
        lse = torch.zeros((1, 1, heads, W), dtype=torch.float32, device="cuda")
        M.mpc_static_evict(qt, kt, kt, kept, out, torch.empty_like(out), keep=1, local_keep=0, sm_scale=sm, causal=True,
                           row_lse=lse)
        torch.cuda.synchronize()
        # the eviction tests' bound on log-sum-exps of such scores
        torch.testing.assert_close(lse[0, 0].double().cpu(), want, rtol=0, atol=6e-6, equal_nan=True, msg=lambda m: f"{kind} {keys[:3]}: {m}")
