"""Rounding of the 16-bit row pass where it can be told apart: how many terms are summed in fp32, and how far a term's
exponent may lie from the row's offset. Log-sum-exps near zero, so that their own rounding does not hide it.
"""
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
