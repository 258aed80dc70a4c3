"""The eviction's top-k at the edges of its dispatch: the kept set against a stable sort of the token scores
that the same call returns (equal scores: lowest position first), so every comparison is exact.
"""
import numpy as np
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu


# older tokens on both sides of each thread-count boundary and of the register / streaming one, odd prompt
# lengths (unaligned score rows of the second head), few and all tokens wanted
SIZES = [(40, 8), (1032, 300), (1033, 1000), (2057, 5), (4105, 2000), (8201, 8192), (16393, 333), (32776, 16000),
         (32777, 9001), (70001, 69993), (131080, 32768)]


@pytest.mark.parametrize("kind", ["distinct", "ties", "equal"])
@pytest.mark.parametrize("T,n_sel", SIZES)
def test_topk_is_a_stable_sort(T, n_sel, kind):
    import paper_2501_06807_amd as M
    loc, d, W = 8, 64, 3
    keep = n_sel + loc
    say(f"[top-k] T={T} keep={keep} {kind}")
    g = torch.Generator(device="cuda").manual_seed(T + n_sel)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    q, v = rand(1, 1, 2, W, d), rand(1, 1, 2, T, d)
    if kind == "distinct":
        k = rand(1, 1, 2, T, d)
    else:  # seven distinct keys, or one: many tokens share a score, without a mask exactly
        pool = rand(7 if kind == "ties" else 1, d)
        k = pool[torch.randint(len(pool), (1, 1, 2, T), generator=g, device="cuda")]
    kept = torch.full((1, 1, 2, keep), -1, dtype=torch.int32, device="cuda")
    k_out = torch.empty((1, 1, 2, keep, d), dtype=torch.bfloat16, device="cuda")
    v_out, score = torch.empty_like(k_out), torch.zeros((1, 1, 2, T), dtype=torch.float32, device="cuda")
    M.mpc_static_evict(q, k.contiguous(), v, kept, k_out, v_out, keep=keep, local_keep=loc, sm_scale=0.125,
                       causal=False, token_score=score)
    torch.cuda.synchronize()
    s = score.cpu().numpy()
    for h in range(2):
        assert kind != "equal" or len(np.unique(s[0, 0, h])) == 1
        best = np.argsort(-s[0, 0, h, :T - loc], kind="stable")[:n_sel]
        want = np.concatenate([np.sort(best), np.arange(T - loc, T)])
        np.testing.assert_array_equal(kept[0, 0, h].cpu().numpy(), want)
