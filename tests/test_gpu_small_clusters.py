"""Cluster representatives of small super-clusters (a wave each where there are many): bit-exact against the oracle, both from a
kept cache and gathered inside the prefill, where the dispatch and the last cluster can go wrong.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import bits_to_torch, build_form, say, torch_to_bits

pytestmark = pytest.mark.gpu

# tokens per cluster, fan-out, kept tokens: whole and partial last clusters and super-clusters, one row, more than
# four waves' super-clusters, clusters shorter than a load of rows and super-clusters longer than four loads. Few
# super-clusters: the workgroup form takes them all
SHAPES = [(4, 2, 64), (4, 2, 61), (4, 3, 90), (4, 4, 130), (8, 2, 72), (8, 2, 1), (16, 1, 100), (2, 2, 40), (4, 8, 100),
          (12, 1, 83), (32, 1, 70)]


@pytest.mark.parametrize("similarity", ["linear", "maxprod", "mean"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp16", 64), ("fp32", 128), ("fp32", 64)])
def test_small_clusters_match_oracle(dtype, d, similarity):
    import paper_2501_06807_amd as M
    td = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    rng = np.random.default_rng(d + len(similarity))
    for s, f, keep in SHAPES:
        say(f"[small clusters] {dtype} d={d} {similarity} s={s} f={f} keep={keep}")
        L, B, H, T, W = 2, 2, 3, keep + 5, 3
        cfg = M.select_cfg(s, f, 1, 1, share_period=1, similarity=similarity)
        R = M.rep_rows(similarity)
        C = -(-keep // s)
        reps = lambda: (torch.zeros(L, B, H, C, R, d, device="cuda"), torch.zeros(L, B, H, -(-C // f), R, d, device="cuda"))  # noqa: E731
        k = torch_to_bits(torch.from_numpy(rng.standard_normal((L, B, H, T, d)).astype(np.float32)).to(td), dtype)
        kt = bits_to_torch(k, dtype)
        q = torch.from_numpy(rng.standard_normal((L, B, H, W, d)).astype(np.float32)).to(td).cuda()
        kept = torch.zeros((L, B, H, keep), dtype=torch.int32, device="cuda")
        k_out = torch.empty((L, B, H, keep, d), dtype=td, device="cuda")
        v_out = torch.empty_like(k_out)
        cent, scent = reps()
        M.mpc_prefill(q, kt, kt, kept, k_out, v_out, cent, scent, cfg, keep=keep, local_keep=1, sm_scale=0.1)
        cent2, scent2 = reps()
        M.mpc_build_clusters(k_out, cent2, scent2, cfg)
        torch.cuda.synchronize()
        assert torch.equal(k_out, kt.gather(3, kept.long()[..., None].expand(-1, -1, -1, -1, d)))
        assert torch.equal(v_out, k_out)
        want = oracle.build_clusters(torch_to_bits(k_out, dtype), dtype, cluster=s, fanout=f, similarity=similarity)
        for got in ((cent, scent), (cent2, scent2)):
            for g, r in zip(got, want):
                np.testing.assert_array_equal(g.cpu().numpy().reshape(r.shape), r)


# clusters per super-cluster, super-clusters per head of 256 heads, rows missing from the last, whether a wave each: both
# sides of the two limits (2048 super-clusters of one or two clusters, 32768 of three or four)
MANY = [(2, 8, 0, True), (2, 8, 3, True), (2, 7, 0, False), (1, 9, 1, True), (4, 128, 1, True), (3, 128, 0, True), (4, 20, 0, False)]


@pytest.mark.parametrize("similarity", ["linear", "maxprod", "mean"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp16", 64), ("fp32", 128), ("fp32", 64)])
def test_many_small_clusters_match_oracle(dtype, d, similarity):
    import paper_2501_06807_amd as M
    td = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    s = 64 * 16 // (d * td.itemsize)  # rows of one load, the shortest cluster of the wave form
    torch.manual_seed(d + len(similarity))
    for f, n_sup, missing, wave in MANY:
        say(f"[many small clusters] {dtype} d={d} {similarity} s={s} f={f} n_sup={n_sup} missing={missing}")
        L, B, H, W = 2, 2, 64, 2
        keep = n_sup * f * s - missing
        cfg = M.select_cfg(s, f, 1, 1, share_period=1, similarity=similarity)
        R, C = M.rep_rows(similarity), -(-keep // s)
        kt = torch.randn(L, B, H, keep + 3, d, dtype=td, device="cuda")
        q = torch.randn(L, B, H, W, d, dtype=td, device="cuda")
        assert build_form(M.dims_of(q, kt, 0), keep, cfg) == wave
        kept = torch.zeros((L, B, H, keep), dtype=torch.int32, device="cuda")
        k_out = torch.empty((L, B, H, keep, d), dtype=td, device="cuda")
        v_out = torch.empty_like(k_out)
        reps = lambda: (torch.zeros(L, B, H, C, R, d, device="cuda"), torch.zeros(L, B, H, n_sup, R, d, device="cuda"))  # noqa: E731
        cent, scent = reps()
        M.mpc_prefill(q, kt, kt, kept, k_out, v_out, cent, scent, cfg, keep=keep, local_keep=1, sm_scale=0.1)
        cent2, scent2 = reps()
        M.mpc_build_clusters(k_out, cent2, scent2, cfg)
        torch.cuda.synchronize()
        assert torch.equal(k_out, kt.gather(3, kept.long()[..., None].expand(-1, -1, -1, -1, d)))
        assert torch.equal(v_out, k_out)
        want = oracle.build_clusters(torch_to_bits(k_out, dtype), dtype, cluster=s, fanout=f, similarity=similarity)
        for got in ((cent, scent), (cent2, scent2)):
            for g, r in zip(got, want):
                np.testing.assert_array_equal(g.cpu().numpy().reshape(r.shape), r)
