"""Host-side checks of the C ABI library (no GPU): symbols, validation, workspace sizing."""
import ctypes
import re

import pytest

import oracle
from paper_2501_06807_amd import _lib as L

HEADER = "include/mpcache.h"


def declared_functions():
    import os
    src = open(os.path.join(os.path.dirname(__file__), "..", HEADER)).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)  # declarations only, not comment text
    return sorted(set(re.findall(r"\b(mpc_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_function():
    lib = L.lib()
    names = declared_functions()
    assert {"mpc_static_evict", "mpc_build_clusters", "mpc_prefill", "mpc_select_clusters",
            "mpc_sparse_decode_attn", "mpc_decode_step"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_owner_layer_matches_oracle_rule():
    for period in (1, 2, 4):
        for start in (0, 2):
            assert [L.owner_layer(l, period, start) for l in range(40)] == \
                   [oracle.owner_layer(l, period, start) for l in range(40)]


def _dims(**kw):
    d = dict(batch=1, layer0=0, n_layers=2, n_q_heads=8, n_kv_heads=2, head_dim=128, dtype=2)
    d.update(kw)
    return L.MpcDims(**d)


def _status(fn, *args):
    lib = L.lib()
    s = getattr(lib, fn)(*args)
    return s, lib.mpc_last_error().decode()


FAKE = ctypes.c_void_p(1 << 20)  # never dereferenced: validation fails before any launch


@pytest.mark.parametrize("dims,expect", [
    (None, L.MPC_EINVAL),
    (_dims(batch=0), L.MPC_EINVAL),
    (_dims(dtype=7), L.MPC_EINVAL),
    (_dims(n_q_heads=6, n_kv_heads=4), L.MPC_ESHAPE),
    (_dims(head_dim=96), L.MPC_EUNSUPPORTED),
])
def test_dims_validation(dims, expect):
    ref = None if dims is None else ctypes.byref(dims)
    cfg = L.select_cfg(16, 4, 2, 4)
    s, msg = _status("mpc_build_clusters", ref, 256, ctypes.byref(cfg), FAKE, FAKE, FAKE, None)
    assert s == expect and msg


def test_select_budget_validation():
    d = _dims()
    # Ts = 300, s = 32 -> C = 10, f = 4 -> S = 3 (tail 2): the smallest candidate set for
    # k_super = 2 is 2*4 - (4-2) = 6
    ok_cfg = L.select_cfg(32, 4, 2, 6)
    bad_k = L.select_cfg(32, 4, 2, 7)
    bad_super = L.select_cfg(32, 4, 4, 2)
    args = lambda c: ("mpc_select_clusters", ctypes.byref(d), 300, ctypes.byref(c), FAKE, FAKE, FAKE,
                      FAKE, None, None, 0, None)
    assert _status(*args(bad_k))[0] == L.MPC_ESHAPE
    assert _status(*args(bad_super))[0] == L.MPC_ESHAPE
    s, _ = _status("mpc_select_clusters", ctypes.byref(d), 300, ctypes.byref(ok_cfg), None, FAKE, FAKE,
                   FAKE, None, None, 0, None)
    assert s == L.MPC_EINVAL  # q is NULL


def test_unknown_similarity_is_rejected_before_any_launch():
    d = _dims()
    cfg = L.select_cfg(32, 4, 2, 6)
    cfg.similarity = 3
    s, msg = _status("mpc_build_clusters", ctypes.byref(d), 300, ctypes.byref(cfg), FAKE, FAKE, FAKE, None)
    assert s == L.MPC_EINVAL and "similarity" in msg
    s, msg = _status("mpc_select_clusters", ctypes.byref(d), 300, ctypes.byref(cfg), FAKE, FAKE, FAKE, FAKE, None,
                     None, 0, None)
    assert s == L.MPC_EINVAL and "similarity" in msg


def test_unknown_group_rule_is_rejected_before_any_launch():
    d = _dims()
    cfg = L.select_cfg(32, 4, 2, 6)
    cfg.group = 3
    s, msg = _status("mpc_select_clusters", ctypes.byref(d), 300, ctypes.byref(cfg), FAKE, FAKE, FAKE, FAKE, None,
                     None, 0, None)
    assert s == L.MPC_EINVAL and "group" in msg


def test_commonality_validation():
    call = lambda L_, u, k, m, idx=FAKE, out=FAKE: _status("mpc_commonality", L_, u, k, m, idx, out, None)
    s, msg = call(4, 3, 5, 4)
    assert s == L.MPC_ESHAPE and "m " in msg          # m must be below L
    assert call(4, 3, 5, -1)[0] == L.MPC_EINVAL
    assert call(0, 3, 5, 0)[0] == L.MPC_EINVAL
    assert call(4, 3, 1025, 1)[0] == L.MPC_EUNSUPPORTED
    assert call(4, 3, 5, 1, idx=None)[0] == L.MPC_EINVAL


def test_decode_validation_and_workspace():
    d = _dims(n_layers=1, n_q_heads=8, n_kv_heads=8)
    s, _ = _status("mpc_sparse_decode_attn", ctypes.byref(d), 256, 0, 16, FAKE, FAKE, FAKE, FAKE, 8, 17, 0.1,
                   FAKE, None, None, 0, None)
    assert s == L.MPC_ESHAPE  # 17 clusters > C = 16
    d3 = _dims(n_layers=1, n_q_heads=24, n_kv_heads=8)
    s, _ = _status("mpc_sparse_decode_attn", ctypes.byref(d3), 256, 0, 16, FAKE, FAKE, FAKE, FAKE, 8, 4, 0.1,
                   FAKE, None, None, 0, None)
    assert s == L.MPC_EUNSUPPORTED  # group of 3
    # one list per kv head (2) or per q-head (8); anything else is a shape error
    d4 = _dims(n_layers=1, n_q_heads=8, n_kv_heads=2)
    s, msg = _status("mpc_sparse_decode_attn", ctypes.byref(d4), 256, 0, 16, FAKE, FAKE, FAKE, FAKE, 4, 4, 0.1,
                     FAKE, None, None, 0, None)
    assert s == L.MPC_ESHAPE and "sel_heads" in msg
    # few units and enough tokens -> split-K -> a workspace is required (validation fails before
    # any launch, so the fake pointers are never used)
    need = L.workspace_bytes(L.MPC_OP_DECODE_ATTN, d, 256)
    assert need > 0
    s, msg = _status("mpc_sparse_decode_attn", ctypes.byref(d), 256, 0, 16, FAKE, FAKE, FAKE, FAKE, 8, 16, 0.1,
                     FAKE, None, None, 0, None)
    assert s == L.MPC_EWORKSPACE and str(need) in msg
    # the workspace size serves one list per kv head and one per q-head alike
    g = _dims(n_layers=1, n_q_heads=8, n_kv_heads=2)
    need_g = L.workspace_bytes(L.MPC_OP_DECODE_ATTN, g, 256)
    for heads in (2, 8):
        s, msg = _status("mpc_sparse_decode_attn", ctypes.byref(g), 256, 0, 16, FAKE, FAKE, FAKE, FAKE, heads, 16,
                         0.1, FAKE, None, None, 0, None)
        assert s == L.MPC_EWORKSPACE and str(need_g) in msg
    # many units -> no split -> no workspace
    big = _dims(n_layers=32, batch=4, n_q_heads=32, n_kv_heads=32)
    assert L.workspace_bytes(L.MPC_OP_DECODE_ATTN, big, 9824) == 0


def test_decode_step_validation_and_workspace():
    big = _dims(n_layers=32, batch=4, n_q_heads=32, n_kv_heads=32)
    cfg = L.select_cfg(32, 8, 20, 15, share_period=4, share_start=2)
    need = L.workspace_bytes(L.MPC_OP_DECODE_STEP, big, 9824, cfg)
    owners = sum(1 for l in range(32) if oracle.owner_layer(l, 4, 2) == l)
    assert owners == 10
    assert need >= 16 + owners * 4 * 32 * 4  # counters + one flag per owner head
    call = lambda d, c, ws, nb: _status(
        "mpc_decode_step", ctypes.byref(d), 9824, 0, ctypes.byref(c), FAKE, FAKE, FAKE, FAKE, FAKE, 0.088, FAKE,
        None, FAKE, None, ws, nb, None)
    s, msg = call(big, cfg, None, 0)
    assert s == L.MPC_EWORKSPACE and str(need) in msg
    assert call(big, cfg, FAKE, need - 1)[0] == L.MPC_EWORKSPACE
    assert call(big, L.select_cfg(32, 8, 20, 161, share_period=4), FAKE, need)[0] == L.MPC_ESHAPE
    assert call(big, L.select_cfg(32, 8, 40, 15, share_period=4), FAKE, need)[0] == L.MPC_ESHAPE
    d3 = _dims(n_layers=32, batch=4, n_q_heads=96, n_kv_heads=32)
    assert call(d3, cfg, FAKE, need)[0] == L.MPC_EUNSUPPORTED  # group of 3
    # a small block also needs the split-K partials of the sequential fallback
    small = _dims(n_layers=1, n_q_heads=8, n_kv_heads=8)
    scfg = L.select_cfg(16, 4, 2, 4)
    assert L.workspace_bytes(L.MPC_OP_DECODE_STEP, small, 256, scfg) >= \
        L.workspace_bytes(L.MPC_OP_DECODE_ATTN, small, 256) > 0


def test_static_evict_validation_and_workspace():
    d = _dims(n_layers=4, batch=1, n_q_heads=8, n_kv_heads=2)
    cfg = L.MpcEvictCfg(window=100, keep=200, local_keep=32, sm_scale=0.088, causal=1, share_period=2,
                        share_start=2)
    need = L.workspace_bytes(L.MPC_OP_STATIC_EVICT, d, 1000, cfg)
    rows = 4 * 8 * 100 * 8
    assert need >= rows + 4 * 2 * 1000 * 4
    call = lambda c, ws, nb: _status("mpc_static_evict", ctypes.byref(d), 1000, ctypes.byref(c), FAKE, FAKE,
                                     FAKE, FAKE, FAKE, FAKE, None, None, ws, nb, None)
    assert call(cfg, None, 0)[0] == L.MPC_EWORKSPACE
    assert call(cfg, FAKE, need - 1)[0] == L.MPC_EWORKSPACE
    bad = L.MpcEvictCfg(window=100, keep=2000, local_keep=32, sm_scale=0.088, causal=1, share_period=2,
                        share_start=2)
    assert call(bad, FAKE, need)[0] == L.MPC_ESHAPE
    bad2 = L.MpcEvictCfg(window=100, keep=200, local_keep=32, sm_scale=float("nan"), causal=1,
                         share_period=2, share_start=2)
    assert call(bad2, FAKE, need)[0] == L.MPC_EINVAL
    misaligned = ctypes.c_void_p((1 << 20) + 4)
    s, _ = _status("mpc_static_evict", ctypes.byref(d), 1000, ctypes.byref(cfg), misaligned, FAKE, FAKE, FAKE,
                   FAKE, FAKE, None, None, FAKE, need, None)
    assert s == L.MPC_EINVAL


def test_evict_workspace_of_the_longest_prompt_serves_the_shorter_ones():
    """The workspace of a block covers every block of no more tokens, window rows, layers, sequences or heads
    (a program makes it once, for its longest prompt), and a block whose rows and scores fit the static scratch
    array stays inside it."""
    def need(n_layers, batch, n_q_heads, n_kv_heads, T, W):
        d = _dims(n_layers=n_layers, batch=batch, n_q_heads=n_q_heads, n_kv_heads=n_kv_heads)
        cfg = L.MpcEvictCfg(window=W, keep=32, local_keep=32, sm_scale=0.088, causal=1, share_period=1, share_start=2)
        base = n_layers * batch * (n_q_heads * W * 8 + n_kv_heads * T * 4)
        got = L.workspace_bytes(L.MPC_OP_STATIC_EVICT, d, T, cfg)
        assert got >= base and (got <= 32 << 20 or base > (32 << 20) - 512), (n_layers, batch, T, W, got)
        return got

    for n_layers, batch, hq, hkv in ((1, 1, 2, 2), (1, 1, 32, 32), (1, 1, 32, 8), (4, 1, 32, 8), (12, 1, 12, 12), (4, 4, 32, 32)):
        for share in (5, 10):
            lengths = [64, 300, 512, 700, 1023, 2048, 3000, 4111, 7177, 8192, 16000, 32768, 40000, 131072]
            sizes = [need(n_layers, batch, hq, hkv, T, max(1, T // share)) for T in lengths]
            assert sizes == sorted(sizes), (n_layers, batch, hq, hkv, share, sizes)
    for T in (512, 7177, 32768):
        for grow in ([need(n, 1, 32, 32, T, T // 5) for n in (1, 2, 3, 4, 8)], [need(1, n, 32, 32, T, T // 5) for n in (1, 2, 3, 4, 8)],
                     [need(1, 1, h, h, T, T // 5) for h in (1, 2, 8, 12, 32, 64)], [need(1, 1, 32, 32, T, W) for W in (1, 9, 100, 512)]):
            assert grow == sorted(grow), (T, grow)


def test_evict_workspace_of_small_blocks_is_small():
    """The room for split passes is what sixteen splits of the block's rows or keys can take, not a fixed size."""
    for n_layers, hq, hkv, T, W in ((1, 12, 12, 512, 102), (1, 2, 2, 64, 12), (1, 32, 8, 300, 60), (1, 2, 2, 3000, 600), (12, 12, 12, 64, 12)):
        d = _dims(n_layers=n_layers, n_q_heads=hq, n_kv_heads=hkv)
        cfg = L.MpcEvictCfg(window=W, keep=32, local_keep=32, sm_scale=0.088, causal=1, share_period=1, share_start=2)
        base = n_layers * (hq * W * 8 + hkv * T * 4)
        got = L.workspace_bytes(L.MPC_OP_STATIC_EVICT, d, T, cfg)
        assert got <= base + 16 * n_layers * max(hq * W * 16, hkv * T * 8) + 512, (n_layers, hq, hkv, T, W, got)


def test_prefill_validation():
    d = _dims(n_layers=4, batch=1, n_q_heads=8, n_kv_heads=2)
    ecfg = L.MpcEvictCfg(window=100, keep=200, local_keep=32, sm_scale=0.088, causal=1, share_period=2,
                         share_start=2)
    need = L.workspace_bytes(L.MPC_OP_STATIC_EVICT, d, 1000, ecfg)

    def call(e, c, ws=FAKE, nb=need, cent=FAKE):
        return _status("mpc_prefill", ctypes.byref(d), 1000, e, c, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, cent, FAKE,
                       None, None, ws, nb, None)[0]

    good = L.select_cfg(16, 4, 2, 4, share_period=2)
    assert call(None, ctypes.byref(good)) == L.MPC_EINVAL
    assert call(ctypes.byref(ecfg), None) == L.MPC_EINVAL
    assert call(ctypes.byref(ecfg), ctypes.byref(good), ws=None, nb=0) == L.MPC_EWORKSPACE
    assert call(ctypes.byref(ecfg), ctypes.byref(good), nb=need - 1) == L.MPC_EWORKSPACE
    assert call(ctypes.byref(ecfg), ctypes.byref(good), cent=None) == L.MPC_EINVAL
    assert call(ctypes.byref(ecfg), ctypes.byref(good), cent=ctypes.c_void_p((1 << 20) + 4)) == L.MPC_EINVAL
    bad_sim = L.select_cfg(16, 4, 2, 4, share_period=2)
    bad_sim.similarity = 9
    assert call(ctypes.byref(ecfg), ctypes.byref(bad_sim)) == L.MPC_EINVAL
    bad_alpha = L.select_cfg(16, 4, 2, 4, alpha=1.5, share_period=2)
    assert call(ctypes.byref(ecfg), ctypes.byref(bad_alpha)) == L.MPC_EINVAL
    bad_keep = L.MpcEvictCfg(window=100, keep=2000, local_keep=32, sm_scale=0.088, causal=1, share_period=2,
                             share_start=2)
    assert call(ctypes.byref(bad_keep), ctypes.byref(good)) == L.MPC_ESHAPE


def test_decode_step_forms():
    """Which form a decode step takes, on both sides of each limit of the rule."""
    from gpu_util import step_form

    def form(units, rows, dtype=2, group="sum", G=1, d=128):
        dims = _dims(n_layers=units, n_q_heads=G, n_kv_heads=1, head_dim=d, dtype=dtype) if units <= 256 else \
            _dims(n_layers=units // 8, n_q_heads=8 * G, n_kv_heads=8, head_dim=d, dtype=dtype)
        cfg = L.select_cfg(16, 4, 64, rows // 16, share_period=1, group=group)
        return step_form(dims, 4096, cfg)

    assert form(256, 1024) == ("self-selecting", 1, 8)
    assert form(32, 384) == ("self-selecting", 1, 8)       # three steps of a workgroup
    assert form(32, 400) == ("self-selecting", 4, 8)
    assert form(128, 512) == ("self-selecting", 2, 8)      # 256 workgroups
    assert form(136, 512) == ("self-selecting", 1, 8)      # no room for a second
    assert form(144, 3200, dtype=0) == ("two kernels", 3, 8)  # 432: two to a compute unit
    assert form(8, 192, dtype=0, G=8) == ("self-selecting", 1, 8)
    assert form(8, 208, dtype=0, G=8) == ("self-selecting", 4, 8)
    assert form(8, 384, G=4, d=64) == ("self-selecting", 1, 8)  # matrix-core scores: 128 rows a step of either width
    assert form(8, 400, G=4, d=64) == ("self-selecting", 4, 8)
    assert form(8, 768, G=2, d=64) == ("self-selecting", 1, 8)
    assert form(8, 784, G=2, d=64) == ("self-selecting", 4, 8)
    assert form(264, 256) == ("claiming", 1, 8)            # 64 KiB a list
    assert form(264, 240) == ("two kernels", 1, 8)
    assert form(512, 256) == ("claiming", 1, 8)
    assert form(520, 256) == ("two kernels", 1, 8)
    assert form(264, 512, d=64) == ("claiming", 1, 8)
    assert form(264, 496, d=64) == ("two kernels", 1, 8)
    assert form(264, 128, dtype=0) == ("claiming", 1, 8)
    assert form(264, 256, G=2, group="head") == ("two kernels", 1, 8)
    assert form(1024, 64) == ("two kernels", 1, 1)         # a wave per list of at most 16 KiB
    assert form(1024, 80) == ("two kernels", 1, 8)


def test_decode_plan_of_very_large_clusters():
    """List sizes in bytes go past 32 bits: one cluster of 2^23 or 2^24 rows (cut off at the cached rows) is not a
    short list, and gets a workgroup per unit."""
    from gpu_util import step_form
    for log2, dtype, d in ((23, 2, 128), (24, 2, 128), (23, 0, 128), (24, 1, 64), (25, 1, 64), (29, 1, 64)):
        dims = _dims(n_layers=128, n_q_heads=8, n_kv_heads=8, head_dim=d, dtype=dtype)
        assert step_form(dims, 1000, L.select_cfg(1 << log2, 1, 1, 1))[1:] == (1, 8), (log2, dtype, d)


def test_status_strings():
    lib = L.lib()
    for s in range(6):
        assert lib.mpc_status_string(s)


def test_append_validation():
    cfg = L.select_cfg(16, 4, 2, 4)
    call = lambda d, Ts, nt, c=cfg: _status("mpc_append_kv", ctypes.byref(d), Ts, nt, ctypes.byref(c), FAKE, FAKE,
                                            FAKE, FAKE, FAKE, FAKE, None, None, None)
    d = _dims(kv_capacity=300)
    s, msg = call(d, 250, 3)
    assert s == L.MPC_ESHAPE and "multiple" in msg      # Ts not a multiple of s
    assert call(d, 256, 17)[0] == L.MPC_ESHAPE            # tail longer than a cluster
    assert call(d, 256, -1)[0] == L.MPC_ESHAPE
    assert call(_dims(), 256, 3)[0] == L.MPC_EINVAL       # no capacity given
    # 288 + 12 = 300 rows in use: no row left for the new token
    s, msg = call(d, 288, 12)
    assert s == L.MPC_ESHAPE and "kv_capacity" in msg
    # a full tail at 272 + 16 is sealed first, and the new row 288 still fits
    bad = L.select_cfg(16, 4, 2, 4)
    bad.similarity = 5
    assert call(d, 272, 16, bad)[0] == L.MPC_EINVAL
    ts_out, tail_out = ctypes.c_int32(-5), ctypes.c_int32(-5)
    s, _ = _status("mpc_append_kv", ctypes.byref(d), 272, 16, ctypes.byref(cfg), None, FAKE, FAKE, FAKE, FAKE, FAKE,
                   ctypes.byref(ts_out), ctypes.byref(tail_out), None)
    assert s == L.MPC_EINVAL                               # k_new is NULL
    assert (ts_out.value, tail_out.value) == (-5, -5)      # the new state is written only on success


def test_decode_step_status_validation():
    flags = ctypes.c_int32(-5)
    s, msg = _status("mpc_decode_step_status", None, 1024, 0, ctypes.byref(flags))
    assert s == L.MPC_EINVAL
    assert _status("mpc_decode_step_status", FAKE, 1024, 0, None)[0] == L.MPC_EINVAL
    assert _status("mpc_decode_step_status", FAKE, 2, 1, ctypes.byref(flags))[0] == L.MPC_EWORKSPACE
    assert flags.value == -5


def test_capacity_and_tail_validation():
    d = _dims(n_layers=1, n_q_heads=8, n_kv_heads=8)
    attn = lambda dd, Ts, nt, k=4: _status("mpc_sparse_decode_attn", ctypes.byref(dd), Ts, nt, 16, FAKE, FAKE,
                                           FAKE, FAKE, 8, k, 0.1, FAKE, None, None, 0, None)
    assert attn(d, 250, 3)[0] == L.MPC_ESHAPE             # a tail after a partial cluster
    assert attn(d, 256, -2)[0] == L.MPC_EINVAL
    assert attn(_dims(n_layers=1, n_q_heads=8, n_kv_heads=8, kv_capacity=260), 256, 5)[0] == L.MPC_ESHAPE
    assert attn(_dims(n_layers=1, n_q_heads=8, n_kv_heads=8, kv_capacity=-1), 256, 0)[0] == L.MPC_EINVAL
    big = _dims(n_layers=1, n_q_heads=8, n_kv_heads=8, kv_capacity=20000)
    assert attn(big, 16000, 16 * 30, k=1000)[0] == L.MPC_EUNSUPPORTED  # 1000 + 30 list entries
    cfg = L.select_cfg(16, 4, 2, 4)
    s, msg = _status("mpc_build_clusters", ctypes.byref(_dims(kv_capacity=200)), 256, ctypes.byref(cfg), FAKE,
                     FAKE, FAKE, None)
    assert s == L.MPC_ESHAPE and "kv_capacity" in msg
    ecfg = L.MpcEvictCfg(window=100, keep=200, local_keep=32, sm_scale=0.088, causal=1, share_period=1,
                         share_start=2)
    s, msg = _status("mpc_static_evict", ctypes.byref(_dims(kv_capacity=150)), 1000, ctypes.byref(ecfg), FAKE, FAKE,
                     FAKE, FAKE, FAKE, FAKE, None, None, FAKE, 1 << 30, None)
    assert s == L.MPC_ESHAPE and "kv_capacity" in msg


def test_noalloc_refuses_a_block_beyond_its_scratch():
    """The entry point without allocation refuses, before touching the GPU, a block whose static
    eviction workspace is larger than its static scratch array (all 32 layers of the 8K workload:
    46 MB against 32 MiB)."""
    d = _dims(n_layers=32, n_q_heads=32, n_kv_heads=32)
    T, W = 8192, 1638
    cfg = L.MpcEvictCfg(window=W, keep=4096, local_keep=32, sm_scale=0.088, causal=1, share_period=4, share_start=2)
    lib = L.lib()
    assert L.workspace_bytes(L.MPC_OP_STATIC_EVICT, d, T, cfg) > lib.mpc_static_evict_noalloc_limit() == 32 << 20
    s, msg = _status("mpc_static_evict_noalloc", ctypes.byref(d), T, ctypes.byref(cfg), FAKE, FAKE, FAKE, FAKE, FAKE,
                     FAKE, None, None, None)
    assert s == L.MPC_EWORKSPACE and "scratch" in msg
    # argument errors come first, as in mpc_static_evict
    s, _ = _status("mpc_static_evict_noalloc", ctypes.byref(d), T, ctypes.byref(cfg), None, FAKE, FAKE, FAKE, FAKE,
                   FAKE, None, None, None)
    assert s == L.MPC_EINVAL


def test_layer_block_limit():
    """Calls whose layers share kept sets or selections take at most 256 layers (the owner tables and
    the prefill's per-layer masks are sized for that); a block of 257 is refused before anything runs."""
    d = _dims(n_layers=257, n_q_heads=2, n_kv_heads=1, head_dim=64)
    dc = _dims(n_layers=257, n_q_heads=2, n_kv_heads=1, head_dim=64, kv_capacity=512)
    ecfg = L.MpcEvictCfg(window=32, keep=64, local_keep=8, sm_scale=0.125, causal=1, share_period=3,
                         share_start=2)
    scfg = L.select_cfg(16, 4, 2, 4, share_period=3)
    ws = 1 << 40  # any workspace size passes: the layer count is refused first
    calls = {
        "mpc_static_evict": ("mpc_static_evict", ctypes.byref(d), 160, ctypes.byref(ecfg), FAKE, FAKE, FAKE, FAKE,
                             FAKE, FAKE, None, None, FAKE, ws, None),
        "mpc_static_evict_noalloc": ("mpc_static_evict_noalloc", ctypes.byref(d), 160, ctypes.byref(ecfg), FAKE,
                                     FAKE, FAKE, FAKE, FAKE, FAKE, None, None, None),
        "mpc_build_clusters": ("mpc_build_clusters", ctypes.byref(d), 256, ctypes.byref(scfg), FAKE, FAKE, FAKE, None),
        "mpc_prefill": ("mpc_prefill", ctypes.byref(d), 160, ctypes.byref(ecfg), ctypes.byref(scfg), FAKE, FAKE, FAKE,
                        FAKE, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, ws, None),
        "mpc_select_clusters": ("mpc_select_clusters", ctypes.byref(d), 256, ctypes.byref(scfg), FAKE, FAKE, FAKE,
                                FAKE, None, FAKE, ws, None),
        "mpc_decode_step": ("mpc_decode_step", ctypes.byref(d), 256, 0, ctypes.byref(scfg), FAKE, FAKE, FAKE, FAKE,
                            FAKE, 0.125, FAKE, None, FAKE, None, FAKE, ws, None),
        "mpc_append_kv": ("mpc_append_kv", ctypes.byref(dc), 256, 3, ctypes.byref(scfg), FAKE, FAKE, FAKE, FAKE,
                          FAKE, FAKE, None, None, None),
    }
    for name, args in calls.items():
        s, msg = _status(*args)
        assert s == L.MPC_EUNSUPPORTED and "256" in msg, (name, s, msg)
