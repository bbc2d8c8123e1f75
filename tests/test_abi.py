"""Host-only checks of the C-ABI library: it loads, exports every declared symbol, and its
pure-host entry points behave (no GPU needed, no kernels run)."""
import ctypes as C
import os
import re

import pytest

from workload import workload, WORKLOAD_NAMES
from paper_2605_29233_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.lib_path()):
        from paper_2605_29233_amd.build import build
        build()
    return binding.load_library()


def test_exports_every_declared_symbol(lib):
    hdr = open(os.path.join(ROOT, "include", "blockbatch.h")).read()
    declared = set(re.findall(r"\b(bb_[a-z0-9_]+)\s*\(", hdr))
    assert {"bb_load_weights", "bb_refresh", "bb_denoise_step", "bb_merge_commit"} <= declared
    for name in declared:
        assert hasattr(lib, name), f"{name} is declared in blockbatch.h but not exported"
    assert set(binding.EXPORTS) == declared


def _cfg(w):
    m = w.model
    mc = binding.bb_model_cfg(m.n_layers, m.d_model, m.n_q_heads, m.n_kv_heads, m.head_dim, m.d_ffn, m.vocab,
                              m.rope_base, m.rms_eps, int(m.qkv_bias), m.mask_id)
    L = max(w.prompt_lens) + w.gen_len
    lim = binding.bb_limits(w.n_requests, len(w.block_sizes), L, w.gen_len, w.n_requests * sum(w.block_sizes))
    return mc, lim


@pytest.mark.parametrize("name", WORKLOAD_NAMES)
def test_workspace_bytes_covers_weights_and_cache(lib, name):
    w = workload(name)
    mc, lim = _cfg(w)
    n = lib.bb_workspace_bytes(C.byref(mc), C.byref(lim))
    m = w.model
    per_layer = ((m.n_q_heads + 2 * m.n_kv_heads) * m.head_dim * m.d_model + m.d_model * m.n_q_heads * m.head_dim
                 + 3 * m.d_ffn * m.d_model)
    weights = 2 * (m.n_layers * per_layer + 2 * m.vocab * m.d_model)
    kv = 2 * 2 * m.n_layers * w.n_requests * (len(w.block_sizes) + 1) * (max(w.prompt_lens) + w.gen_len) * m.n_kv_heads * m.head_dim
    assert n >= weights + kv
    assert n < 230 * 2 ** 30, "must fit one MI355X (288 GB) with room to spare"


def test_struct_sizes_match_header_layout():
    assert C.sizeof(binding.bb_model_cfg) == 11 * 4
    assert C.sizeof(binding.bb_decode_cfg) == 6 * 4
    assert C.sizeof(binding.bb_limits) == 5 * 4
    assert C.sizeof(binding.BranchState) == 10 * 4
    assert C.sizeof(binding.RequestStats) == 9 * 4 + 8 * 40


def test_bad_shapes_are_rejected(lib):
    w = workload("tiny")
    mc, lim = _cfg(w)
    mc.head_dim = 80
    assert lib.bb_workspace_bytes(C.byref(mc), C.byref(lim)) == 0
    mc, lim = _cfg(w)
    lim.max_branches = 9
    assert lib.bb_workspace_bytes(C.byref(mc), C.byref(lim)) == 0
    mc, lim = _cfg(w)
    mc.mask_id = mc.vocab
    assert lib.bb_workspace_bytes(C.byref(mc), C.byref(lim)) == 0
    ctx = C.c_void_p()
    assert lib.bb_create(C.byref(ctx), C.byref(mc), None, C.byref(lim), None, 0, None) == -1
    assert lib.bb_destroy(None) == -1
    assert lib.bb_last_error(None) == b"null context"


def test_static_gemm_rejects_bad_sizes_before_touching_a_device(lib):
    """Argument and limit checks of the entry point that allocates nothing run on the host alone."""
    fake = C.c_void_p(4096)                      # never dereferenced: every call below is refused first
    f = lib.bb_gemm_static
    assert f(None, fake, fake, 8, 64, 64, 0, None) == -1
    assert f(fake, fake, fake, 0, 64, 64, 0, None) == -1          # no rows
    assert f(fake, fake, fake, 8, 48, 64, 0, None) == -1          # N not a multiple of 32
    assert f(fake, fake, fake, 8, 64, 24, 0, None) == -1          # K not a multiple of 16
    assert f(fake, fake, fake, 129, 64, 64, 0, None) == -3        # beyond the row limit
    assert f(fake, fake, fake, 8, 4128, 64, 0, None) == -3        # beyond the column limit
    assert f(fake, fake, fake, 8, 2048, 4096, 0, None) == -3      # N * K beyond 4 Mi
    assert f(fake, fake, fake, 8, 64, 64, 5, None) == -3          # k split beyond 4


def test_gemm_plans_cover_k_fit_the_chip_and_the_register_file(lib):
    """Host logic of the launch plans (no device): for every shape the k splits cover all 64-k chunks without an
    empty split, a workgroup holds at most 12 accumulator tiles (the AGPR budget of the wide kernel), the fused
    SwiGLU candidate keeps two tiles per wave, and the tile the query states (rows and columns of a workgroup, as the
    header describes it) gives the number of workgroups it states, at most one per CU and k split."""
    shapes = [(n, k) for n in (512, 4096, 4608, 12288, 24576, 37888, 49152, 49184) for k in (512, 3584, 4096, 12288, 18944)]
    for wide in (False, True):
        for M in (1, 32, 56, 64, 65, 120, 128, 129, 160, 192, 252, 256, 257, 300, 768, 1920, 3072, 4608, 20480):
            for N, K in shapes:
                for fusable in (False, True):
                    p = binding.gemm_plan(M, N, K, wide, fusable)
                    chunks = (K + 63) // 64
                    assert 1 <= p["split_k"] <= 16 and p["nt"] in (1, 2, 3), (M, N, K, p)
                    assert p["split_k"] * p["chunks_per_split"] >= chunks > (p["split_k"] - 1) * p["chunks_per_split"], (M, N, K, p)
                    assert p["nt"] * p["mt"] <= 12, (M, N, K, p)
                    m_tiles, columns = (M + 31) // 32, 128 * p["nt"]
                    if not wide:
                        assert p["mt"] == 4, (M, N, K, p)
                    elif M > 256 and p["nt"] == 2:          # tiles of 128 or 192 rows x 256 columns
                        assert p["mt"] in (4, 6), (M, N, K, p)
                    else:           # a body per number of m-tiles, two groups of them above 128 rows; 384 columns: the body of four
                        groups = (m_tiles + 3) // 4
                        assert p["mt"] == (4 if p["nt"] == 3 else (m_tiles + groups - 1) // groups), (M, N, K, p)
                        if M <= 64 and p["nt"] == 2 and N <= 49152:
                            columns = 192
                    tiles = -(-N // columns) * -(-m_tiles // p["mt"])
                    want = min(tiles * p["split_k"], 256) if wide and M > 256 and p["nt"] == 2 else min(tiles, 256) * p["split_k"]
                    assert p["workgroups"] == want, (M, N, K, p, want)
    # more than 256 rows: tiles of 128 columns (nt == 1) where a small matrix leaves most CUs without work
    for M, N, K, small in ((384, 768, 256, True), (384, 256, 256, True), (384, 256, 688, True), (1400, 768, 256, True), (640, 4096, 512, True),
                           (272, 128, 4096, True), (640, 768, 4096, False), (768, 4096, 4096, False), (1400, 4096, 512, False), (3072, 12288, 4096, False)):
        p = binding.gemm_plan(M, N, K, True)
        assert (p["nt"] == 1) == small and (not small or p["workgroups"] <= 256), (M, N, K, p)
    # the shapes the fused SwiGLU epilogue is used on: gate/up of the refresh and of the 16-request step
    for M in (768, 1920, 3072):
        p = binding.gemm_plan(M, 24576, 4096, True, True)
        assert p["nt"] == 2 and p["split_k"] == 1, p
    with pytest.raises(ValueError):
        binding.gemm_plan(0, 4096, 4096)
    with pytest.raises(ValueError):
        binding.gemm_plan(64, 4100, 4096)


@pytest.mark.parametrize("hq,hkv,hd,L,branches,full", [
    (4, 4, 64, 4096, 1, False),         # 128 workgroups of four tiles
    (4, 4, 64, 2048, 4, False),         # 256: one for each CU
    (4, 4, 64, 2176, 4, True),          # 272
    (32, 32, 128, 768, 1, False),       # 192
    (32, 32, 128, 896, 1, True),        # 224
    (28, 4, 128, 768, 1, False),        # 168
    (28, 4, 128, 1536, 3, True),
    (28, 4, 128, 128, 1, False),        # a wide window of a block step with grouped heads
    (32, 32, 128, 511, 4, False),       # fewer than 512 query rows per branch: a workgroup per tile whatever their number
])
def test_attention_shares_pages_in_a_workgroup_only_with_more_workgroups_than_cus(lib, hq, hkv, hd, L, branches, full):
    mc = binding.bb_model_cfg(2, 256, hq, hkv, hd, 256, 1024, 10000.0, 1e-5, 0, 1023)
    lim = binding.bb_limits(1, 4, 4160, 64, 256)
    rows, out = (C.c_int * branches)(*([L] * branches)), (C.c_int * 2)()
    assert lib.bb_debug_attention_plan(C.byref(mc), C.byref(lim), rows, branches, L, out) == 0
    assert (out[1] == 0) == full and out[0] >= 1 and out[1] in (0, 4, 8)
    rows[0] = 0
    assert lib.bb_debug_attention_plan(C.byref(mc), C.byref(lim), rows, branches, L, out) == -1
