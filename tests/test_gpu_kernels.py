"""Kernel-level GPU checks through the C ABI: the MFMA GEMM path (tile edges, split-K, K = 688)
the q|k|v projection under every tile width and k split, and the bit-equality of the input generator on the
two devices."""
import types

import numpy as np
import pytest
import torch

from workload import workload
from workload.configs import ModelShape, DecodeParams
from workload.gen import gen_normal_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bb():
    from paper_2605_29233_amd import BlockBatch, Limits
    shape = ModelShape("gemmtest", 1, 1024, 8, 8, 128, 2752, 4096)
    b = BlockBatch(shape, DecodeParams(), Limits(1, 3, 512, 128, 256))
    yield b
    b.close()


def test_generator_is_bit_identical_on_gpu():
    a = gen_normal_bf16(0, "x", 100003, 0.02, "cpu")
    b = gen_normal_bf16(0, "x", 100003, 0.02, "cuda:0").cpu()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("M,N,K,split", [
    (32, 32, 16, 1), (1, 64, 32, 1), (56, 768, 256, 0), (120, 1376, 256, 0), (37, 256, 688, 0),
    (130, 1024, 256, 0), (128, 4096, 1024, 1), (120, 1024, 2752, 0), (120, 1024, 2752, 3),
    (200, 2752, 1024, 2), (300, 96, 4096, 7),
    (1536, 5632, 128, 0),          # 12 row groups x 176 column tiles: the plan takes 384-column tiles here
])
def test_mfma_gemm_matches_fp64(bb, M, N, K, split):
    rng = np.random.default_rng(M * 7 + N)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Wb = gen_normal_bf16(1, f"w{N}x{K}", N * K, 0.05).view(torch.int16).numpy().view(np.uint16).reshape(N, K)
    W = (Wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    print(f"gemm case M={M} N={N} K={K} split={split}", flush=True)
    C = bb.debug_gemm(A, Wb, split)
    ref = A.astype(np.float64) @ W.T
    scale = np.abs(ref).max()
    err = np.abs(C - ref).max()
    # hi+lo bf16 keeps >= 16 bits of each activation; fp32 accumulation over K terms
    assert err <= 2e-5 * scale * max(1.0, (K / 256) ** 0.5), (err, scale)


@pytest.mark.parametrize("M,N,K,split", [
    (32, 32, 16, 1), (1, 64, 32, 1), (56, 768, 256, 0), (37, 256, 688, 0), (130, 1024, 256, 0),
    (300, 96, 4096, 7), (384, 1376, 256, 0), (700, 4608, 512, 0), (1536, 5632, 128, 0), (3000, 512, 2752, 2),
    # shapes whose plan takes the 192-row workgroup tile: a ragged last row group; k split in four; a number of column
    # tiles that is no multiple of eight
    (3000, 4096, 1024, 0), (740, 4096, 4096, 0), (1100, 4192, 768, 0),
])
def test_wide_format_gemm_matches_fp64(bb, M, N, K, split):
    """The fp16 + fp8 operand kernels: activation = fp16 term + e5m2 remainder,
    weight = row-scaled fp16 (exact) and e4m3.  Per product the error is about 2^-16 relative (e4m3 rounding of
    the weight times the 2^-12 remainder, e5m2 rounding of the remainder), random in sign."""
    rng = np.random.default_rng(M * 11 + N)
    A = (rng.standard_normal((M, K)) * np.exp(rng.uniform(-3, 3, (M, 1)))).astype(np.float32)     # rows of very different size
    Wb = gen_normal_bf16(1, f"w{N}x{K}", N * K, 0.05).view(torch.int16).numpy().view(np.uint16).reshape(N, K).copy()
    Wb[0::7] = ((Wb[0::7].astype(np.uint32) << 16).view(np.float32) * 2.0 ** -12).view(np.uint32) >> 16   # some tiny rows
    W = (Wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    from paper_2605_29233_amd.binding import gemm_plan
    if (M, N, K) in ((3000, 4096, 1024), (740, 4096, 4096), (1100, 4192, 768)):
        assert gemm_plan(M, N, K, wide=True)["mt"] == 6, "this case is here for the 192-row tile"
    print(f"wide gemm case M={M} N={N} K={K} split={split}", flush=True)
    C = bb.debug_gemm(A, Wb, split, wide=True)
    ref = A.astype(np.float64) @ W.T
    # error scale of one output: |a| . |w| (sum of magnitudes), of which a random 2^-15 per term survives
    mag = np.abs(A).astype(np.float64) @ np.abs(W).T
    err = np.abs(C - ref)
    assert (err <= 2.0 ** -13 * mag / np.sqrt(K) * 4 + 1e-30).all(), float((err / (mag + 1e-300)).max())


@pytest.mark.parametrize("M,N,K,split,tile_rows", [
    (257, 32, 64, 1, 128),          # nine m-tiles, one column tile, a single chunk of 64 k: half a unit of the fp8 step
    (289, 288, 192, 1, 128),        # an odd number of chunks, column tiles that are no multiple of eight
    (385, 96, 688, 3, 128),         # splits of four chunks, the last one of three with a padded end
    (520, 512, 1088, 3, 128),       # splits of an odd number of chunks
    (1030, 256, 128, 1, 128),       # one unit; the last row group is one m-tile
    (1190, 4192, 64, 0, 192),       # a single chunk; the last row group has two m-tiles; column tiles that are no multiple of eight
    (1100, 4192, 192, 0, 192),      # three chunks: a unit and a half; the last row group has five m-tiles
    (740, 5664, 1344, 0, 192),      # two splits of 12 and 9 chunks; one column tile over a multiple of eight
])
def test_many_row_gemm_at_the_edges_of_its_tiles(bb, M, N, K, split, tile_rows):
    """Tiles of 256 columns (more than 256 rows) with both tile heights, where units, k splits, row and column groups end:
    against fp64, bound as in test_wide_format_gemm_matches_fp64.  (A forced split takes the 128-row tile.  Without one these
    small matrices take tiles of 128 columns: test_small_matrices_of_many_rows.)"""
    if split == 0:
        from paper_2605_29233_amd.binding import gemm_plan
        p = gemm_plan(M, N, K, wide=True)
        chunks = (K + 63) // 64
        assert p["mt"] == tile_rows // 32, p
        assert p["nt"] == 2, "256 columns"
        assert tile_rows == 128 or (chunks - (p["split_k"] - 1) * p["chunks_per_split"]) % 2, "the 192-row cases end in half a unit"
    rng = np.random.default_rng(M * 13 + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Wb = gen_normal_bf16(2, f"m{N}x{K}", N * K, 0.05).view(torch.int16).numpy().view(np.uint16).reshape(N, K)
    W = (Wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    print(f"many-row gemm case M={M} N={N} K={K} split={split}", flush=True)
    C = bb.debug_gemm(A, Wb, split, wide=True)
    err = np.abs(C - A.astype(np.float64) @ W.T)
    mag = np.abs(A).astype(np.float64) @ np.abs(W).T
    assert (err <= 2.0 ** -13 * mag / np.sqrt(K) * 4 + 1e-30).all(), float((err / (mag + 1e-300)).max())


@pytest.mark.parametrize("M,N,K", [
    (257, 32, 64),              # nine m-tiles: three row groups of three; one column tile, one chunk
    (320, 224, 192),            # ten: 4 + 4 + 2; column tiles that are no multiple of four
    (385, 256, 688),            # k splits of an odd number of chunks with a padded end
    (1030, 768, 1088),          # 33 m-tiles: the last row group has one
    (4096, 96, 256),
    (272, 128, 4096),           # 16 k splits
])
def test_small_matrices_of_many_rows(bb, M, N, K):
    """More than 256 rows over a matrix so small that tiles of 128 columns fit one round: against fp64,
    bound as in test_wide_format_gemm_matches_fp64."""
    from paper_2605_29233_amd.binding import gemm_plan
    assert gemm_plan(M, N, K, wide=True)["nt"] == 1, "128 columns"
    rng = np.random.default_rng(M * 17 + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Wb = gen_normal_bf16(3, f"s{N}x{K}", N * K, 0.05).view(torch.int16).numpy().view(np.uint16).reshape(N, K)
    W = (Wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    print(f"small matrix M={M} N={N} K={K}", flush=True)
    err = np.abs(bb.debug_gemm(A, Wb, 0, wide=True) - A.astype(np.float64) @ W.T)
    mag = np.abs(A).astype(np.float64) @ np.abs(W).T
    assert (err <= 2.0 ** -13 * mag / np.sqrt(K) * 4 + 1e-30).all(), float((err / (mag + 1e-300)).max())


@pytest.mark.parametrize("M,N,K,nt,mt", [
    (129, 32, 64, 1, 3),            # five m-tiles: 3 + 2; one column tile, half a unit
    (160, 96, 688, 1, 3),           # two splits of three units, the last one padded; waves without a column tile
    (193, 32, 1088, 1, 4),          # seven m-tiles: 4 + 3
    (129, 16416, 192, 2, 3),        # a unit and a half; a last column group of one tile
    (256, 16416, 192, 2, 4),
    (225, 32992, 192, 3, 4),        # 384 columns; eight m-tiles, the last one of one row
    # long k ranges: the ring of four chunks goes round more than twice, remainders are fetched nine times into one buffer
    (129, 12288, 1216, 1, 3),       # nine units and a half
    (193, 12288, 1088, 1, 4),       # eight and a half
    (160, 16416, 1216, 2, 3),
    (225, 16416, 1088, 2, 4),
    (192, 32992, 1216, 3, 4),
    (256, 32992, 1088, 3, 4),
    (144, 16416, 1152, 2, 3),       # nine whole units
    (224, 32992, 1024, 3, 4),       # eight
])
def test_two_row_groups_at_the_edges_of_their_tiles(bb, M, N, K, nt, mt):
    """129 to 256 rows: every tile the plan can take, where units, k splits, row and column groups end: against fp64,
    bound as in test_wide_format_gemm_matches_fp64."""
    from paper_2605_29233_amd.binding import gemm_plan
    p = gemm_plan(M, N, K, wide=True)
    assert (p["nt"], p["mt"]) == (nt, mt), p
    rng = np.random.default_rng(M * 19 + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Wb = gen_normal_bf16(4, f"g{N}x{K}", N * K, 0.05).view(torch.int16).numpy().view(np.uint16).reshape(N, K)
    W = (Wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    print(f"two row groups M={M} N={N} K={K}", flush=True)
    err = np.abs(bb.debug_gemm(A, Wb, 0, wide=True) - A.astype(np.float64) @ W.T)
    mag = np.abs(A).astype(np.float64) @ np.abs(W).T
    assert (err <= 2.0 ** -13 * mag / np.sqrt(K) * 4 + 1e-30).all(), float((err / (mag + 1e-300)).max())


@pytest.mark.parametrize("hq,hkv,hd,bias", [(4, 2, 64, True), (2, 1, 128, False), (6, 2, 64, True)])
def test_qkv_projection_gives_the_same_cache_and_logits_under_every_plan(hq, hkv, hd, bias):
    """The q|k|v projection of the block forward with tiles of 128, 256 or 384 columns and with k whole or split in
    two (partial tiles summed by the epilogue kernel that applies bias and RoPE and writes q and the K,V cache):
    every plan must give the same cache and logits up to fp32 summation order, for block sizes with and without
    whole runs of 8 rows, with grouped heads of 64 and 128 dims.  The cache entries of layer 0 come straight from the fp32 sums
    (1e-5 of their scale).  Layer 1's cache and the logits pass through repacked activations: where a different summation
    order flips the rounding of an activation's fp16 term, its e5m2 remainder (3 significant bits) absorbs the half
    ulp only to 2^-3, so one element's operand moves by up to 2^-14 of its value; logits of magnitude 10 may
    therefore differ by a few 1e-4 (measured: 3e-5 of their scale), and the bound below is 2e-4 of the logits' scale."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("qkvtest", 2, 512, hq, hkv, hd, 512, 1024, qkv_bias=bias)
    decode = DecodeParams(0.9, 0.5, 4, 8)
    weights = dict(gen_weights(shape, 3))
    prompt = gen_prompt(shape, 3, 0, 37)
    G, blocks = 48, (4, 8, 16)
    results = {}
    for nt, split in [(1, 2), (1, 1), (2, 1), (3, 1), (2, 2)]:
        print(f"qkv plan nt={nt} split={split} heads={hq}/{hkv} hd={hd}", flush=True)
        b = BlockBatch(shape, decode, Limits(1, 3, 37 + G, G, 32), poison_workspace=True)
        try:
            b.load_weights(weights.items())
            b.keep_logits(True)
            b.set_gemm_plan(3, nt, split)
            rid = b.request_open(prompt, G, blocks)
            b.refresh([rid], BB_INIT)
            b.merge_commit([rid])
            out = []
            for step in range(3):
                v = b.denoise_step([rid])
                out.append(v.logits().copy())
                b.merge_commit([rid])
            kv = [b.get_kv(rid, k, layer) for k in range(3) for layer in range(2)]
            results[(nt, split)] = (out, kv, b.get_tokens(rid))
        finally:
            b.close()
    ref_out, ref_kv, ref_X = results[(1, 2)]
    for key, (out, kv, X) in results.items():
        assert np.array_equal(X, ref_X), key
        for a, r in zip(out, ref_out):
            tol = 2e-4 * max(1.0, float(np.abs(r).max()))
            assert a.shape == r.shape and np.abs(a - r).max() <= tol, (key, np.abs(a - r).max(), tol)
        for i, ((K, V), (Kr, Vr)) in enumerate(zip(kv, ref_kv)):
            rel = 1e-5 if i % 2 == 0 else 1e-4          # layer 0: fp32 sums of identical operands; layer 1: repacked operands
            assert np.abs(K - Kr).max() <= rel * max(1.0, np.abs(Kr).max()), (key, i)
            assert np.abs(V - Vr).max() <= rel * max(1.0, np.abs(Vr).max()), (key, i)


def test_wide_format_forward_agrees_with_two_bf16_terms():
    """A periodic refresh (3 x 150 rows: wide format) followed by block steps of 240 rows (wide format as well) against
    the same calls with the wide format switched off (two bf16 terms everywhere): caches agree to a few 1e-4 of their
    scale (the fp16 + fp8 products are good to about 2^-16 each), logits to well inside the parity tolerance."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT, BB_PERIODIC
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("widetest", 3, 512, 8, 2, 64, 1376 + 16, 2048, qkv_bias=True)      # d_ffn % 64 != 0: padded panels
    decode = DecodeParams(0.9, 0.5, 4, 2)
    weights = dict(gen_weights(shape, 5))
    prompt = gen_prompt(shape, 5, 0, 22)
    G, blocks = 128, (16, 96, 128)
    res = {}
    for wide in (True, False):
        b = BlockBatch(shape, decode, Limits(1, 3, 22 + G, G, 240), poison_workspace=True)
        try:
            b.load_weights(weights.items())
            b.keep_logits(True)
            b.wide_format(wide)
            rid = b.request_open(prompt, G, blocks)
            b.refresh([rid], BB_INIT)
            b.merge_commit([rid])
            outs = []
            for step in range(3):
                v = b.denoise_step([rid])
                assert v.m_q == 240
                outs.append((v.logits().copy(), v.argmax().copy()))
                st = b.merge_commit([rid])[0]
                if st.refresh_due:
                    b.refresh([rid], BB_PERIODIC)
            res[wide] = (outs, [b.get_kv(rid, k, l) for k in range(3) for l in range(3)], b.get_tokens(rid))
        finally:
            b.close()
    (ow, kvw, Xw), (ob, kvb, Xb) = res[True], res[False]
    worst = 0.0
    for (lw, aw), (lb, ab) in zip(ow, ob):
        assert lw.shape == lb.shape
        worst = max(worst, float(np.abs(lw[:, :-1] - lb[:, :-1]).max()))
    print("wide vs two-term: max logit difference", worst, flush=True)
    assert worst <= 5e-3
    for (Kw, Vw), (Kb, Vb) in zip(kvw, kvb):
        assert np.abs(Kw - Kb).max() <= 5e-4 * np.abs(Kb).max() and np.abs(Vw - Vb).max() <= 5e-4 * np.abs(Vb).max()


def test_swiglu_in_the_gemm_epilogue_with_the_deferred_norm_scale():
    """Block steps of at most 128 rows pack the FFN input without its RMSNorm scale; with very many FFN columns the
    gate/up plan has two tiles per wave and k whole, and the wide-format kernel's epilogue then applies SiLU(gate) * up
    itself, scaling both by 1 / rms.  With the wide format off the same forward goes through the two-term kernel and
    the separate SwiGLU kernel: logits agree to well inside the parity tolerance, caches to a few 1e-4 of their scale."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from paper_2605_29233_amd.binding import gemm_plan
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("fusetest", 2, 256, 4, 4, 64, 16640 + 16, 1024, qkv_bias=False)       # d_ffn % 64 != 0 as well
    ngu = (shape.d_ffn + 63) // 64 * 128
    p = gemm_plan(56, ngu, shape.d_model, wide=True)
    assert p["nt"] == 2 and p["split_k"] == 1, p        # the case this test is here for
    decode = DecodeParams(0.9, 0.5, 4, 8)
    weights = dict(gen_weights(shape, 7))
    prompt = gen_prompt(shape, 7, 0, 40)
    G, blocks = 64, (8, 16, 32)
    res = {}
    for wide in (True, False):
        b = BlockBatch(shape, decode, Limits(1, 3, 40 + G, G, 56), poison_workspace=True)
        try:
            b.load_weights(weights.items())
            b.keep_logits(True)
            b.wide_format(wide)
            rid = b.request_open(prompt, G, blocks)
            b.refresh([rid], BB_INIT)
            b.merge_commit([rid])
            outs = []
            for step in range(3):
                v = b.denoise_step([rid])
                outs.append(v.logits().copy())
                b.merge_commit([rid])
            res[wide] = (outs, [b.get_kv(rid, k, l) for k in range(3) for l in range(2)])
        finally:
            b.close()
    for a, r in zip(res[True][0], res[False][0]):
        assert a.shape == r.shape and np.isfinite(a).all()
        assert np.abs(a - r).max() <= 1e-2, np.abs(a - r).max()
    for (K, V), (Kr, Vr) in zip(res[True][1], res[False][1]):
        assert np.abs(K - Kr).max() <= 1e-3 * max(1.0, np.abs(Kr).max())
        assert np.abs(V - Vr).max() <= 1e-3 * max(1.0, np.abs(Vr).max())


@pytest.mark.parametrize("blocks,d_ffn", [
    ((8,), 688),                    # one m-tile, most of its rows padding; an odd number of column tiles per wave and group, padded columns
    ((32,), 1392),                  # one, full
    ((32, 24), 688),                # two, the second with padding rows
    ((64, 32), 1376 + 16),          # three
    ((64, 48, 16), 33024 + 16),     # four; more column groups than workgroups (one each of 256): the halves' place is used again
])
def test_swiglu_across_two_waves_is_the_one_within_a_wave(blocks, d_ffn):
    """The gate/up projection with one column tile per wave and k whole finishes SiLU(gate) * up with halves that two waves swap through
    LDS; with two tiles per wave both factors are in one wave's registers.  Same sums, same expressions: logits and caches equal bit for bit.
    Neither has a SwiGLU launch of its own: the step's launches between the GEMMs are three per layer, the final norm, the vocabulary merge
    and the packing; with the k range in two there is one more per layer.  (Rows of 512 columns: fewer than eight chunks of k are not split.)"""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("swaptest", 2, 512, 4, 4, 64, d_ffn, 1024, qkv_bias=False)
    assert (d_ffn + 63) // 64 * 4 >= 8          # column tiles: with fewer than eight, two per wave would be taken back to one
    weights = dict(gen_weights(shape, 11))
    prompt = gen_prompt(shape, 11, 0, 40)
    G, res, glue = 64, {}, {}
    for nt, split in ((1, 1), (2, 1), (1, 2)):
        b = BlockBatch(shape, DecodeParams(0.9, 0.5, 4, 8), Limits(1, len(blocks), 40 + G, G, sum(blocks)), poison_workspace=True)
        try:
            b.load_weights(weights.items())
            b.keep_logits(True)
            b.set_gemm_plan(2, nt, split)
            rid = b.request_open(prompt, G, blocks)
            b.refresh([rid], BB_INIT)
            b.merge_commit([rid])
            print(f"swiglu swap blocks={blocks} d_ffn={d_ffn} nt={nt} split={split}", flush=True)
            b.profile_enable()
            v = b.denoise_step([rid])
            glue[nt, split] = b.profile_read()["glue"]["launches"]
            res[nt, split] = [v.logits().copy()] + [x for k in range(len(blocks)) for l in range(2) for x in b.get_kv(rid, k, l)]
        finally:
            b.close()
    assert glue == {(1, 1): 9, (2, 1): 9, (1, 2): 11}, glue
    for a, r in zip(res[1, 1], res[2, 1]):
        assert np.isfinite(a[..., :-1]).all() and np.array_equal(a, r)


@pytest.mark.parametrize("M", [1, 31, 33, 63, 65, 95, 97, 128, 129, 160, 191, 193, 256])
@pytest.mark.parametrize("N,K", [(224, 64), (160, 208), (4640, 320), (608, 1040), (33280, 128)])
def test_wide_format_gemm_for_every_number_of_row_tiles(bb, M, N, K):
    """Up to 256 rows the wide-format kernel has a body per number of 32-row tiles (two groups of three or four above 128
    rows), with tiles 128 or 256 columns wide: k ranges of 1, 4, 5 and 17 chunks (less than, equal to and beyond the rings
    of three and four), column counts that fill no tile, rows that fill no 32.  Tolerance as in the test above."""
    rng = np.random.default_rng(M * 13 + N)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Wb = gen_normal_bf16(1, f"w{N}x{K}", N * K, 0.05).view(torch.int16).numpy().view(np.uint16).reshape(N, K)
    W = (Wb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    print(f"wide gemm rows M={M} N={N} K={K}", flush=True)
    err = np.abs(bb.debug_gemm(A, Wb, 0, wide=True) - A.astype(np.float64) @ W.T)
    mag = np.abs(A).astype(np.float64) @ np.abs(W).T
    assert (err <= 2.0 ** -13 * mag / np.sqrt(K) * 4 + 1e-30).all(), float((err / (mag + 1e-300)).max())


@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 97, 129, 161, 225, 257])
def test_lm_head_row_groups(n):
    """n rows receive logits: one to nine m-tiles, each a row group of its own (four column groups; taller row groups: test_lm_head_tiles,
    test_vocabulary_ties_in_every_body_of_the_lm_head).  The launch is sized for the same n rows (fewer live ones than it is
    sized for: test_step_with_fewer_live_rows_than_it_is_sized_for).  Logits against the oracle (fp64);
    token, confidence and log-sum-exp against a reduction of the returned logits in fp64: 1 / c and exp(lse - max) are
    sums of up to 1024 exponentials in fp32, each good to 2 ulp of an argument below 2^7."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    from oracle.model import OracleModel
    from oracle.blockbatch import OracleRequest
    shape = ModelShape("lmtest", 1, 256, 4, 4, 64, 688, 1024)
    decode = DecodeParams(0.9, 0.5, 4, 8)
    weights = dict(gen_weights(shape, 11))
    prompt = gen_prompt(shape, 11, 0, 20)
    print("lm head rows", n, flush=True)
    b = BlockBatch(shape, decode, Limits(1, 1, 20 + 257, 257, 64), poison_workspace=True)
    try:
        b.load_weights(weights.items())
        b.keep_logits(True)
        rid = b.request_open(prompt, n, (32,))
        b.refresh([rid], BB_INIT)
        v = b.latest_view()
        assert v.m_lm == n
        logits, am, conf, lse = v.logits().astype(np.float64), v.argmax(), v.conf(), v.lse()
    finally:
        b.close()
    want = OracleRequest(OracleModel(shape, weights), prompt, n, (32,), decode).init_forward().logits
    assert np.abs(logits[:, :-1] - want[:, :-1]).max() <= 3e-2
    x = logits[:, :-1]                      # (the last column is the mask token)
    assert np.array_equal(am, x.argmax(1))
    ref = x.max(1) + np.log(np.exp(x - x.max(1, keepdims=True)).sum(1))
    assert np.abs(lse - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())
    assert np.abs(conf * np.exp(ref - x.max(1)) - 1).max() <= 2e-5


def test_a_model_without_layers_sees_its_embeddings():
    """No layer: the final norm and the LM head work on the token embeddings, in the initial forward and in a block step
    after tokens were committed.  Logits against the same in fp64."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("nolayer", 0, 256, 4, 4, 64, 688, 1024)
    decode = DecodeParams(0.9, 0.5, 4, 8)
    weights = dict(gen_weights(shape, 17))
    print("model without layers", flush=True)
    b = BlockBatch(shape, decode, Limits(1, 2, 84, 64, 40), poison_workspace=True)
    try:
        b.load_weights(weights.items())
        b.keep_logits(True)
        rid = b.request_open(gen_prompt(shape, 17, 0, 20), 64, (8, 32))
        b.refresh([rid], BB_INIT)
        init = b.latest_view().logits()
        b.merge_commit([rid])
        X = b.get_tokens(rid)
        v = b.denoise_step([rid])
        gbr, pos = (a[v.lm_rows()] for a in v.rows())
        step = v.logits()
    finally:
        b.close()
    E, g, W = (weights[n].double().numpy() for n in ("tok_emb", "final_norm", "lm_head"))

    def logits(tokens):
        h = E[tokens]
        return h / np.sqrt((h * h).mean(1, keepdims=True) + shape.rms_eps) * g.reshape(-1) @ W.T

    for got, tokens in ((init, np.full(64, shape.mask_id)), (step, X[gbr, pos])):
        want = logits(tokens)
        assert got.shape == want.shape and np.abs(got - want)[:, :-1].max() <= 3e-2


def test_plan_overrides_leave_larger_panels_alone():
    """The tuning override is for panels of at most 128 rows (the buffers of partial tiles hold any of its splits only up
    to there): block steps of 240 rows have the same logits and tokens, bit for bit, whatever it is set to."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("overtest", 2, 512, 8, 2, 64, 1376, 2048)
    weights = dict(gen_weights(shape, 19))
    G, blocks = 128, (16, 96, 128)
    b = BlockBatch(shape, DecodeParams(0.9, 0.5, 4, 2), Limits(1, 3, 22 + G, G, 240), poison_workspace=True)
    try:
        b.load_weights(weights.items())
        b.keep_logits(True)
        rid = b.request_open(gen_prompt(shape, 19, 0, 22), G, blocks)
        b.refresh([rid], BB_INIT)
        ref = None
        for kind, nt, split in [(0, 0, 0), (1, 1, 0), (1, 3, 0), (2, 1, 2), (2, 3, 0), (3, 1, 4), (3, 3, 0)]:
            print("override", kind, nt, split, flush=True)
            if kind:
                b.set_gemm_plan(kind, nt, split)
            v = b.denoise_step([rid])
            assert v.m_q == 240
            got = v.logits(), v.argmax()
            ref = ref or got
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]), (kind, nt, split)
            if kind:
                b.set_gemm_plan(kind, 0, 0)
    finally:
        b.close()


@pytest.mark.parametrize("requests,blocks,G", [
    (1, (16,), 32),                 # one branch, four waves
    (1, (4, 8, 16, 32, 8), 32),     # five branches, as many waves
    (3, (80, 16, 100), 224),        # nine; windows of more than 64 positions, over two and three pages
    (2, (4, 8, 16, 32, 4, 8, 16, 32), 32),      # sixteen: the most waves
    (6, (4, 8, 16), 32),            # eighteen: some waves have two branches
    (32, (4, 4, 8, 8, 16, 16, 4, 8), 32),       # 256: the most there can be
])
def test_packed_rows_of_many_branches(requests, blocks, G):
    """The block step's row list for one to sixteen branches per wave of the packing kernel: rows in branch order, every position of
    every unfinished window, the masked ones listed for the LM head in the same order; from the windows and tokens set before.  And its list of pages
    to copy: after the step the keys and values outside the windows are those before it, bit for bit, in pages that the branches owned and in
    those they shared, and inside the windows those of a refresh of the same tokens (another GEMM plan: to 1e-3 of the largest value)."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT, BB_PERIODIC
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("packtest", 1, 128, 2, 2, 64, 128, 512, qkv_bias=False)
    Lp, N = 20, len(blocks)
    rng = np.random.default_rng(requests)
    b = BlockBatch(shape, DecodeParams(0.9, 0.5, 4, 8), Limits(requests, N, Lp + G, G, requests * sum(blocks)), poison_workspace=True)
    try:
        b.load_weights(gen_weights(shape, 3))
        b.keep_logits(True)
        ids = [b.request_open(gen_prompt(shape, 3, i, Lp), G, blocks) for i in range(requests)]
        rows, lm, live = [], [], []
        for i, rid in enumerate(ids):
            b.refresh([rid], BB_INIT)
            X = rng.integers(0, shape.vocab - 1, (N, Lp + G), dtype=np.int32)
            windows = []
            for k, blk in enumerate(blocks):
                start = Lp + blk * int(rng.integers(0, G // blk))
                done = N > 1 and rng.random() < 0.2
                w = types.SimpleNamespace(start=start, end=start + blk, done=int(done), mean_conf=0.5)
                masked = rng.random(blk) < 0.6
                masked[int(rng.integers(0, blk))] = True
                X[k, start:start + blk][masked] = shape.mask_id
                windows.append(w)
                if not done:
                    lm += [len(rows) + j for j in range(blk) if masked[j]]
                    rows += [(rid * N + k, start + j) for j in range(blk)]
                    live.append((rid, k, slice(start, start + blk)))
            b.set_state(rid, X, windows)
        before = [b.get_kv(rid, k, 0) for rid in ids for k in range(N)]
        print(f"packed rows requests={requests} branches={N}", flush=True)
        v = b.denoise_step(ids)
        gbr, pos = v.rows()
        assert list(zip(gbr.tolist(), pos.tolist())) == rows
        assert v.lm_rows().tolist() == lm
        assert np.isfinite(v.conf()).all()
        after = [b.get_kv(rid, k, 0) for rid in ids for k in range(N)]
        b.refresh(ids, BB_PERIODIC)
        windows = {(rid, k): w for rid, k, w in live}
        for i, (rid, k) in enumerate((rid, k) for rid in ids for k in range(N)):
            outside = np.ones(Lp + G, dtype=bool)
            w = windows.get((rid, k))
            if w is not None:
                outside[w] = False
                for x, r in zip(after[i], b.get_kv(rid, k, 0)):
                    assert np.abs(x[w] - r[w]).max() <= 1e-3 * np.abs(r).max()
            for x, x0 in zip(after[i], before[i]):
                assert np.isfinite(x).all() and np.array_equal(x[outside], x0[outside])
    finally:
        b.close()


def test_a_rows_norm_does_not_depend_on_the_pass_it_runs_in():
    """The first layer's keys and values of a row, from an initial forward of 1024 rows (a workgroup per row in the norm kernel) and from a
    refresh of 2048 (eight rows per workgroup): same tokens, same sums in the projection, and the squares of a row of more than 2048
    columns are added in one order by both norm kernels, so the caches are equal bit for bit."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT, BB_PERIODIC
    from paper_2605_29233_amd.binding import gemm_plan
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("normtest", 1, 2112, 4, 4, 128, 64, 512, qkv_bias=False)
    L, G, blocks = 1024, 64, (16, 32)
    few, many = (gemm_plan(rows, 3 * 512, shape.d_model) for rows in (L, 2 * L))
    assert (few["split_k"], few["chunks_per_split"]) == (many["split_k"], many["chunks_per_split"]), (few, many)
    b = BlockBatch(shape, DecodeParams(0.9, 0.5, 4, 8), Limits(1, 2, L, G, sum(blocks)), poison_workspace=True)
    try:
        b.load_weights(gen_weights(shape, 13))
        rid = b.request_open(gen_prompt(shape, 13, 0, L - G), G, blocks)
        b.refresh([rid], BB_INIT)
        first = [b.get_kv(rid, k, 0) for k in range(2)]
        print("norm of a row in passes of 1024 and 2048 rows", flush=True)
        b.refresh([rid], BB_PERIODIC)
        again = [b.get_kv(rid, k, 0) for k in range(2)]
    finally:
        b.close()
    for kv, kv2 in zip(first, again):
        for x, y in zip(kv, kv2):
            assert np.isfinite(x).all() and np.array_equal(x, y), np.abs(x - y).max()


def _class_us(b, ids, klass, steps=20):
    """Shortest of three runs: microseconds per block step in the launches of one profile class."""
    best = float("inf")
    b.profile_enable()
    for _ in range(3):
        b.synchronize()
        b.profile_read()
        for _ in range(steps):
            b.denoise_step(ids, want_view=False)
        best = min(best, b.profile_read()[klass]["total_ms"] * 1e3 / steps)
    b.profile_enable(False)
    return best


def test_empty_slots_cost_split_attention_nothing():
    """One request whose attention tiles are split over three workgroups each, in a context of its own and in one of 64 requests x 4
    branches: same plan, same logits bit for bit, and no time for the partial results of the 255 empty segments (3 x 255 x 32 tiles of 16.6 KB,
    406 MB: at the 8 TB/s of the memory 51 us, where the launches themselves take about 20)."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("slottest", 1, 256, 32, 32, 128, 256, 1024, qkv_bias=False)
    weights = dict(gen_weights(shape, 5, device="cuda:0"))
    prompt = gen_prompt(shape, 5, 0, 704)
    out, us = [], []
    for requests, branches in ((1, 1), (64, 4)):
        b = BlockBatch(shape, DecodeParams(0.9, 0.5, 4, 8), Limits(requests, branches, 768, 64, 32), poison_workspace=True)
        try:
            assert b.attention_plan([32], 768) == (3, 4)
            b.load_weights(weights.items())
            b.keep_logits(True)
            rid = b.request_open(prompt, 64, (32,))
            b.refresh([rid], BB_INIT)
            print(f"empty slots: {requests} x {branches}", flush=True)
            out.append(b.denoise_step([rid]).logits().copy())
            us.append(_class_us(b, [rid], "attention"))
        finally:
            b.close()
    print("attention us per step:", us, flush=True)
    assert np.isfinite(out[0][:, :-1]).all() and np.array_equal(out[0], out[1])
    assert us[1] < 2 * us[0], us


def test_finished_branches_cost_the_kernels_between_the_gemms_little():
    """A step sized for 128 rows of which four are live, against all 128: the kernels that add up the k splits of a projection (sixteen here,
    the partial results of a layer 470 MB) leave the rows past the live count alone, so the first takes a fraction of the second's time."""
    from paper_2605_29233_amd import BlockBatch, Limits, BB_INIT
    from workload.gen import gen_weights, gen_prompt
    shape = ModelShape("deadtest", 2, 8192, 64, 64, 128, 8192, 512, qkv_bias=False)
    L_p, G, blocks = 40, 128, (4, 124)
    b = BlockBatch(shape, DecodeParams(0.9, 0.5, 200, 8), Limits(1, 2, L_p + G, G, 128), poison_workspace=True)
    try:
        b.load_weights(gen_weights(shape, 5, device="cuda:0"))
        for kind in (1, 2, 3):
            b.set_gemm_plan(kind, 1, 16)
        rid = b.request_open(gen_prompt(shape, 5, 0, L_p), G, blocks)
        b.refresh([rid], BB_INIT)
        X = b.get_tokens(rid)
        us = []
        for done in (0, 1):
            windows = [types.SimpleNamespace(start=L_p, end=L_p + blk, done=done and k, mean_conf=0.5) for k, blk in enumerate(blocks)]
            b.set_state(rid, X, windows)
            print("finished branches:", done, flush=True)
            assert b.denoise_step([rid]).m_q == (4 if done else 128)
            us.append(_class_us(b, [rid], "glue"))
    finally:
        b.close()
    print("glue us per step:", us, flush=True)
    assert us[1] < 0.7 * us[0], us          # (0.47 to 0.49; 0.89 with every row read)
