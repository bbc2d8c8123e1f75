// Wide-format MFMA GEMM for passes of more than 128 activation rows (wide block steps, refreshes, initial forwards, many requests):
//     C[m][n] = sum_k A[m][k] * W[n][k]          (operands and precision as in gemm_wide.hip)
//
// What bounds it: first the matrix pipes, but not they alone: they are busy 0.63 of the time at 2.05 GHz (0.70 of the cycles in which
// the waves are resident).  Nothing but its MFMAs take 0.79 us per 64 k of a 128 x 256 tile at the clock that the chip's power allows
// with all CUs at it, LDS reads add 0.04, the conversions to e4m3 0.1, the loads from the L2s 0.1, weights that come from HBM another 0.1.
// A chunk of 192 x 256 takes 1.6 us with all CUs at work (1.2 of MFMAs alone) and 1.2 with half of them, and about 9 us per tile of prologue,
// drain and epilogue leave the pipes idle (1536 tiles of 24576 x 3072 rows over k = 512 to 8192).  Hence 16 x 16 MFMAs (16x16x32 fp16, 16x16x128
// fp8), whose accumulators pass half as often per product as those of 32 x 32 (2.07 PFLOP/s of the mix against 1.84), and operands that
// move as little as they can: four waves, one per SIMD, each with 32 NT columns of weights in registers and the activation panel in LDS for all of them.  (Eight
// waves in a grid of 2 x 4, both operands through LDS, read 1.3 to 1.6 times as much LDS per product and convert each weight twice.)
// A wave owns 2 NT x 2 MT accumulator tiles: 128 x 256 and 192 x 256 per workgroup, 96 or 128 rows x 128 or 384 columns where that
// fills the chip better.
//
// Pipeline, in units of 128 k (two chunks, four halves).  Weights: global -> registers, a half four ahead.  Activations: direct-to-LDS
// loads, the fp16 terms into a ring of four chunks, the remainders of a unit into one buffer.  One wave per SIMD has nothing to hide a stall,
// so each half is cut into slots of 2 NT MFMAs with an even share of the LDS reads, conversions and loads.
//     half 0 | barrier | half 1 (requests this unit's remainders) | half 2 | barrier | half 3 | barrier | fp8 MFMAs of the unit
// Measured, us per launch, before = the eight-wave kernel (more than 256 rows) and four waves with 32 x 32 MFMAs (up to 256), in turn on one
// box: 240 rows, 12288 x 4096 44.0 -> 42.5, 4096 x 12288 42.7 -> 39.7, 3584 x 18944 60.2 -> 51.6, gate/up with SwiGLU (24576 x 4096) 84.2 ->
// 79.7; 768 rows, 12288 x 4096 101.6 -> 98.3, gate/up 209.7 -> 203.5, 4096 x 12288 90.9 -> 90.4; 1536 rows, 4096 x 12288 167.2 -> 164.4; 3072 rows,
// gate/up 686 -> 671 (the 192-row tile holds 450 of 512 registers: with an applied norm scale in its epilogue it took 511 and 695 us).
#include "bb_internal.h"
#include "lds.h"
#include "sched.h"
#include <hip/hip_ext.h>
#include <algorithm>
#include <type_traits>

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ f16x8 as_f16x8(const u32x4& v) { return __builtin_bit_cast(f16x8, v); }

#define PEPI_PARTIAL 0
#define PEPI_SWIGLU 1

template <int MT, int NT, int EPI>
__global__ __launch_bounds__(256, 1) void gemm_panel_kernel(const u32x4* __restrict__ Wt, const float* __restrict__ wscale,
                                                            const u32x4* __restrict__ Apk, float* __restrict__ P,
                                                            size_t split_stride, int ldp, int mt_total, int n_tiles,
                                                            int total_chunks, int chunks_per_split, int n_split, int tiles_x,
                                                            const int* __restrict__ rows_live, u32x4* __restrict__ Opk) {
    constexpr int T = 2 * NT, R = 2 * MT;                   // 16 x 16 accumulator tiles per wave: T of columns, R of rows
    constexpr int STAGE = MT * 4096, LO = 4 * STAGE, LO_CHUNK = MT * 2048;      // LDS: fp16 fragments of four chunks, remainders of a unit
    constexpr int LDT = 16 * T + 4;                         // store slices: row stride in floats
    constexpr int STAGED = LO + 2 * LO_CHUNK, SLICES = 4 * 32 * LDT * 4;
    __shared__ __attribute__((aligned(16))) char lds[STAGED > SLICES ? STAGED : SLICES];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    // Items = (k split, tile); a round of at most 256 of them is dealt to the XCDs (workgroups go to them round robin) in
    // contiguous runs, and tiles are numbered in bands of four row groups, row group fastest: the 32 workgroups of an
    // XCD then work on about 4 row groups x 8 column groups, whose chunks its L2 fetches once.
    const int live_mt = rows_live ? min(mt_total, (*rows_live + 31) >> 5) : mt_total;
    const int tiles_y = (live_mt + MT - 1) / MT, tiles = tiles_x * tiles_y, items = tiles * n_split;
    constexpr int BAND = 4;
    for (int base = 0; base < items; base += gridDim.x) {
    const int n_round = min((int)gridDim.x, items - base), lin = blockIdx.x;
    if (lin >= n_round) break;
    const int e = lin & 7, item = base + e * (n_round >> 3) + min(e, n_round & 7) + (lin >> 3);
    const int split_id = item / tiles, tile = item % tiles;
    const int band = tile / (BAND * tiles_x), in_band = tile % (BAND * tiles_x), band_h = min(BAND, tiles_y - band * BAND);
    const int bx = in_band / band_h, by = band * BAND + in_band % band_h;
    const int mt0 = by * MT, mt_cnt = min(MT, live_mt - mt0);
    const int c0 = split_id * chunks_per_split, c1 = min(c0 + chunks_per_split, total_chunks), n_chunks = c1 - c0;

    const unsigned lane16 = lane * 16, lds0 = lds_offset(lds), frag_lane = (g >> 1) * 1024 + (c16 + 32 * (g & 1)) * 16;
    const size_t a_chunk = (size_t)mt_total * (BB_WFRAGS * 1024);
    const char* panel = (const char*)Apk + (size_t)mt0 * (BB_WFRAGS * 1024) + c0 * a_chunk;
    unsigned a_mt[MT];                                      // (missing m-tiles read a valid one)
#pragma unroll
    for (int i = 0; i < MT; ++i) a_mt[i] = min(i, mt_cnt - 1) * (BB_WFRAGS * 1024);
    // Wave w fetches fragment w of every m-tile of a chunk's fp16 terms, and of a unit's remainders fragment 4 + w % 2 of
    // chunk w / 2.  Past the end all lanes read one address of the last chunk's fp16 terms.
    const char *hi_src = panel + wave * 1024, *lo_src = panel + (4 + (wave & 1)) * 1024 + (wave >> 1) * a_chunk;
    unsigned hi_lane = lane16, hi_dst = lds0 + wave * 1024;
    const unsigned lo_dst = lds0 + LO + (wave >> 1) * LO_CHUNK + (wave & 1) * 1024;
    int hi_c = 0;
    auto hi_next = [&]() {
        ++hi_c;
        const bool in = hi_c < n_chunks;
        hi_src += in ? a_chunk : 0;
        hi_lane = in ? lane16 : 0u;
        hi_dst = (hi_c & 3) == 0 ? hi_dst - 3 * STAGE : hi_dst + STAGE;
    };
    auto fetch_hi = [&](auto I) { load_to_lds<0>(hi_src + a_mt[decltype(I)::value], hi_lane, hi_dst + decltype(I)::value * 4096); };
    auto fetch_lo = [&](auto I) { load_to_lds<0>(lo_src + a_mt[decltype(I)::value], lane16, lo_dst + decltype(I)::value * 2048); };
    // (The pointers pass through assembly so that the compiler takes the weight loads for reads of memory that the direct-to-LDS
    // loads may write: their order, which the waits count on, is then the order written here.)
    typedef const __attribute__((address_space(1))) char* gchar;
    typedef const __attribute__((address_space(1))) u32x4* gvec;
    gchar wsrc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        wsrc[t] = (gchar)Wt + ((size_t)min((bx * 4 + wave) * NT + t, n_tiles - 1) * total_chunks + c0) * 4096;      // clamped loads; stores are guarded
        asm volatile("" : "+s"(wsrc[t]));
    }
    unsigned w_lane = frag_lane;
    int w_c = 0;
    auto w_next = [&]() {
        ++w_c;
        const bool in = w_c < n_chunks;
#pragma unroll
        for (int t = 0; t < NT; ++t) { wsrc[t] += in ? 4096 : 0; asm volatile("" : "+s"(wsrc[t])); }
        w_lane = in ? frag_lane : 0u;
    };
    constexpr int D = R > 8 ? R / 2 : R;                    // activation fragments read ahead
    u32x4 w[4][T], b[D];                                    // weights of a unit's four halves
    i32x8 w8[T];
    auto fetch_w = [&](auto S, int t) {
        constexpr int s = decltype(S)::value;
        const gvec p = (gvec)(wsrc[t >> 1] + (size_t)w_lane + (s & 1) * 2048 + (t & 1) * 256);
        w[s][t] = *p;
    };
    auto fetch_w_half = [&](auto S) { unroll<T>([&](auto t) { fetch_w(S, t); }); };
    f32x4 acc[T][R];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int m = 0; m < R; ++m) {
            acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
            asm("" : "+v"(acc[t][m]));                      // (as constants the compiler carries them through the loop element by element, and copies)
        }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) w8[t][j] = 0;

    constexpr int H1 = (MT + 1) / 2;                        // of a chunk's MT pieces, those issued in the half before
    unroll<MT>([&](auto I) { fetch_hi(I); });
    hi_next();
    fetch_w_half(IC(0)); fetch_w_half(IC(1));
    unroll<MT>([&](auto I) { fetch_hi(I); });
    hi_next();
    w_next();
    fetch_w_half(IC(2)); fetch_w_half(IC(3));
    unroll<H1>([&](auto I) { fetch_hi(I); });
    // all but the latest `Later` loads of this wave have landed; after the barrier so have the others'
    auto landed = [&](auto Later) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(Later)::value) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    landed(IC(4 * T + MT + H1));

    const char *cur = lds + frag_lane, *lo_at = lds + LO + frag_lane;
    unsigned odd_unit = 0;
    auto read_b = [&](int m, const char* at, int h) { b[m % D] = *reinterpret_cast<const u32x4*>(at + (m >> 1) * 4096 + h * 2048 + (m & 1) * 256); };
#pragma unroll
    for (int m = 0; m < D; ++m) read_b(m, cur, 0);
    // conversion i of 4 T of a half: two fp16 weights of tile i / 4 -> half a dword of its e4m3 operand
    auto convert = [&](auto S, auto I) {
        constexpr int s = decltype(S)::value, i = decltype(I)::value, t = i / 4, q = i % 4, j = 2 * s + q / 2;
        const unsigned d = w[s][t][q];
        const int old = w8[t][j];
        w8[t][j] = __builtin_bit_cast(int, __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(__builtin_bit_cast(i16x2, old), __builtin_bit_cast(f16x2, d), (float)(1 << BB_LO_SHIFT), (q & 1) != 0));
    };
    // Half S of a unit: a slot per row tile.  In a slot: T MFMAs, this row tile's fragment of the next half (at nxt, half 1 - S % 2 of its
    // chunk), a share of the conversions and of the N pieces that fetch() issues.  Then the weights of the half four ahead.
    auto half = [&](auto S, const char* here, const char* nxt, auto N, auto&& fetch, auto Last) {
        constexpr int s = decltype(S)::value, n = decltype(N)::value;
        unroll<R>([&](auto M) {
            constexpr int m = decltype(M)::value;
#pragma unroll
            for (int t = 0; t < T; ++t)
                acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(w[s][t]), as_f16x8(b[m % D]), acc[t][m], 0, 0, 0);
            if constexpr (m + D < R) read_b(m + D, here, s & 1);
            else read_b(m + D - R, nxt, 1 - (s & 1));
            unroll<4 * T * (m + 1) / R - 4 * T * m / R>([&](auto I) { convert(S, IC(4 * T * m / R + decltype(I)::value)); });
            unroll<n * (m + 1) / R - n * m / R>([&](auto I) { fetch(IC(n * m / R + decltype(I)::value)); });
            if constexpr (m == R - 1 && !decltype(Last)::value) fetch_w_half(S);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    u32x4 lo[2][2];
    auto remainders = [&](auto Whole) {
        constexpr bool whole = decltype(Whole)::value;
        auto read_lo = [&](int m) {
            lo[m & 1][0] = *reinterpret_cast<const u32x4*>(lo_at + (m >> 1) * 2048 + (m & 1) * 256);
            if constexpr (whole) lo[m & 1][1] = *reinterpret_cast<const u32x4*>(lo_at + LO_CHUNK + (m >> 1) * 2048 + (m & 1) * 256);
        };
        read_lo(0);
        unroll<R>([&](auto M) {
            constexpr int m = decltype(M)::value;
            if constexpr (m + 1 < R) read_lo(m + 1);
            i32x8 b8;
#pragma unroll
            for (int j = 0; j < 4; ++j) { b8[j] = (int)lo[m & 1][0][j]; b8[4 + j] = whole ? (int)lo[m & 1][1][j] : 0; }
            // A operand e4m3 (format 0), B operand e5m2 (format 1), both block scales 2^0
#pragma unroll
            for (int t = 0; t < T; ++t)
                acc[t][m] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w8[t], b8, acc[t][m], 0, 1, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // (what a wait leaves on its way is counted from the order in which the pieces and weights of the last unit were issued)
    // The waits: of the loads of the last unit, those issued after the pieces waited for may still be on their way.  A place in LDS
    // is requested anew only behind a barrier that all waves reach after their last read of it.
    std::false_type on;
    std::true_type last;
    int c = 0;
    for (; c + 2 <= n_chunks; c += 2) {
        w_next();
        half(IC(0), cur, cur, IC(MT - H1), [&](auto I) { fetch_hi(IC(H1 + decltype(I)::value)); }, on);
        landed(IC(3 * T + MT));
        half(IC(1), cur, cur + STAGE, IC(MT), fetch_lo, on);
        hi_next();
        lo_src += 2 * a_chunk;
        w_next();
        half(IC(2), cur + STAGE, cur + STAGE, IC(MT), fetch_hi, on);
        landed(IC(3 * T + 2 * MT));
        hi_next();
        odd_unit ^= 1u;
        const char* second = cur + STAGE;
        cur = lds + frag_lane + odd_unit * (2 * STAGE);
        half(IC(3), second, cur, IC(H1), fetch_hi, on);
        landed(IC(3 * T + MT + H1));
        remainders(std::true_type{});
    }
    // every load that the waits count was made: none of them may go because nothing reads it
#pragma unroll
    for (int i = 0; i < 4 * T; ++i) asm volatile("" ::"v"(w[i / T][i % T]));
    if (c < n_chunks) {                                     // an odd chunk is left: half a unit, nothing more to fetch but its remainders
        half(IC(0), cur, cur, IC(0), fetch_lo, last);
        landed(IC(0));                                      // (here only the barrier counts: all waves are done with the last unit's remainders)
        half(IC(1), cur, cur, IC(MT), [&](auto I) { load_to_lds_below(wave >> 1, 1, lo_src + a_mt[decltype(I)::value], lane16, lo_dst + decltype(I)::value * 2048); }, last);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int j = 4; j < 8; ++j) w8[t][j] = 0;
        landed(IC(0));
        remainders(std::false_type{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // undo the per-row weight scale: register r of lane (c16, g) holds weight row 4 g + r of tile t, activation row c16
    const int x0 = (bx * 4 + wave) * NT;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const float4 s4 = *reinterpret_cast<const float4*>(&wscale[min(x0 + (t >> 1), n_tiles - 1) * 32 + 16 * (t & 1) + 4 * g]);
#pragma unroll
        for (int m = 0; m < R; ++m) { acc[t][m][0] *= s4.x; acc[t][m][1] *= s4.y; acc[t][m][2] *= s4.z; acc[t][m][3] *= s4.w; }
    }
    __syncthreads();                                        // all waves are done with the staged operands
    if constexpr (EPI == PEPI_SWIGLU) {
        static_assert(EPI != PEPI_SWIGLU || NT == 2, "gate and up tiles of a feature group sit in one wave");
        // 32 gate rows (tiles 0, 1) alternate with the 32 up rows (2, 3) of the same features.  The panel wants 8
        // consecutive features in one lane: lanes g and g ^ 1 swap the four they do not own.
        if (x0 < n_tiles) {
#pragma unroll
            for (int m = 0; m < R; ++m) {
                if (m / 2 >= mt_cnt) break;
                const int row = (mt0 + m / 2) * 32 + (m & 1) * 16 + c16;
                float act[2][4], y[8];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float gt = acc[tt][m][r], up = acc[T - 2 + tt][m][r];
                        act[tt][r] = gt / (1.0f + expf(-gt)) * up;
                    }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(act[0][r]), __float_as_uint(act[1][r]), false, false);
                    y[r] = __uint_as_float(sw[0]);
                    y[4 + r] = __uint_as_float(sw[1]);
                }
                store_panel8(Opk, row, (x0 / 2) * 4 + 2 * (g & 1) + (g >> 1), mt_total, y, 1);
            }
        }
        continue;
    }
    // Partial tiles go out through LDS (each wave its own slice, one m-tile at a time) as whole 128-byte lines.
    float* tl = reinterpret_cast<float*>(lds) + wave * (32 * LDT);
    float* Ps = P + (size_t)split_id * split_stride;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (mt >= mt_cnt) break;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                *reinterpret_cast<float4*>(&tl[(s * 16 + c16) * LDT + t * 16 + 4 * g]) =
                    make_float4(acc[t][2 * mt + s][0], acc[t][2 * mt + s][1], acc[t][2 * mt + s][2], acc[t][2 * mt + s][3]);
        wave_lds_order();                                   // (the same wave wrote and reads: no barrier needed)
        constexpr int LPR = 4 * T;                          // lanes per row
#pragma unroll
        for (int it = 0; it < 32 * LPR / 64; ++it) {
            const int idx = it * 64 + lane, r = idx / LPR, c4 = idx % LPR * 4;
            const float4 v = *reinterpret_cast<const float4*>(&tl[r * LDT + c4]);
            if (x0 * 32 + c4 < n_tiles * 32) *reinterpret_cast<float4*>(&Ps[(size_t)((mt0 + mt) * 32 + r) * ldp + x0 * 32 + c4]) = v;
        }
        wave_lds_order();                                   // (the next m-tile overwrites the slice)
    }
    __syncthreads();                                        // the next tile's loads overwrite the LDS slices
    }
}

void launch_gemm_panel(const u32x4* Wt, const float* wscale, const u32x4* Apk, float* P, int mt_total, int N, int K, GemmPlan plan,
                       hipStream_t s, const int* rows_live, u32x4* swiglu_out, LaunchStamps st) {
    const int n_tiles = N / 32, total_chunks = (K + 63) / 64, tiles_x = (n_tiles + 4 * plan.nt - 1) / (4 * plan.nt), tiles_y = (mt_total + plan.mt - 1) / plan.mt;
    const size_t split_stride = (size_t)mt_total * 32 * N;
    dim3 grid(std::min(tiles_x * tiles_y * plan.split_k, 256));
#define PARGS Wt, wscale, Apk, P, split_stride, N, mt_total, n_tiles, total_chunks, plan.chunks_per_split, plan.split_k, tiles_x, rows_live, swiglu_out
#define PLAUNCH(MT_, NT_, EPI_) hipExtLaunchKernelGGL(HIP_KERNEL_NAME(gemm_panel_kernel<MT_, NT_, EPI_>), grid, dim3(256), 0, s, st.start, st.stop, 0, PARGS)
#define PLAUNCH_MT(NT_, EPI_) do { if (plan.mt == 3) PLAUNCH(3, NT_, EPI_); else PLAUNCH(4, NT_, EPI_); } while (0)
    if (plan.mt == 6) { if (swiglu_out) PLAUNCH(6, 2, PEPI_SWIGLU); else PLAUNCH(6, 2, PEPI_PARTIAL); }
    else if (swiglu_out) PLAUNCH_MT(2, PEPI_SWIGLU);
    else if (plan.nt == 3) PLAUNCH(4, 3, PEPI_PARTIAL);
    else if (plan.nt == 2) PLAUNCH_MT(2, PEPI_PARTIAL);
    else PLAUNCH_MT(1, PEPI_PARTIAL);
#undef PLAUNCH_MT
#undef PLAUNCH
#undef PARGS
}
