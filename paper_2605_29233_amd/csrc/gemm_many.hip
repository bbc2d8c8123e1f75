// Wide-format MFMA GEMM for passes of more than 256 activation rows (full-sequence refresh, initial forward, many requests):
//     C[m][n] = sum_k A[m][k] * W[n][k]          (operands and precision as in gemm_wide.hip)
//
// What bounds it: power.  With random operands the chip sustains 1.7 PFLOP/s of nothing but 32x32x16 fp16 MFMAs but 1.95
// of 16x16x32 ones, whose fp32 accumulators pass half as often per product; for the mix of four fp16 and one fp8 step
// 1.84 and 2.07 (in bf16 equivalents).  So this kernel computes in 16 x 16 tiles (16x16x32 fp16,
// 16x16x128 fp8), keeps an operand for consecutive MFMAs, and moves as little as it can: a kernel with 32 x 32 tiles
// that kept the pipes busier than the one before it ran no faster, its clock fell instead.
// Eight waves per workgroup, two per SIMD: one wave per SIMD left the matrix pipe idle at every wait.  Workgroup tile =
// 64 MTW rows x 256 columns, waves in a grid of 2 (rows) x 4 (columns), a wave owns 2 MTW x 4 accumulator tiles; both
// operands reach LDS by direct-to-LDS loads, which pass through no register.
// Measured (3072 rows; before = four waves, 32 x 32 tiles, weights in registers): gate/up with SwiGLU (24576 x 4096)
// 775 -> 700 us, down (4096 x 12288) 370 -> 332 us, 1.33 PFLOP/s in bf16 equivalents; 20480 rows of gate/up 5.13 -> 4.61 ms;
// 4206 rows, 3584 x 18944: 861 -> 665 us.  The matrix pipes are busy 0.65 of the elapsed cycles at 1.9 GHz (0.60 before;
// counters, every launch alone), 0.73 of those in which its waves are resident (0.66).
// Small matrices, whose tiles leave most CUs without work, go to gemm_wide_kernel (gemm_plan_wide has the rule).
#include "bb_internal.h"
#include "lds.h"
#include <hip/hip_ext.h>
#include <algorithm>
#include <type_traits>

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ f16x8 as_f16x8(const u32x4& v) { return __builtin_bit_cast(f16x8, v); }

template <int N, int I = 0, class F> static __device__ __forceinline__ void unroll(F&& f) {
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); unroll<N, I + 1>(f); }
}
#define IC(v) std::integral_constant<int, (v)>{}

#define MEPI_PARTIAL 0
#define MEPI_SWIGLU 1

template <int MTW, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_many_kernel(const u32x4* __restrict__ Wt, const float* __restrict__ wscale,
                                                           const u32x4* __restrict__ Apk, float* __restrict__ P,
                                                           size_t split_stride, int ldp, int mt_total, int n_tiles,
                                                           int total_chunks, int chunks_per_split, int n_split, int tiles_x,
                                                           const int* __restrict__ rows_live, u32x4* __restrict__ Opk) {
    constexpr int MT = 2 * MTW;                     // m-tiles of 32 rows per workgroup
    constexpr int NM = 2 * MTW;                     // accumulator tiles of 16 rows per wave (times four of 16 columns)
    // LDS: a ring of four halves (32 k) of fp16 operands, and the remainders of two units (128 k)
    constexpr int W_BYTES = 8 * 2048, STAGE = W_BYTES + MT * 2048, LO_HALF = MT * 1024, LO_UNIT = 4 * LO_HALF;
    __shared__ __attribute__((aligned(16))) char lds[4 * STAGE + 2 * LO_UNIT];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wr = wave >> 2, wc = wave & 3, g = lane >> 4, c16 = lane & 15;

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
    const int c0 = split_id * chunks_per_split, c1 = min(c0 + chunks_per_split, total_chunks);

    // A half (32 k) is 2 weight fragments per 32-row tile and, per m-tile, 2 fp16 fragments and one of e5m2 remainders.
    // Wave w fetches the weights of tile w (pieces 0, 1) and every eighth activation fragment (pieces 2, ...): for each of
    // those the offset in the chunk's panel, the LDS offset and the strides of the latter are kept in scalar registers.
    constexpr int A_FRAGS = 3 * MT, A_EACH = A_FRAGS / 8, A_REST = A_FRAGS % 8, A_PIECES = A_EACH + (A_REST != 0), PIECES = 2 + A_PIECES;
    const unsigned lane16 = lane * 16, lds0 = lds_offset(lds);
    unsigned a_off[2][A_PIECES], a_dst[A_PIECES], a_stage[A_PIECES], a_unit[A_PIECES];
#pragma unroll
    for (int i = 0; i < A_PIECES; ++i) {
        const int f = i * 8 + wave, mt = min(f / 3, mt_cnt - 1), j = f % 3;                     // missing m-tiles read a valid one
        a_off[0][i] = mt * (BB_WFRAGS * 1024) + (j < 2 ? j * 1024 : 4 * 1024);
        a_off[1][i] = a_off[0][i] + (j < 2 ? 2048 : 1024);
        a_dst[i] = lds0 + (j < 2 ? W_BYTES + (f / 3) * 2048 + j * 1024 : 4 * STAGE + LO_UNIT + (f / 3) * 1024);
        a_stage[i] = j < 2 ? STAGE : LO_HALF;
        a_unit[i] = j < 2 ? 0u : 0u - LO_UNIT;      // (the first point_at moves to buffer 0)
    }
    const size_t a_chunk = (size_t)mt_total * (BB_WFRAGS * 1024);
    const int n_chunks = c1 - c0, n_units = (n_chunks + 1) >> 1;
    const char *wsrc[2], *asrc[2];                   // the two chunks of the unit whose loads are being issued
    wsrc[0] = (const char*)Wt + ((size_t)min(bx * 8 + wave, n_tiles - 1) * total_chunks + c0) * 4096;             // clamped loads; stores are guarded
    asrc[0] = (const char*)Apk + (size_t)mt0 * (BB_WFRAGS * 1024) + c0 * a_chunk;
    auto point_at = [&](int unit) {                  // (past the end: the last unit again, which nothing reads; an odd last chunk twice)
        const bool next = unit > 0 && unit < n_units, pair = min(unit, n_units - 1) * 2 + 1 < n_chunks;
        wsrc[0] += next ? 2 * 4096 : 0;
        asrc[0] += next ? 2 * a_chunk : 0;
        wsrc[1] = wsrc[0] + (pair ? 4096 : 0);
        asrc[1] = asrc[0] + (pair ? a_chunk : 0);
#pragma unroll
        for (int i = 0; i < A_PIECES; ++i) { a_dst[i] += a_unit[i]; a_unit[i] = 0u - a_unit[i]; }     // remainders: the other unit's buffer
    };
    // piece i of the loads for half S of that unit by this wave
    auto fetch_piece = [&](auto I, auto S) {
        constexpr int i = decltype(I)::value, h = decltype(S)::value;
        if constexpr (i < 2) load_to_lds<i * 1024>(wsrc[h >> 1] + (h & 1) * 2048, lane16, lds0 + h * STAGE + wave * 2048);
        else {
            const char* src = asrc[h >> 1] + a_off[h & 1][i - 2];
            const unsigned to = a_dst[i - 2] + h * a_stage[i - 2];
            if constexpr (i < 2 + A_EACH) load_to_lds<0>(src, lane16, to);
            else load_to_lds_first<A_REST>(wave, src, lane16, to);
        }
    };

    // A pair of 32 x 16 fragments in LDS read as 16 x 32 MFMA operands: lane (c16, g) takes row c16 (+ 16) and the 8 k of
    // k-step g / 2, lane half g % 2; its 32 e5m2 remainders of 128 k are those of the same k in the same order.
    const int frag_lane = (g >> 1) * 1024 + (c16 + 32 * (g & 1)) * 16;
    const char* wl = lds + frag_lane + wc * 4096;
    const char* al = lds + W_BYTES + frag_lane + wr * MTW * 2048;
    const char* ll = lds + 4 * STAGE + (g >> 1) * LO_HALF + (c16 + 32 * (g & 1)) * 16 + wr * MTW * 1024;
    f32x4 acc[4][NM];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int m = 0; m < NM; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 w[4], b[NM];
    i32x8 w8[4];
    auto read_w = [&](int t, int stage) { w[t] = *reinterpret_cast<const u32x4*>(wl + stage * STAGE + (t >> 1) * 2048 + (t & 1) * 256); };
    auto read_b = [&](int m, int stage) { b[m] = *reinterpret_cast<const u32x4*>(al + stage * STAGE + (m >> 1) * 2048 + (m & 1) * 256); };
    // k-half p (4 values) of the fp16 weights of tile t -> e4m3
    auto convert = [&](int t, int H, int p) { w8[t][2 * H + p] = fp16x4_to_e4m3x4(w[t][2 * p], w[t][2 * p + 1], w8[t][2 * H + p]); };
    auto mfma2 = [&](int t, int m) {
        acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(w[t]), as_f16x8(b[m]), acc[t][m], 0, 0, 0);
        acc[t + 1][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(w[t + 1]), as_f16x8(b[m]), acc[t + 1][m], 0, 0, 0);
    };
    u32x4 lo[2][2];
    auto read_lo = [&](int unit, int m) {
        const char* lu = ll + (unit & 1) * LO_UNIT;
#pragma unroll
        for (int q = 0; q < 2; ++q) lo[m & 1][q] = *reinterpret_cast<const u32x4*>(lu + q * (2 * LO_HALF) + (m >> 1) * 1024 + (m & 1) * 256);
    };
    // One half (32 k; H = its place in the unit of 128 k = its ring stage).  First the weight tiles 0, 1 against all rows,
    // while tiles 2, 3 are read: then this stage has been read whole.  After the barrier tiles 2, 3,
    // while the first operands of the next half replace what is done with, and the freed stage takes the loads of the
    // half after next but two.  A load keeps the address path busy for 16 cycles, so they are spread over the MFMAs:
    // eight waves that issued theirs in one go stood in line for half of the chunk's time.
    auto half = [&](auto HC, int unit) {
        constexpr int H = decltype(HC)::value, N = (H + 1) & 3;
        read_w(2, H); read_w(3, H);
        unroll<NM>([&](auto M) {
            constexpr int m = decltype(M)::value;
            mfma2(0, m);
            if constexpr (m < 4) convert(m >> 1, H, m & 1);
            __builtin_amdgcn_sched_barrier(0);
        });
        // of this wave's loads those of the halves after next may still be on their way
        if constexpr (MTW == 3) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (H == 0) point_at(unit + 1);
        read_w(0, N); read_w(1, N);
        unroll<NM>([&](auto M) {
            constexpr int m = decltype(M)::value;
            mfma2(2, m);
            read_b(m, N);
            if constexpr (m < 4) convert(2 + (m >> 1), H, m & 1);
            if constexpr (m < PIECES) fetch_piece(M, HC);
            if constexpr (H == 3 && m == NM - 1) read_lo(unit, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
        unroll<(PIECES > NM ? PIECES - NM : 0)>([&](auto R) { fetch_piece(IC(NM + decltype(R)::value), HC); });
    };
    // A operand e4m3 (format 0), B operand e5m2 (format 1), both block scales 2^0
    auto remainders = [&](int unit, bool whole) {
        unroll<NM>([&](auto M) {
            constexpr int m = decltype(M)::value;
            if constexpr (m + 1 < NM) read_lo(unit, m + 1);
            i32x8 b8;
#pragma unroll
            for (int j = 0; j < 4; ++j) { b8[j] = (int)lo[m & 1][0][j]; b8[4 + j] = whole ? (int)lo[m & 1][1][j] : 0; }
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t][m] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w8[t], b8, acc[t][m], 0, 1, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    point_at(0);
    unroll<4>([&](auto S) { unroll<PIECES>([&](auto I) { fetch_piece(I, S); }); });
    if constexpr (MTW == 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_w(0, 0); read_w(1, 0);
#pragma unroll
    for (int m = 0; m < NM; ++m) read_b(m, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) w8[t][j] = 0;
    int unit = 0;
    for (; unit * 2 + 2 <= n_chunks; ++unit) {
        half(IC(0), unit);
        half(IC(1), unit);
        half(IC(2), unit);
        half(IC(3), unit);
        remainders(unit, true);
    }
    if (unit < n_units) {                        // an odd chunk is left: half a unit
        half(IC(0), unit);
        half(IC(1), unit);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 4; j < 8; ++j) w8[t][j] = 0;
        read_lo(unit, 0);
        remainders(unit, false);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // undo the per-row weight scale: register r of lane (c16, g) holds weight row 4 g + r of tile t, activation row c16
    const int x0 = bx * 8 + wc * 2, mtw0 = mt0 + wr * MTW, mtw_cnt = min(MTW, live_mt - mtw0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float4 s4 = *reinterpret_cast<const float4*>(&wscale[min(x0 + (t >> 1), n_tiles - 1) * 32 + 16 * (t & 1) + 4 * g]);
#pragma unroll
        for (int m = 0; m < NM; ++m) { acc[t][m][0] *= s4.x; acc[t][m][1] *= s4.y; acc[t][m][2] *= s4.z; acc[t][m][3] *= s4.w; }
    }
    __syncthreads();                                        // all waves are done with the staged operands
    if constexpr (EPI == MEPI_SWIGLU) {
        // 32 gate rows (tiles 0, 1) alternate with the 32 up rows (2, 3) of the same features.  The panel wants 8
        // consecutive features in one lane: lanes g and g ^ 1 swap the four they do not own.
        if (x0 < n_tiles) {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                if (m / 2 >= mtw_cnt) break;
                float act[2][4], y[8];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float gt = acc[tt][m][r], up = acc[2 + tt][m][r];
                        act[tt][r] = gt / (1.0f + expf(-gt)) * up;
                    }
                const bool odd = g & 1;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float mine = odd ? act[1][r] : act[0][r], recv = __shfl_xor(odd ? act[0][r] : act[1][r], 16, 64);
                    y[r] = odd ? recv : mine;
                    y[4 + r] = odd ? mine : recv;
                }
                store_panel8(Opk, (mtw0 + m / 2) * 32 + (m & 1) * 16 + c16, (x0 / 2) * 4 + 2 * (g & 1) + (g >> 1), mt_total, y, 1);
            }
        }
        continue;
    }
    // Partial tiles go out through LDS (each wave its own slice, one m-tile at a time) as whole 128-byte lines.
    constexpr int LDT = 64 + 4;                             // row stride in floats (16-byte aligned, conflict-free)
    static_assert(8 * 32 * LDT * 4 <= (int)sizeof(lds), "store slices exceed the staging buffers");
    float* tl = reinterpret_cast<float*>(lds) + wave * (32 * LDT);
    float* Ps = P + (size_t)split_id * split_stride;
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
        if (mt >= mtw_cnt) break;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                *reinterpret_cast<float4*>(&tl[(s * 16 + c16) * LDT + t * 16 + 4 * g]) =
                    make_float4(acc[t][2 * mt + s][0], acc[t][2 * mt + s][1], acc[t][2 * mt + s][2], acc[t][2 * mt + s][3]);
        wave_lds_order();                                   // (the same wave wrote and reads: no barrier needed)
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int r = it * 4 + g, c4 = c16 * 4;
            const float4 v = *reinterpret_cast<const float4*>(&tl[r * LDT + c4]);
            if (x0 * 32 + c4 < n_tiles * 32) *reinterpret_cast<float4*>(&Ps[(size_t)((mtw0 + mt) * 32 + r) * ldp + x0 * 32 + c4]) = v;
        }
        wave_lds_order();                                   // (the next m-tile overwrites the slice)
    }
    __syncthreads();                                        // the next tile's loads overwrite the LDS slices
    }
}

void launch_gemm_many(const u32x4* Wt, const float* wscale, const u32x4* Apk, float* P, int mt_total, int N, int K, GemmPlan plan,
                      hipStream_t s, const int* rows_live, u32x4* swiglu_out, LaunchStamps st) {
    const int n_tiles = N / 32, total_chunks = (K + 63) / 64, tiles_x = (n_tiles + 7) / 8, m_groups = (mt_total + plan.mt - 1) / plan.mt;
    const size_t split_stride = (size_t)mt_total * 32 * N;
    dim3 grid(std::min(tiles_x * m_groups * plan.split_k, 256));
#define MARGS Wt, wscale, Apk, P, split_stride, N, mt_total, n_tiles, total_chunks, plan.chunks_per_split, plan.split_k, tiles_x, rows_live, swiglu_out
#define MLAUNCH(MTW_, EPI_) hipExtLaunchKernelGGL(HIP_KERNEL_NAME(gemm_many_kernel<MTW_, EPI_>), grid, dim3(512), 0, s, st.start, st.stop, 0, MARGS)
    if (plan.mt == 6) { if (swiglu_out) MLAUNCH(3, MEPI_SWIGLU); else MLAUNCH(3, MEPI_PARTIAL); }
    else { if (swiglu_out) MLAUNCH(2, MEPI_SWIGLU); else MLAUNCH(2, MEPI_PARTIAL); }
#undef MLAUNCH
#undef MARGS
}
