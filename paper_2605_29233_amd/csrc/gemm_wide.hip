// Wide-format MFMA GEMM for passes of up to 128 rows (block steps); gemm_panel.hip takes the others:
//     C[m][n] = sum_k A[m][k] * W[n][k]          (fp32 accumulate)
// with the operands in the wide format of bb_internal.h: the activation as fp16 + a scaled e5m2 remainder, the
// weight as row-scaled fp16, converted in registers to e4m3 for the remainder's product.  Per 64 k and 32x32 tile
// that is four 32x32x16 fp16 MFMAs and one 32x32x64 fp8 MFMA, three quarters of the matrix work of two bf16 terms, at an
// accuracy of about 2^-16 per product.  Structure as the two-term
// kernel: C^T tiles with the weight fragment as the MFMA A-operand, one workgroup per CU, four waves that own
// 32 * NT weight rows each and share the activation chunk (32 MT rows x 64 k = 6 MT KiB) through LDS stages;
// weights stream HBM -> registers in a ring.  A workgroup walks its column groups with the grid's stride.  (The kernel of
// gemm_panel.hip keeps fewer weights on their way and is slower where the weight stream sets the pace: block steps of 120 rows 5.9 ms
// with this one, 6.1 with that; of 252 rows 4.9 with this one in two row groups, 4.7 with that.)
//
// What bounds it: what a CU draws, 30 KB per us of HBM lines with all 256 at it, 60 with 128, 92 with 64, however much more
// than 32 KB is requested ahead (plain load loops), of which a 256-column tile of 128 rows spends 24 of every
// 56 KB on activations; with few rows also the issue of MFMAs and LDS reads.  Hence a body per number of m-tiles: m-tiles past
// the rows the launch is sized for are neither fetched nor multiplied.  (Rows of finished branches and clipped windows inside
// them are: the kernel does not read the live row count.)  Measured, us per launch, body of 4 -> of 1 m-tile at
// 32 rows: 12288 x 4096 26.7 -> 19.9, 24576 x 4096 45.0 -> 33.8, 4096 x 12288 27.6 -> 18.7 (5.4 TB/s; reading the weights
// alone takes 17.6); of 2 at 56 rows: 27.5 -> 22.0, 45.5 -> 39.4, 27.6 -> 20.7; of 3 at 96 rows: 29.2 -> 24.0, 43.4 -> 41.6.
#include "bb_internal.h"
#include "lds.h"
#include "sched.h"
#include <hip/hip_ext.h>
#include <type_traits>
#include <algorithm>
#include <cmath>

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define KC 4                                    // fp16 k-steps (of 16) per chunk = weight fragments per (tile, chunk)

#define WEPI_PARTIAL 0
#define WEPI_SWIGLU 1

static __device__ __forceinline__ f16x8 as_f16x8(const u32x4& v) { return *reinterpret_cast<const f16x8*>(&v); }
static __device__ __forceinline__ i32x8 as_i32x8(const u32x4& a, const u32x4& b) {
    i32x8 r;
    r[0] = (int)a[0]; r[1] = (int)a[1]; r[2] = (int)a[2]; r[3] = (int)a[3];
    r[4] = (int)b[0]; r[5] = (int)b[1]; r[6] = (int)b[2]; r[7] = (int)b[3];
    return r;
}
// Eight fp16 weights (scaled by 2^S) -> eight e4m3 values of w 2^(S - BB_LO_SHIFT): the hardware conversion divides by its scale
// operand and rounds to nearest even; |w 2^S| < 2^15 keeps the result below e4m3's 448.  Each conversion writes one half of its
// destination and keeps the other, which the second one overwrites: starting from the sources saves clearing a register.
static __device__ __forceinline__ void fp16x8_to_e4m3x8(const u32x4& w, int& lo, int& hi) {
    // (the dwords are copied out first: a bit cast applied directly to a vector element picked element 0 every time)
    const unsigned int d0 = w[0], d1 = w[1], d2 = w[2], d3 = w[3];
    const float sc = (float)(1 << BB_LO_SHIFT);
    i16x2 a = __builtin_bit_cast(i16x2, d0), b = __builtin_bit_cast(i16x2, d2);
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(a, __builtin_bit_cast(f16x2, d0), sc, false);
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(a, __builtin_bit_cast(f16x2, d1), sc, true);
    b = __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(b, __builtin_bit_cast(f16x2, d2), sc, false);
    b = __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(b, __builtin_bit_cast(f16x2, d3), sc, true);
    lo = __builtin_bit_cast(int, a); hi = __builtin_bit_cast(int, b);
}

// WEPI_PARTIAL: P[split][m][n] (fp32, leading dimension ldp) = this workgroup's share of the k range.
// WEPI_SWIGLU: the weight matrix is the fused gate/up projection (32 gate rows alternate with the 32 up rows of the
// same features; k not split): writes SiLU(gate) * up as the wide-format panel Opk of the down projection.  With two tiles per
// wave both factors are in its registers; with one, waves 2 i and 2 i + 1 hold them and swap halves through LDS, so that each
// finishes 16 of the 32 features.  (Before, these passes stored the projection and a launch of its own read it back: us per
// layer, 24576 x 4096 at 32 rows 36.0 + 4.6 -> 36.3, 1408 x 256 at 56 rows 5.4 + 3.8 -> 8.1.)
//
// Chunk pipeline (one wave per SIMD, nothing else hides a stall), five phases per 64 k:
//   fp16 k-step 0: MFMAs | LDS reads of step 1 | LDS writes of chunk c+1's activations (loaded during c-AD), first half
//   fp16 k-step 1: MFMAs | LDS reads of step 2 | second half | global loads of chunk c+1+AD's activations, first half     -> barrier
//   fp16 k-step 2: MFMAs | LDS reads of step 3 | second half | chunk c+DW-1's weight fragment 0
//   fp16 k-step 3: MFMAs | LDS reads of the fp8 fragments | weight fragment 1 | this chunk's weights -> e4m3
//   fp8 step:      MFMAs | LDS reads of step 0 of chunk c+1 | weight fragments 2, 3
// With three or four m-tiles so; with fewer the activations are written in the first phase and requested in the second, and the weights
// in the third and fourth, two fragments each.  (All that in so few phases left four m-tiles waiting for the LDS in the first, 24 KB written and 16 read
// in 256 cycles, and for the load path in the next three.  us per launch at 112 rows, bunched -> spread, in turn: 24576 x 4096 49.6 -> 48.4,
// 37888 x 3584 72.4 -> 69.1, 3584 x 18944 36.3 -> 35.6, 4096 x 12288 28.4 -> 28.0, but 4096 x 4096, eight chunks per split, 14.7 -> 15.9; of three
// m-tiles within 1 %.  Whole steps: 37888 x 3584, 28 layers, 5642 -> 5496, 5729 -> 5647 on a second box, none on a third; 24576 x 4096 none.
// With one m-tile the even spread is 1 % slower, its weights come later.)
// With few accumulator tiles the registers hold a ring of four weight chunks, and activations that are requested two
// chunks ahead instead of one (64-row body, 37888 x 3584: 62.5 -> 57.4 us; with more tiles the deeper ring gains nothing).
template <int NT, int EPI, int MT, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 1) void gemm_wide_kernel(const u32x4* __restrict__ Wt, const float* __restrict__ wscale,
                                                           const u32x4* __restrict__ Apk, float* __restrict__ P,
                                                           size_t split_stride, int ldp, int mt_total, int n_tiles,
                                                           int total_chunks, int chunks_per_split, int tiles_x,
                                                           u32x4* __restrict__ Opk, const float* __restrict__ ssq, int nblk,
                                                           float inv_d, float eps) {
    static_assert(NT >= 1 && NT <= 2 && MT >= 1 && MT <= 4, "one or two weight tiles per wave, one to four m-tiles");
    constexpr int THREADS = 64 * WAVES;
    constexpr int WCHUNK_U4 = MT * BB_WFRAGS * 64;          // uint4 per staged activation chunk (6 KiB per m-tile)
    constexpr int WA_PER_THREAD = (WCHUNK_U4 + THREADS - 1) / THREADS;  // (an odd MT: the last half piece repeats valid data past the chunk's end)
    constexpr bool DEEP = NT * MT <= 4 && MT < 4, SPREAD = MT >= 3;
    constexpr int DW = DEEP ? 4 : 3, AD = DEEP ? 2 : 1;     // chunks in the weight ring and LDS; activation chunks in registers
    constexpr int COLS = 32 * NT, LDT = COLS + 4;           // store slices: row stride in floats (16-byte aligned, conflict-free)
    constexpr int MPP = NT <= 2 && MT % 2 == 0 ? 2 : 1;     // m-tiles per store pass
    constexpr int STAGES_U4 = DW * WA_PER_THREAD * THREADS, SLICES_U4 = WAVES * 32 * MPP * LDT / 4;
    __shared__ u32x4 lds_raw[STAGES_U4 > SLICES_U4 ? STAGES_U4 : SLICES_U4];
    u32x4 (*lds)[WA_PER_THREAD * THREADS] = reinterpret_cast<u32x4 (*)[WA_PER_THREAD * THREADS]>(lds_raw);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // Weight loads carry the non-temporal hint (every line is used once), and with a k split the (column group, split) items
    // are dealt to the 8 XCDs in contiguous runs in split-major order, so that an XCD's workgroups share one or two k ranges of
    // the activation panel (as in the two-term kernel).
    int first_tile = blockIdx.x, split_id = blockIdx.z;
    if (gridDim.z > 1) {
        const int n = gridDim.x * gridDim.z, lin = blockIdx.x + gridDim.x * blockIdx.z, e = lin & 7;
        const int item = e * (n >> 3) + min(e, n & 7) + (lin >> 3);
        first_tile = item % gridDim.x;
        split_id = item / gridDim.x;
    }
    for (int bx = first_tile; bx < tiles_x; bx += gridDim.x) {
    constexpr int mt0 = 0;
    const int mt_cnt = min(MT, mt_total - mt0);
    const int c0 = split_id * chunks_per_split;
    const int c1 = min(c0 + chunks_per_split, total_chunks);
    if (c0 >= c1) continue;

    const u32x4* wbase[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int x = min((bx * WAVES + wave) * NT + t, n_tiles - 1);      // clamped loads; stores are guarded
        wbase[t] = Wt + (size_t)x * total_chunks * (KC * 64);
    }
    unsigned aoff[WA_PER_THREAD];
#pragma unroll
    for (int i = 0; i < WA_PER_THREAD; ++i) {
        const int idx = i * THREADS + threadIdx.x, mt = idx / (BB_WFRAGS * 64), rem = idx % (BB_WFRAGS * 64);
        aoff[i] = min(mt, mt_cnt - 1) * (BB_WFRAGS * 64) + rem;        // missing m-tiles read a valid one
    }
    const u32x4* abase = Apk + (size_t)mt0 * (BB_WFRAGS * 64);
    const size_t a_chunk = (size_t)mt_total * (BB_WFRAGS * 64);
    // Past the end of the k range the loads are issued for the wait counts only: all lanes then read one address (a mask, not a
    // choice, which would cut the pipeline's block in two).  Before, they fetched the last chunk again two or three times, which
    // the epilogue then waited for.  us per launch, with the scalar bases and the prologue's order that came with it: at 32 rows,
    // 12288 x 4096 in two splits 20.7 -> 19.0, 24576 x 4096 37.5 -> 35.7, 4096 x 4096 and 4096 x 12288 in eight 14.9 -> 14.2 on
    // average; at 120 rows within 1 %.
    auto inside = [&](int c) { return (unsigned)((c - c1) >> 31); };
    auto load_a = [&](u32x4 (&a)[WA_PER_THREAD], int c, int lo, int hi) {
        const u32x4* p = abase + (size_t)min(c, c1 - 1) * a_chunk;
#pragma unroll
        for (int i = lo; i < hi; ++i) a[i] = p[aoff[i] & inside(c)];
    };
    auto load_w = [&](u32x4 (&w)[KC][NT], int c, int f_lo, int f_hi) {
        const size_t off = (size_t)min(c, c1 - 1) * (KC * 64);
        const unsigned l = lane & inside(c);
#pragma unroll
        for (int f = f_lo; f < f_hi; ++f)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                w[f][t] = __builtin_nontemporal_load(wbase[t] + off + f * 64 + l);
            }
    };
    auto read_bh = [&](u32x4 (&b)[MT], int stage, int k) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) b[mt] = lds[stage][(mt * BB_WFRAGS + k) * 64 + lane];
    };
    auto read_bl = [&](u32x4 (&b)[MT][2], int stage) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int p = 0; p < 2; ++p) b[mt][p] = lds[stage][(mt * BB_WFRAGS + 4 + p) * 64 + lane];
    };

    f32x16 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][mt][r] = 0.f;
    auto mfma_hi = [&](const u32x4 (&w)[NT], const u32x4 (&b)[MT]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(w[t]), as_f16x8(b[mt]), acc[t][mt], 0, 0, 0);
    };
    // A operand e4m3 (format 0), B operand e5m2 (format 1), both block scales 2^0
    auto mfma_lo = [&](const i32x8 (&w8)[NT], const u32x4 (&b)[MT][2]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t][mt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8[t], as_i32x8(b[mt][0], b[mt][1]),
                                                                            acc[t][mt], 0, 1, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
    };
    // k-steps 0, 2, 1, 3 of a lane's fp16 weights become the four 8-byte pieces of its fp8 operand (the order of the
    // panel's e5m2 fragments)
    auto convert_w = [&](i32x8 (&w8)[NT], const u32x4 (&w)[KC][NT]) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < KC; ++j) {
                int lo, hi;
                fp16x8_to_e4m3x8(w[j][t], lo, hi);
                const int o = 4 * (j & 1) + 2 * (j >> 1);
                w8[t][o] = lo; w8[t][o + 1] = hi;
            }
    };

    u32x4 w[DW][KC][NT], a[AD][WA_PER_THREAD], bh[2][MT], bl[MT][2];
    i32x8 w8[NT];
    // prologue: chunk c0 staged, AD chunks of activations in registers, weights of DW - 1 chunks in flight; loads in the
    // order the loop issues them (activations of a chunk, then its weights), so that the wait counts at the loop head, the
    // more cautious of the two ways in, are those of the steady state
    auto first_a = [&](u32x4 (&a)[WA_PER_THREAD], int c) { load_a(a, c, 0, WA_PER_THREAD); __builtin_amdgcn_sched_barrier(0); };
    auto first_w = [&](u32x4 (&w)[KC][NT], int c) { unroll<KC>([&](auto F) { load_w(w, c, F, F + 1); __builtin_amdgcn_sched_barrier(0); }); };
    unroll<AD>([&](auto I) { first_a(a[I], c0 + I); first_w(w[I], c0 + I); });
#pragma unroll
    for (int i = 0; i < WA_PER_THREAD; ++i) lds[0][i * THREADS + threadIdx.x] = a[0][i];
    first_a(a[0], c0 + AD);
    unroll<DW - 1 - AD>([&](auto I) { first_w(w[AD + I], c0 + AD + I); });
    __syncthreads();
    read_bh(bh[0], 0, 0);

    constexpr int WA1 = SPREAD ? (WA_PER_THREAD + 1) / 2 : WA_PER_THREAD, W1 = SPREAD ? 1 : 2, W2 = SPREAD ? 2 : KC;     // activation pieces and weight fragments up to a phase
    auto write_a = [&](auto Stage, auto As, auto Lo, auto Hi) {
#pragma unroll
        for (int i = decltype(Lo)::value; i < decltype(Hi)::value; ++i) lds[decltype(Stage)::value][i * THREADS + threadIdx.x] = a[decltype(As)::value][i];
    };
    auto chunk = [&](auto U, int c) {
        constexpr int u = decltype(U)::value, st = u, st1 = (u + 1) % DW, slot2 = (u + DW - 1) % DW, as = (u + 1) % AD;
        __builtin_amdgcn_sched_barrier(0);  // (a conversion moved up from a later chunk would wait for that chunk's loads)
        // fp16 k-step 0
        read_bh(bh[1], st, 1);
        write_a(IC(st1), IC(as), IC(0), IC(WA1));
        mfma_hi(w[u][0], bh[0]);
        sched_groups<MT, NT, MT, WA1, 0>();
        // fp16 k-step 1
        read_bh(bh[0], st, 2);
        write_a(IC(st1), IC(as), IC(WA1), IC(WA_PER_THREAD));
        load_a(a[as], c + 1 + AD, 0, WA1);
        mfma_hi(w[u][1], bh[1]);
        sched_groups<MT, NT, MT, WA_PER_THREAD - WA1, WA1>();
        __syncthreads();                    // chunk c+1 is staged; the stage of chunk c-1 is free again
        // fp16 k-step 2
        read_bh(bh[1], st, 3);
        load_a(a[as], c + 1 + AD, WA1, WA_PER_THREAD);
        load_w(w[slot2], c + DW - 1, 0, W1);
        mfma_hi(w[u][2], bh[0]);
        sched_groups<MT, NT, MT, 0, WA_PER_THREAD - WA1 + W1 * NT>();
        // fp16 k-step 3 (and the conversion of this chunk's weights for the fp8 step)
        read_bl(bl, st);
        load_w(w[slot2], c + DW - 1, W1, W2);
        convert_w(w8, w[u]);
        mfma_hi(w[u][3], bh[1]);
        sched_groups<MT, NT, 2 * MT, 0, (W2 - W1) * NT>();
        // fp8 step (reads the first fp16 fragments of the next chunk)
        read_bh(bh[0], st1, 0);
        load_w(w[slot2], c + DW - 1, W2, KC);
        mfma_lo(w8, bl);
        sched_groups<MT, NT, MT, 0, (KC - W2) * NT>();
    };
    int c = c0;
    for (; c + DW <= c1; c += DW) unroll<DW>([&](auto U) { chunk(U, c + U); });
    unroll<DW - 1>([&](auto U) { if (c + U < c1) chunk(U, c + U); });

    // undo the per-row weight scale: register r of lane (m = l % 32, g = l / 32) holds weight row 8 (r/4) + 4 g + r%4
    const int x0 = (bx * WAVES + wave) * NT, g = lane >> 5;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int x = min(x0 + t, n_tiles - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 s4 = *reinterpret_cast<const float4*>(&wscale[x * 32 + 8 * q + 4 * g]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                acc[t][mt][4 * q] *= s4.x; acc[t][mt][4 * q + 1] *= s4.y; acc[t][mt][4 * q + 2] *= s4.z; acc[t][mt][4 * q + 3] *= s4.w;
            }
        }
    }
    __syncthreads();                                        // all waves are done with the staged activations
    if constexpr (EPI == WEPI_SWIGLU) {
        static_assert(WAVES % 2 == 0 || NT == 2, "gate and up tiles of a feature group sit in one wave or in two neighbours");
        static_assert(NT == 2 || WAVES * MT * 128 <= STAGES_U4, "the swapped halves");
        float4* swap = reinterpret_cast<float4*>(lds_raw);
        if constexpr (NT == 1) {                            // half 0 (features 0..15 of the group) is the gate wave's, half 1 the up wave's
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    float4 v;
                    const int r = 4 * q;
                    v.x = wave & 1 ? acc[0][mt][r] : acc[0][mt][8 + r]; v.y = wave & 1 ? acc[0][mt][r + 1] : acc[0][mt][9 + r];
                    v.z = wave & 1 ? acc[0][mt][r + 2] : acc[0][mt][10 + r]; v.w = wave & 1 ? acc[0][mt][r + 3] : acc[0][mt][11 + r];
                    swap[((wave * MT + mt) * 2 + q) * 64 + lane] = v;
                }
            __syncthreads();
        }
        // The panel wants the 8 features of group q in one lane of lane-half q % 2: lane halves swap the 4-feature
        // pieces they do not own, then each lane stores the groups q = g and g + 2.
        if (x0 < n_tiles) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (mt >= mt_cnt) break;
                // ssq: the activation rows were packed without their RMSNorm scale (sums of squares per block of
                // columns instead); both factors of the product take 1 / rms of this lane's row here
                float inv = 1.0f;
                if (ssq) {
                    const int m = (mt0 + mt) * 32 + (lane & 31);
                    float t = 0.f;
                    for (int b = 0; b < nblk; ++b) t += ssq[m * nblk + b];
                    inv = 1.0f / sqrtf(t * inv_d + eps);
                }
                auto pair = [&](int p2, const float (&act)[8]) {        // features 16 p2 .. 16 p2 + 15 of the group
                    float y[8];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float e0 = act[i], e1 = act[4 + i];
                        const float mine = g == 0 ? e0 : e1;                     // group q = 2 p2 + g is mine
                        const float send = g == 0 ? e1 : e0;                     // the other lane half owns that group
                        const float recv = __shfl_xor(send, 32, 64);
                        y[i] = g == 0 ? mine : recv;
                        y[4 + i] = g == 0 ? recv : mine;
                    }
                    store_panel8(Opk, (mt0 + mt) * 32 + (lane & 31), (x0 / 2) * 4 + 2 * p2 + g, mt_total, y, 1);
                };
                auto swiglu = [&](float gate, float up) {
                    const float gt = gate * inv, u = up * inv;
                    return gt / (1.0f + expf(-gt)) * u;
                };
                if constexpr (NT == 2) {
#pragma unroll
                    for (int p2 = 0; p2 < 2; ++p2) {
                        float act[8];
#pragma unroll
                        for (int r = 0; r < 8; ++r) act[r] = swiglu(acc[0][mt][8 * p2 + r], acc[NT - 1][mt][8 * p2 + r]);
                        pair(p2, act);
                    }
                } else {
                    float act[8];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const float4 v = swap[(((wave ^ 1) * MT + mt) * 2 + q) * 64 + lane];
                        const float o[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = 4 * q + i;
                            act[r] = wave & 1 ? swiglu(o[i], acc[0][mt][8 + r]) : swiglu(acc[0][mt][r], o[i]);
                        }
                    }
                    pair(wave & 1, act);
                }
            }
        }
        if constexpr (NT == 1) __syncthreads();             // the next tile's prologue overwrites the halves
        continue;
    }
    // Partial tiles go out through LDS so that a wave stores whole 128-byte lines.
    float* tl = reinterpret_cast<float*>(lds_raw) + wave * (32 * MPP * LDT);
    float* Ps = P + (size_t)split_id * split_stride;
#pragma unroll
    for (int pass = 0; pass < MT / MPP; ++pass) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int mh = 0; mh < MPP; ++mh)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x16& a4 = acc[t][MPP * pass + mh];
                    *reinterpret_cast<float4*>(&tl[(mh * 32 + (lane & 31)) * LDT + t * 32 + 8 * q + 4 * g]) =
                        make_float4(a4[4 * q], a4[4 * q + 1], a4[4 * q + 2], a4[4 * q + 3]);
                }
        wave_lds_order();                                   // (the same wave wrote and reads: no barrier needed)
        constexpr int LPR = COLS / 4;                       // lanes per row
        const int rows_valid = min(32 * MPP, (mt_cnt - MPP * pass) * 32);
#pragma unroll
        for (int it = 0; it < 32 * MPP * LPR / 64; ++it) {
            const int idx = it * 64 + lane, r = idx / LPR, c4 = (idx % LPR) * 4;
            const float4 v = *reinterpret_cast<const float4*>(&tl[r * LDT + c4]);
            const int n = x0 * 32 + c4;
            if (r < rows_valid && n < n_tiles * 32)
                *reinterpret_cast<float4*>(&Ps[(size_t)((mt0 + MPP * pass) * 32 + r) * ldp + n]) = v;
        }
        wave_lds_order();                                   // (the next pass overwrites the slice)
    }
    __syncthreads();                                        // the next tile's prologue overwrites the LDS slices
    }
}

// Up to 256 rows: row groups of at most four m-tiles, dealt evenly (384-column tiles have the body of four only).
static int block_step_body(int mt_total, int nt) {
    const int groups = (mt_total + 3) / 4;
    return nt == 3 ? 4 : (mt_total + groups - 1) / groups;
}

// fusable: only bb_debug_gemm_plan and the sizing of the buffers set it here.  A forward of up to 128 rows does not, since its norm
// is deferred, although it does take SwiGLU from the epilogue of any plan that leaves k whole, with one tile per wave too: neither
// the SwiGLU launch behind a split plan nor the partial tiles that a fused one does not write are in the price of its plans.
static GemmPlan plan_one_group(int mt_total, int N, int K, bool fusable) {
    const int n_tiles = N / 32, total_chunks = (K + 63) / 64;
    GemmPlan best;
    double best_t = 1e30;
    for (int nt = 1; nt <= 2; ++nt) {
        if (nt > 1 && n_tiles < 4 * nt) continue;
        const int base = (n_tiles + 4 * nt - 1) / (4 * nt);
        for (int sp = 1; sp <= BB_MAX_SPLITK && sp <= std::max(1, total_chunks / 4) && (sp == 1 || base * sp <= 256); ++sp) {
            const int cps = (total_chunks + sp - 1) / sp;
            if ((total_chunks + cps - 1) / cps != sp) continue;
            const double live = std::min(base * sp, 256), weights_kb = 16.4 * nt, acts_kb = 6.1 * mt_total;
            const double own_us = (nt == 1 ? 0.68 : 1.08) * (mt_total == 4 ? 1.0 : 0.88);
            const double chunk_us = std::max(own_us, live * std::max(weights_kb / 6.0e3, (weights_kb + acts_kb) / 15e3));
            const bool fused = fusable && sp == 1 && nt == 2;
            const double partial_mb = (double)sp * mt_total * 32 * N * 4e-6;
            const double t = ((base * sp + 255) / 256) * (cps * chunk_us + 6.0) + (fused ? 3.0 : 0.34 * partial_mb + (fusable ? 8.0 : 0.0));
            if (t < best_t) { best_t = t; best.nt = nt; best.split_k = sp; best.chunks_per_split = cps; }
        }
    }
    return best;
}

static GemmPlan plan_two_groups(int mt_total, int N, int K, bool fusable) {
    const int n_tiles = N / 32, total_chunks = (K + 63) / 64, groups = 2;
    GemmPlan best;
    double best_t = 1e30;
    for (int nt = 1; nt <= 3; ++nt) {
        if (nt > 1 && n_tiles < 4 * nt) continue;
        const int body = block_step_body(mt_total, nt), base = (n_tiles + 4 * nt - 1) / (4 * nt) * groups;
        const double own = body == 3 ? (nt == 1 ? 0.535 : 0.80) : nt == 1 ? 0.60 : nt == 2 ? 0.93 : 1.43;
        for (int sp = 1; sp <= BB_MAX_SPLITK && sp <= std::max(1, total_chunks / 4) && (sp == 1 || base * sp <= 256); ++sp) {
            const int cps = sp == 1 ? total_chunks : ((total_chunks + sp - 1) / sp + 1) / 2 * 2;
            if ((total_chunks + cps - 1) / cps != sp) continue;
            const int items = base * sp;
            const double live = std::min(items, 256), fill = live / 256, last = (items % 256) / 256.0;
            const double own_us = own * (nt == 1 ? 1.0 : 1.0 + 0.126 * fill * fill);
            const double fetch_us = live * (16.4 * nt / groups / 7.46e3 + 6.1 * body / 18.3e3);
            const double rounds = items <= 256 ? 1.0 : items / 256 + (last > 0 ? 0.62 + 0.38 * last : 0.0);
            const bool fused = fusable && sp == 1 && nt == 2;
            const double partial_mb = fused ? 0.0 : (double)sp * mt_total * 32 * N * 4e-6;
            const double t = rounds * (cps * sqrt(own_us * own_us + fetch_us * fetch_us) + 0.47 * nt * body) + 0.22 * partial_mb + (fusable && !fused ? 8.0 : 0.0);
            if (t < best_t) { best_t = t; best.nt = nt; best.split_k = sp; best.chunks_per_split = cps; }
        }
    }
    return best;
}

// Plan of a wide-format GEMM.
//
// Up to 64 rows: tiles 128 columns wide wherever one round holds them: activations are then little of what a CU
// fetches, and few k splits are written and read back (12288 x 4096 at 32 rows, two splits against five of 256 columns: 19.9
// against 21.4 us and a shorter consumer; 24576 x 4096 33.8, unsplit, against 35.9).  Else 192 (three waves) if that is one
// round: 198 of the CUs have work instead of 148 (37888 x 3584, 56 rows, with SwiGLU: 50.1 against 57.5 us; at 120 rows, where
// the waves' own work sets the pace, 74.2 against 68.2).
//
// 65 to 128 rows: the candidates (tile width, k split) are priced by a model of 150 measured launches at 120 and 240 rows (those of 240
// with the two row groups that this kernel had then; the body of three m-tiles by one common factor): time of one 64-k chunk of a workgroup, at least what its share of the weight stream takes (6 TB/s; of
// everything the L2s deliver, 15 TB/s), 6 us of prologue and store per tile, and the partial tiles, written here and read by the
// consumer.  (12288 x 4096 at 120 rows: four splits on 192 CUs 27.6 us, five on 240 27.5 and a longer consumer.)
//
// 129 to 256 rows, two row groups of gemm_panel_kernel: the same by a model of 1486 measured launches (72..256 rows, N 256..37888, K
// 256..18944; 6 % rms): a chunk takes the root of the squares of the waves' own work and of its share of what HBM (7.5 TB/s, each
// weight line once) and the L2s (18 TB/s) deliver; partial tiles cost 0.07 us per MB here and 0.15 in the consumer.  Its choice costs 0.6 % more
// than the best of the measured plans (37888 x 3584 at 240 rows: one round of 384 columns 119 us and a SwiGLU launch, two of 256
// columns with SwiGLU in the epilogue 148; 24576 x 4096 in one round of 256 columns 84).  Splits take whole units of 128 k.
//
// With more rows tiles of 128 or 192 rows x 256 columns and their k splits
// are priced by a model fitted to 800 measured launches of the eight-wave kernel that these passes had before (272..4206 rows, N 3584..37888, K
// 3584..18944; 4.6 % rms): time of one 64-k chunk of a workgroup tile, a fixed cost per tile, whole rounds of 256
// workgroups except that a last round which leaves CUs idle runs at a higher clock, and
// the partial tiles, written here and read by the consumer launch once per k split.  The constants are not those of gemm_panel_kernel (a chunk of 192
// rows takes it 1.6 us, a tile 9 us more); its choices were measured on it, 68 shapes of 273..4120 rows with every tile and up to eight splits: 0.3 % more than
// the best on average, 5 % at 931 x 3584 x 3584, and just above 256 rows, where tiles of 96 rows x 128 columns would be better, 6 to 9 % and once 27 % (273 x 3584 x 3584).
// Where both tiles price within 5 % the larger one is taken: it fetches a fifth less per product.  fusable: the caller
// can take SiLU(gate) * up from the epilogue when k is not split; then there are no partial tiles and no launch for it.
// Beside them tiles of 128 columns, where they and their k splits fit one round: small matrices leave
// most CUs without work either way, and the smaller tile is through sooner.  Its price is fitted to 175
// shapes (272..4096 rows, N 128..4096, K 64..4096) of the kernels before; on the present one, us of 256 / of 128 columns: 768 x 256 at 512 rows 8.8 /
// 5.9, 256 x 688 at 1024 rows 10.5 / 6.9, 1408 x 256 at 1536 rows 9.8 / 7.1, but 3584 x 3584 at 1024 rows 38 / 43.
GemmPlan gemm_plan_wide(int m_rows, int N, int K, int forced_split, int forced_nt, bool fusable) {
    const int mt_total = (m_rows + 31) / 32;
    if (mt_total <= 8) {
        GemmPlan p;
        if (forced_split > 0 || forced_nt > 0) p = gemm_plan(m_rows, N, K, forced_split, forced_nt);
        else if (mt_total <= 2) {
            p = gemm_plan(m_rows, N, K, 0, (N / 32 + 3) / 4 <= 256 ? 1 : 0);
            if (p.nt == 2 && p.split_k == 1 && (N / 32 + 5) / 6 <= 256) p.wv = 3;
        } else p = mt_total <= 4 ? plan_one_group(mt_total, N, K, fusable) : plan_two_groups(mt_total, N, K, fusable);
        p.mt = block_step_body(mt_total, p.nt);
        return p;
    }
    if (forced_split > 0) return gemm_plan(m_rows, N, K, forced_split, forced_nt);
    const int n_tiles = N / 32, total_chunks = (K + 63) / 64;
    GemmPlan best;
    best.nt = 2;
    double best_t = 1e30;
    for (int mt = 4; mt <= 6; mt += 2) {
        const double chunk_us = mt == 6 ? 1.67 : 1.18, tile_us = 3.8;
        const long tiles = (long)((n_tiles + 7) / 8) * ((mt_total + mt - 1) / mt);
        for (int sp = 1; sp <= BB_MAX_SPLITK && sp <= std::max(1, total_chunks / 4); ++sp) {
            const int cps = sp == 1 ? total_chunks : ((total_chunks + sp - 1) / sp + 1) / 2 * 2, sp_eff = (total_chunks + cps - 1) / cps;
            const long items = tiles * sp_eff;
            const double last = (items % 256) / 256.0, rounds = items / 256 + (last > 0 ? 0.62 + 0.38 * last : 0.0);
            double t = 2.0 + rounds * (cps * chunk_us + tile_us);
            if (!(fusable && sp_eff == 1)) t += (fusable ? 8.0 : 0.0) + sp_eff * (double)mt_total * 32 * N * 4 * (0.066e-6 + 0.1e-6);
            if (mt == 6) t *= 0.95;
            if (t < best_t) { best_t = t; best.split_k = sp_eff; best.chunks_per_split = cps; best.mt = mt; }
        }
    }
    const int base = (n_tiles + 3) / 4 * ((mt_total + 3) / 4);
    for (int sp = 1; sp <= BB_MAX_SPLITK && sp <= std::max(1, total_chunks / 4) && base * sp <= 256; ++sp) {
        const int cps = (total_chunks + sp - 1) / sp;
        if ((total_chunks + cps - 1) / cps != sp) continue;
        const double fill = base * sp / 256.0, partial = sp * (double)mt_total * 32 * N * 4 * (sp == 1 ? 0.166e-6 : 0.25e-6);
        const double t = 4.0 + cps * 0.585 * (1.0 + 0.8 * fill * fill * fill) + partial + (fusable ? 8.0 : 0.0);
        if (t < best_t) { best_t = t; best.split_k = sp; best.chunks_per_split = cps; best.nt = 1; best.mt = block_step_body(mt_total, 1); }
    }
    return best;
}

void launch_gemm_wide(const u32x4* Wt, const float* wscale, const u32x4* Apk, float* P, int mt_total, int N, int K,
                      GemmPlan plan, hipStream_t s, u32x4* swiglu_out, LaunchStamps st, const float* ssq, int nblk, float rms_eps,
                      const int* rows_live) {
    if (mt_total > 4 || plan.nt == 3) {         // (up to 256 rows both row groups are computed whatever the live row count: only the passes of more rows look at it)
        launch_gemm_panel(Wt, wscale, Apk, P, mt_total, N, K, plan, s, mt_total > 8 ? rows_live : nullptr, swiglu_out, st);
        return;
    }
    const int n_tiles = N / 32, total_chunks = (K + 63) / 64, nt = plan.nt;
    const size_t split_stride = (size_t)mt_total * 32 * N;
    const int tiles_x = (n_tiles + plan.wv * nt - 1) / (plan.wv * nt);
    dim3 grid(std::min(tiles_x, 256), 1, plan.split_k);
#define WARGS Wt, wscale, Apk, P, split_stride, N, mt_total, n_tiles, total_chunks, plan.chunks_per_split, tiles_x, swiglu_out, ssq, nblk, 1.0f / (float)K, rms_eps
#define WLAUNCH(NT_, EPI_, MT_, WV_) hipExtLaunchKernelGGL(HIP_KERNEL_NAME(gemm_wide_kernel<NT_, EPI_, MT_, WV_>), grid, dim3(64 * WV_), 0, s, st.start, st.stop, 0, WARGS)
#define WLAUNCH_MT(NT_, EPI_) do { \
        if (mt_total == 1) WLAUNCH(NT_, EPI_, 1, 4); \
        else if (mt_total == 2) WLAUNCH(NT_, EPI_, 2, 4); \
        else if (mt_total == 3) WLAUNCH(NT_, EPI_, 3, 4); \
        else WLAUNCH(NT_, EPI_, 4, 4); \
    } while (0)
    if (plan.wv == 3) {
        if (swiglu_out) { if (mt_total == 1) WLAUNCH(2, WEPI_SWIGLU, 1, 3); else WLAUNCH(2, WEPI_SWIGLU, 2, 3); }
        else { if (mt_total == 1) WLAUNCH(2, WEPI_PARTIAL, 1, 3); else WLAUNCH(2, WEPI_PARTIAL, 2, 3); }
    } else if (swiglu_out && nt == 2) WLAUNCH_MT(2, WEPI_SWIGLU);
    else if (swiglu_out) WLAUNCH_MT(1, WEPI_SWIGLU);
    else if (nt == 2) WLAUNCH_MT(2, WEPI_PARTIAL);
    else WLAUNCH_MT(1, WEPI_PARTIAL);
#undef WLAUNCH_MT
#undef WLAUNCH
#undef WARGS
}

// bf16 weights [rows][K] -> row-scaled fp16 in the tiled layout of the bf16 copy.  One workgroup per source row: the
// row's largest magnitude fixes its power-of-two scale 2^S (largest value into [2^14, 2^15)); fp16(w 2^S) is then
// exact unless w is below 2^-29 of the row's largest value; scale_out[row] = 2^-S.  K is padded to whole chunks of 64
// (the padding must be zero: the destination is cleared beforehand).  interleave: fused gate/up, 32 rows of one
// alternate with 32 of the other.
__global__ __launch_bounds__(256) void tile_weights_wide_kernel(const uint16_t* __restrict__ src, int K, u32x4* __restrict__ dst,
                                                                float* __restrict__ scale_out, int row0, int interleave, int ksteps_pad) {
    __shared__ float sh[4];
    const int r = blockIdx.x;
    const int n = interleave ? (r / 32) * 64 + r % 32 + row0 : row0 + r;
    const u32x4* row = reinterpret_cast<const u32x4*>(src + (size_t)r * K);
    const int k8s = K >> 3;
    float mx = 0.f;
    for (int k8 = threadIdx.x; k8 < k8s; k8 += 256) {
        const u32x4 v = row[k8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            mx = fmaxf(mx, fabsf(bf16_to_f32((uint16_t)(v[j] & 0xFFFFu))));
            mx = fmaxf(mx, fabsf(bf16_to_f32((uint16_t)(v[j] >> 16))));
        }
    }
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
    int S = 0;
    if (mx > 0.f && mx < INFINITY) {
        int e; (void)frexpf(mx, &e);            // mx = f 2^e, f in [0.5, 1)
        S = max(-100, min(100, 15 - e));        // mx 2^S in [2^14, 2^15)
    }
    const float up = ldexpf(1.0f, S);
    if (threadIdx.x == 0) scale_out[n] = ldexpf(1.0f, -S);
    for (int k8 = threadIdx.x; k8 < k8s; k8 += 256) {
        const u32x4 v = row[k8];
        f16x8 hi;
#pragma unroll
        for (int j = 0; j < 8; ++j) hi[j] = (half_t)(bf16_to_f32((uint16_t)((v[j >> 1] >> (16 * (j & 1))) & 0xFFFFu)) * up);
        dst[tileW_u4(n, k8, ksteps_pad)] = __builtin_bit_cast(u32x4, hi);
    }
}

void launch_tile_weights_wide(const uint16_t* src, int rows, int K, u32x4* dst, float* scale_out, int dst_row0, int interleave,
                              hipStream_t s) {
    tile_weights_wide_kernel<<<rows, 256, 0, s>>>(src, K, dst, scale_out, dst_row0, interleave, (K + 63) / 64 * 4);
}

// fp32 row-major [M][K] -> wide-format panel; rows >= M and columns >= K (padding to whole chunks) are zero.
__global__ void pack_rows_wide_kernel(const float* __restrict__ A, int M, int K, u32x4* __restrict__ Apk, int mt_total) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    int k8s = (K + 63) / 64 * 8;
    if (i >= (size_t)mt_total * 32 * k8s) return;
    int m = (int)(i / k8s), k8 = (int)(i % k8s);
    float y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = m < M && k8 * 8 < K ? A[(size_t)m * K + k8 * 8 + j] : 0.f;
    store_panel8(Apk, m, k8, mt_total, y, 1);
}

void launch_pack_rows_wide(const float* A, int M, int K, u32x4* Apk, int mt_total, hipStream_t s) {
    size_t n = (size_t)mt_total * 32 * ((K + 63) / 64 * 8);
    pack_rows_wide_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(A, M, K, Apk, mt_total);
}
