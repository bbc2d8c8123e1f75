// Bidirectional softmax attention of packed query rows against a branch's paged KV cache row.
//
// Work is cut into tiles of 32 "flattened" query rows (the query heads that share a kv head are
// folded into the row dimension, so the K/V tiles a wave reads serve all of them), one kv head,
// one branch segment.  K and V are found page by page (64 tokens) through the branch's page
// table: shared or private physical row.  Two kernels:
//   attention_kernel (block steps, and full passes with few tiles): one tile per workgroup, the waves take the
//            row's pages round robin, each keeping a running max / sum / output (online
//            softmax), and the partial results are combined through LDS in a fixed order;
//   attention_full_kernel (full-sequence passes with many tiles): four tiles per workgroup, one per
//            wave; the waves walk the pages together, through LDS.
// Either way the result does not depend on scheduling.
//
// Q, K, V and the probabilities P each enter as two fp16 terms (hi + lo); every product keeps
// the three leading cross terms (hi.hi + lo.hi + hi.lo), i.e. ~22 bits per operand.
//
// MFMA use (fp16 inputs, fp32 accumulate, 32x32x16):
//   S^T[key][query]  = K[key][:] . Q[query][:]      A = K fragments (the cache stores them ready-made), B = Q rows
//   O^T[d][query]   += V^T[d][key] . P^T[key][query] A = V^T fragments (likewise),
//                                                    B = P taken straight from the S^T
//                                                    accumulators (same lane owns the same
//                                                    query), keys permuted consistently.
#include "bb_internal.h"
#include "lds.h"
#include <algorithm>
#include <type_traits>

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

static __device__ __forceinline__ f16x8 as_f16x8(const u32x4& v) { return *reinterpret_cast<const f16x8*>(&v); }
#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0)

// One page of the online softmax for a lane's 32 scores (16 consecutive keys of each key tile, one query).
// Scores arrive in the log2 domain (the queries were scaled by log2(e) / sqrt(hd) when they were written),
// so the exponentials are single v_exp_f32.  Updates the running max / sum, rescales the output
// accumulators when some lane's max moved, and returns P as two fp16 terms in B-fragment order
// (fragment kk = 2 kt + h: slot j of lane group g holds key 32 kt + 16 g + 8 h + j).
template <int DT>
static __device__ __forceinline__ void softmax_page(f32x16 (&s)[2], bool partial_page, int t0, int L, int g, float& m_run,
                                                    float& l_run, f32x16 (&o)[DT], f16x8 (&ph)[4], f16x8 (&pl)[4]) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    if (partial_page) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (t0 + 32 * kt + 16 * g + r >= L) s[kt][r] = -INFINITY;
    }
    float mx = s[0][0];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);                           // finite: every page holds a valid key
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);      // 2^-inf = 0 on the first page
    float sum = 0.f;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const f32x2 p = {__builtin_amdgcn_exp2f(s[kt][r] - m_new), __builtin_amdgcn_exp2f(s[kt][r + 1] - m_new)};
            sum += p[0] + p[1];
            const f16x2 hi = __builtin_convertvector(p, f16x2);
            const f32x2 rem = p - __builtin_convertvector(hi, f32x2);
            const f16x2 lo = __builtin_convertvector(rem, f16x2);
            const int kk = 2 * kt + (r >> 3);
            ph[kk][r & 7] = hi[0]; ph[kk][(r & 7) + 1] = hi[1];
            pl[kk][r & 7] = lo[0]; pl[kk][(r & 7) + 1] = lo[1];
        }
    l_run = l_run * alpha + sum;
    m_run = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f)) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
    }
}

// WAVES waves per workgroup, two per SIMD either way: eight of one workgroup, or four each of two.  What bounds it: the K,V
// stream, which short rows and few tiles leave at the 50-60 KB per us that a CU draws by itself (long ones: 4.5 TB/s of 671 MB
// over 256 workgroups), and each wave's own chain of loads, MFMAs and exponentials, which the second wave of its SIMD fills.  So a wave keeps to
// 256 registers: two quarters of a K or V page in flight, and Q in LDS (all waves use the same fragments), in the space
// that the waves' results take after the last page.
// Measured, us per launch (heads of 128; before = four waves with 512 registers each, half pages in flight): 768 keys, 320 tiles
// 46.8 -> 43.3, 160 tiles 27.3 -> 26.5, 32 tiles in three splits 14.2 -> 13.1; 5120 keys, 256 tiles 149 -> 149.
template <int HD, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void attention_kernel(Dev D, const half_t* __restrict__ Q, u32x4* __restrict__ Apk,
                                                        int layer, int mt_total, int seg_base, int n_splits,
                                                        float* __restrict__ part, int wide) {
    constexpr int KS = HD / 16;         // k-steps of the score contraction
    constexpr int DT = HD / 32;         // 32-wide tiles of the output's head dimension
    constexpr int THREADS = 64 * WAVES;
    __shared__ u32x4 sQO[(WAVES * 32 * (HD + 1) + 3) / 4];
    static_assert(2 * KS * 64 <= (int)(sizeof(sQO) / 16), "Q fragments exceed the results' space");
    float (*sO)[32][HD + 1] = reinterpret_cast<float (*)[32][HD + 1]>(sQO);
    __shared__ float sM[WAVES][32], sL[WAVES][32];

    // Grid = (kv head, query tile [x split], segment).  The kv head is the fastest index on purpose: workgroups go
    // to the eight XCDs round robin by linear id, so with a multiple of eight kv heads all query tiles and page
    // splits of one (branch, kv head) land on the same XCD and its L2 fetches that row's pages from HBM once.
    const int gbr = seg_base + blockIdx.z;
    const int seg_rows = D.seg_rows[gbr];
    if (seg_rows == 0) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 5, c = lane & 31;
    const int group = D.hq / D.hkv, nflat = seg_rows * group;
    // a row's pages may also be split over n_splits workgroups (blockIdx.y = tile * n_splits + split)
    const int split = blockIdx.y % n_splits, qtile = blockIdx.y / n_splits, wg_base = qtile * 32;
    if (wg_base >= nflat) return;
    const int kvh = blockIdx.x, seg_off = D.seg_off[gbr];
    const int L = D.hdr[gbr / D.max_br].L, n_pages = (L + BB_PAGE - 1) / BB_PAGE;

    const int pps = (n_pages + n_splits - 1) / n_splits;           // pages per split
    const int p0 = split * pps + wave, p1 = min(n_pages, (split + 1) * pps);
    // A page's K and V fragments (NF x 1 KiB each way) pass through a ring of two quarters: a quarter is requested as soon as
    // the MFMAs that read its place in the ring have been issued.
    constexpr int NF = 4 * KS, QF = NF / 4;         // (NF = DT * 4 * 2 as well)
    u32x4 kv[2][QF];
    auto block = [&](const half_t* cache, int page) {
        const int phys = D.table[(size_t)gbr * D.n_pages + page];
        return reinterpret_cast<const u32x4*>(cache + kv_block_off(D, layer, phys, page, kvh)) + lane;
    };
    auto fetch = [&](int q, const u32x4* src) {     // quarter q of a block
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < QF; ++i) kv[q & 1][i] = src[(q * QF + i) * 64];
        __builtin_amdgcn_sched_barrier(0);
    };
    const u32x4* Kp = block(D.Kc, min(p0, D.n_pages - 1));
    if (p0 < p1) { fetch(0, Kp); fetch(1, Kp); }
    // Q fragments (B operand).  The contraction index may be enumerated in any order as long as K uses the
    // same one: k-step ks, lane group g, slot j  <->  head dim (HD/2) g + 8 ks + j, so a lane's KS fragments
    // of a row are one contiguous run of HD/2 values.  Rows past the end repeat the last row (never stored).
    for (int i = wave; i < 2 * KS; i += WAVES) {    // fragment i = term * KS + ks
        const int f = min(wg_base + c, nflat - 1), hig = f / seg_rows, r = f % seg_rows;
        sQO[i * 64 + lane] = *reinterpret_cast<const u32x4*>(Q + ((size_t)(seg_off + r) * D.hq + kvh * group + hig) * 2 * HD + (HD / 2) * g +
                                                             (i / KS) * HD + 8 * (i % KS));
    }
    __syncthreads();
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    for (int page = p0; page < p1; page += WAVES) {
        const int t0 = page * BB_PAGE, nxt = page + WAVES;
        const u32x4* Vp = block(D.Vt, page);
        const u32x4* Kn = block(D.Kc, min(nxt, D.n_pages - 1));
        // scores: two tiles of 32 keys.  The cache stores MFMA row i of a tile as key pi(i) = i%4 + 4 (i/8) + 16 ((i/4)%2),
        // which makes the 16 accumulator registers of a lane the 16 consecutive keys t0 + 32 kt + 16 g + r
        // (query c): the order of the V^T fragments' contraction index.  Fragment pair (kt, ks) = pair kt KS + ks of the page.
        f32x16 s[2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int i = 0; i < QF / 2; ++i) {
                const int kt = (q * (QF / 2) + i) / KS, ks = (q * (QF / 2) + i) % KS;
                if (ks == 0)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
                const f16x8 qh = as_f16x8(sQO[ks * 64 + lane]), ql = as_f16x8(sQO[(KS + ks) * 64 + lane]);
                const f16x8 kh = as_f16x8(kv[q & 1][2 * i]), kl = as_f16x8(kv[q & 1][2 * i + 1]);
                s[kt] = MFMA16(kl, qh, s[kt]);
                s[kt] = MFMA16(kh, ql, s[kt]);
                s[kt] = MFMA16(kh, qh, s[kt]);
            }
            if (q < 2) fetch(q + 2, Kp);
            else fetch(q - 2, Vp);
        }
        f16x8 ph[4], pl[4];
        softmax_page<DT>(s, t0 + BB_PAGE > L, t0, L, g, m_run, l_run, o, ph, pl);
        // fragment pair (dt, kk) = pair dt 4 + kk of the page
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int i = 0; i < QF / 2; ++i) {
                const int dt = (q * (QF / 2) + i) / 4, kk = (q * (QF / 2) + i) % 4;
                const f16x8 vh = as_f16x8(kv[q & 1][2 * i]), vl = as_f16x8(kv[q & 1][2 * i + 1]);
                o[dt] = MFMA16(vl, ph[kk], o[dt]);
                o[dt] = MFMA16(vh, pl[kk], o[dt]);
                o[dt] = MFMA16(vh, ph[kk], o[dt]);
            }
            if (q < 2) fetch(q + 2, Vp);
            else if (nxt < p1) fetch(q - 2, Kn);
        }
        Kp = Kn;
    }
    __syncthreads();                                // all waves are done with Q
    // per-wave results -> LDS.  o[dt][r] is O^T[d = 32 dt + 8 (r/4) + 4 g + r%4][query c].
    {
        const float l = l_run + __shfl_xor(l_run, 32, 64);
        if (g == 0) { sM[wave][c] = m_run; sL[wave][c] = l; }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) sO[wave][c][32 * dt + 8 * (r >> 2) + 4 * g + (r & 3)] = o[dt][r];
    }
    __syncthreads();
    // a row's results, combined over the waves in a fixed order
    auto combine = [&](int q, float (&wgt)[WAVES], float& M) {
        M = sM[0][q];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) M = fmaxf(M, sM[w][q]);
        float lsum = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            wgt[w] = sM[w][q] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sM[w][q] - M);           // maxima are in the log2 domain
            lsum += wgt[w] * sL[w][q];
        }
        return lsum;
    };
    if (n_splits > 1) {
        // unnormalised partial result of this split: max[32], sum[32], O[32][HD]; attention_combine_kernel finishes
        float* dst = part + ((((size_t)blockIdx.z * gridDim.x + blockIdx.x) * (gridDim.y / n_splits) + qtile) * n_splits + split) * (64 + 32 * HD);
        for (int item = threadIdx.x; item < 32 * (HD / 4); item += THREADS) {
            const int q = item / (HD / 4), d4 = item % (HD / 4);
            float wgt[WAVES], M;
            const float lsum = combine(q, wgt, M);
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                acc.x += wgt[w] * sO[w][q][d4 * 4 + 0]; acc.y += wgt[w] * sO[w][q][d4 * 4 + 1];
                acc.z += wgt[w] * sO[w][q][d4 * 4 + 2]; acc.w += wgt[w] * sO[w][q][d4 * 4 + 3];
            }
            *reinterpret_cast<float4*>(dst + 64 + q * HD + d4 * 4) = acc;
            if (d4 == 0) { dst[q] = M; dst[32 + q] = lsum; }
        }
        return;
    }
    // normalise, split into two terms and store as the O-projection's packed activation panel (row = packed query row,
    // k = head * HD + d); neighbouring lanes take neighbouring rows, which are adjacent there.
    for (int item = threadIdx.x; item < 32 * (HD / 8); item += THREADS) {
        const int q = item & 31, d8 = item >> 5, f = wg_base + q;
        if (f >= nflat) continue;
        float wgt[WAVES], M, y[8];
        const float inv = 1.0f / combine(q, wgt, M);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float acc = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) acc += wgt[w] * sO[w][q][d8 * 8 + e];
            y[e] = acc * inv;
        }
        const int hig = f / seg_rows, r = f % seg_rows;
        store_panel8(Apk, seg_off + r, ((kvh * group + hig) * HD) / 8 + d8, mt_total, y, wide);
    }
}

// Many query rows per segment (full-sequence passes): four waves, 32 query rows each, walk the row's pages together.
// What bounds it: the matrix pipes (96 MFMAs per wave and page at HD = 128, 3072 cycles), beside some 1600 cycles of
// exponentials and conversions and, per CU, the 64 KB of a page.  So a page is fetched once per workgroup into LDS, by
// direct-to-LDS loads (with every wave fetching it for itself, a page step was 256 KB through the CU's load path: 4096 cycles
// and more, the longest of the three), and two workgroups share a CU, so that one's softmax runs beside the other's MFMAs:
// hence 64 KB of LDS each, K and V once, no second buffers.  K of the next page is on its way while V is being used, and V
// while K is:
//   [K landed] barrier | request V | scores | barrier | request next K | softmax | [V landed] barrier | P.V
// Measured, us per launch (heads of 128; before = every wave fetching for itself, one workgroup per CU): 4 x 5120 rows and
// keys, 32 heads 5443 -> 4041 (1.27 PFLOP/s in MFMAs; the pipes alone sustain 1.7 with such MFMAs at the power limit), 4 x 768
// 156 -> 118, 3 x 1402 with 28 query and 4 kv heads 327 -> 240.  (A workgroup alone on its CU is slower so: attention_plan.)
// A higher wave priority around the MFMAs was slower (4222).
template <int HD>
__global__ __launch_bounds__(256, 2) void attention_full_kernel(Dev D, const half_t* __restrict__ Q, u32x4* __restrict__ Apk,
                                                                int layer, int mt_total, int seg_base, int wide) {
    constexpr int KS = HD / 16, DT = HD / 32, NF = 4 * KS;         // k-steps of the scores, output tiles, fragments of a K (or V) page
    constexpr int PAGE_BYTES = NF * 1024, LDO = 64 + 1;            // store slice: 32 rows x 64 dims, odd row stride
    __shared__ __attribute__((aligned(16))) char lds[2 * PAGE_BYTES > 4 * 32 * LDO * 4 ? 2 * PAGE_BYTES : 4 * 32 * LDO * 4];
    const int gbr = seg_base + blockIdx.z, seg_rows = D.seg_rows[gbr];
    if (seg_rows == 0) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 5, c = lane & 31;
    const int group = D.hq / D.hkv, nflat = seg_rows * group, wg_base = blockIdx.y * 128;
    if (wg_base >= nflat) return;
    const int tile_base = wg_base + 32 * wave;      // (waves past the end repeat the last row, take part in the loads and store nothing)
    const int kvh = blockIdx.x, seg_off = D.seg_off[gbr];
    const int L = D.hdr[gbr / D.max_br].L, n_pages = (L + BB_PAGE - 1) / BB_PAGE;
    const unsigned lane16 = lane * 16, lds0 = lds_offset(lds);
    // this wave's quarter of a page: KS fragments in a row
    auto request = [&](const half_t* cache, int phys, int page, int buf) {
        const char* src = reinterpret_cast<const char*>(cache + kv_block_off(D, layer, phys, page, kvh)) + wave * (KS * 1024);
        const unsigned dst = lds0 + buf * PAGE_BYTES + wave * (KS * 1024);
#pragma unroll
        for (int q = 0; q < KS / 4; ++q) {
            load_to_lds<0>(src + q * 4096, lane16, dst + q * 4096);
            load_to_lds<1024>(src + q * 4096, lane16, dst + q * 4096);
            load_to_lds<2048>(src + q * 4096, lane16, dst + q * 4096);
            load_to_lds<3072>(src + q * 4096, lane16, dst + q * 4096);
        }
    };
    // all but the latest `Later` requests of this wave have landed and its LDS reads are done; after the barrier so are the others'
    auto landed = [&](auto Later) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(decltype(Later)::value) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    typedef std::integral_constant<int, 0> None;
    typedef std::integral_constant<int, KS> OnePage;
    u32x4 qf[2][KS];                    // Q fragments as in attention_kernel
    {
        const int f = min(tile_base + c, nflat - 1), hig = f / seg_rows, r = f % seg_rows;
        const half_t* qp = Q + ((size_t)(seg_off + r) * D.hq + kvh * group + hig) * 2 * HD + (HD / 2) * g;
#pragma unroll
        for (int term = 0; term < 2; ++term)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[term][ks] = *reinterpret_cast<const u32x4*>(qp + term * HD + 8 * ks);
    }
    // the page table, 64 entries at a time, one per lane (a load per page would stand in line behind the page's own)
    const int* table = D.table + (size_t)gbr * D.n_pages;
    int entries = table[min(lane, n_pages - 1)], phys = __builtin_amdgcn_readlane(entries, 0);
    request(D.Kc, phys, 0, 0);
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    const u32x4 *kl = reinterpret_cast<const u32x4*>(lds) + lane, *vl = kl + NF * 64;
    for (int page = 0; page < n_pages; ++page) {
        landed(None{});                     // K
        request(D.Vt, phys, page, 1);
        if (((page + 1) & 63) == 0) entries = table[min(page + 1 + lane, n_pages - 1)];
        phys = __builtin_amdgcn_readlane(entries, min(page + 1, n_pages - 1) & 63);
        f32x16 s[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            f16x8 kh[2], klo[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) { kh[kt] = as_f16x8(kl[((kt * KS + ks) * 2) * 64]); klo[kt] = as_f16x8(kl[((kt * KS + ks) * 2 + 1) * 64]); }
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) s[kt] = MFMA16(klo[kt], as_f16x8(qf[0][ks]), s[kt]);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) s[kt] = MFMA16(kh[kt], as_f16x8(qf[1][ks]), s[kt]);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) s[kt] = MFMA16(kh[kt], as_f16x8(qf[0][ks]), s[kt]);
        }
        landed(OnePage{});                  // (V may still be on its way: every wave is done with K)
        request(D.Kc, phys, min(page + 1, n_pages - 1), 0);        // (past the end: the last page again, which nothing reads)
        f16x8 ph[4], pl[4];
        softmax_page<DT>(s, page * BB_PAGE + BB_PAGE > L, page * BB_PAGE, L, g, m_run, l_run, o, ph, pl);
        landed(OnePage{});                  // V
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            f16x8 vh[DT], vlo[DT];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) { vh[dt] = as_f16x8(vl[((dt * 4 + kk) * 2) * 64]); vlo[dt] = as_f16x8(vl[((dt * 4 + kk) * 2 + 1) * 64]); }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = MFMA16(vlo[dt], ph[kk], o[dt]);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = MFMA16(vh[dt], pl[kk], o[dt]);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = MFMA16(vh[dt], ph[kk], o[dt]);
        }
    }
    // Normalise and store as the O-projection's panel (row = packed query row, k = head * HD + d), 64 dims at a time through
    // this wave's slice of LDS.  o[dt][r] is O^T[d = 32 dt + 8 (r/4) + 4 g + r%4][query c]; a lane then takes 8 dims of one
    // row, neighbouring lanes neighbouring rows, which are adjacent in the panel.
    const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32, 64));
    landed(None{});                                         // all waves are done with V, and no request is on its way
    float* so = reinterpret_cast<float*>(lds) + wave * (32 * LDO);
    const int f = tile_base + c, hig = min(f, nflat - 1) / seg_rows, m = seg_off + min(f, nflat - 1) % seg_rows;
#pragma unroll
    for (int half = 0; half < DT / 2; ++half) {
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) so[c * LDO + 32 * dt + 8 * (r >> 2) + 4 * g + (r & 3)] = o[2 * half + dt][r] * inv;
        wave_lds_order();                                   // (the same wave wrote and reads: no barrier needed)
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int d8 = 2 * it + g;
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = so[c * LDO + d8 * 8 + e];
            if (f < nflat) store_panel8(Apk, m, ((kvh * group + hig) * HD + 64 * half) / 8 + d8, mt_total, y, wide);
        }
        wave_lds_order();                                   // (the next half overwrites the slice)
    }
}

// Merge the splits of one tile in split order, normalise, and store the packed hi/lo panel.
template <int HD>
__global__ __launch_bounds__(256) void attention_combine_kernel(Dev D, const float* __restrict__ part, u32x4* __restrict__ Apk,
                                                                int mt_total, int seg_base, int n_splits, int wide) {
    const int gbr = seg_base + blockIdx.z;
    const int seg_rows = D.seg_rows[gbr], seg_off = D.seg_off[gbr];
    const int group = D.hq / D.hkv, nflat = seg_rows * group, wg_base = blockIdx.y * 32, kvh = blockIdx.x;
    if (wg_base >= nflat) return;
    const float* src = part + (((size_t)blockIdx.z * gridDim.x + blockIdx.x) * gridDim.y + blockIdx.y) * n_splits * (64 + 32 * HD);
    // The loads of four splits are on their way together.  us per launch: 32 tiles in three splits 6.4 -> 4.8, 100 in two
    // 5.6 -> 5.0.  (None before the segment's size is known: the grid has a place for every tile of every slot of the context, and
    // reading those of 255 empty segments, 32 tiles in three splits each, took 64 us.)
    for (int item = threadIdx.x; item < 32 * (HD / 8); item += 256) {
        const int q = item / (HD / 8), d8 = item % (HD / 8), f = wg_base + q;
        if (f >= nflat) break;          // (items go through the tile's rows in order)
        float M = -INFINITY, lsum = 0.f, y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < n_splits; s0 += 4) {
            float m[4], l[4];
            float4 a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float* ps = src + min(s0 + u, n_splits - 1) * (64 + 32 * HD);
                m[u] = ps[q]; l[u] = ps[32 + q];
                a[u] = *reinterpret_cast<const float4*>(ps + 64 + q * HD + d8 * 8);
                b[u] = *reinterpret_cast<const float4*>(ps + 64 + q * HD + d8 * 8 + 4);
            }
            if (s0 == 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) M = fmaxf(M, m[u]);
                for (int s = 4; s < n_splits; ++s) M = fmaxf(M, src[s * (64 + 32 * HD) + q]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (s0 + u >= n_splits) break;
                const float wgt = m[u] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[u] - M);
                lsum += wgt * l[u];
                y[0] += wgt * a[u].x; y[1] += wgt * a[u].y; y[2] += wgt * a[u].z; y[3] += wgt * a[u].w;
                y[4] += wgt * b[u].x; y[5] += wgt * b[u].y; y[6] += wgt * b[u].z; y[7] += wgt * b[u].w;
            }
        }
        const float inv = 1.0f / lsum;
        const int hig = f / seg_rows, r = f % seg_rows;
        const int m = seg_off + r, k8 = ((kvh * group + hig) * HD) / 8 + d8;
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] *= inv;
        store_panel8(Apk, m, k8, mt_total, y, wide);
    }
}

AttentionPlan attention_plan(const Dev& D, int max_seg_rows, int n_segs, int max_pages, int seg_tiles, size_t part_elems) {
    const int nflat = max_seg_rows * (D.hq / D.hkv);
    // Many query rows per segment: the waves of a workgroup take different tiles and share each page.  Only where these workgroups
    // outnumber the CUs: one alone on its CU has nothing to run at its three barriers per page, while a workgroup per tile, its
    // waves on different pages, has four times the workgroups and walks a quarter (or an eighth) of the pages.  us per launch,
    // this kernel / a workgroup per tile, by 128-row workgroups: heads of 64: 64 (4096 keys, 4 heads: 128) 129 / 64, 256 (32 pages)
    // 75 / 68, 288 (47 pages) 119 / 112, 376 141 / 147, 512 205 / 250; heads of 128: 128 32 / 22, 168 44 / 37, 192 46 / 39, 224 57 /
    // 60, 256 63 / 65, 352 115 / 141, 512 189 / 257.
    if (nflat >= 512 && seg_tiles * D.hkv > 4 * (D.hd == 64 ? 256 : 192)) return {0, 1};
    // Otherwise a workgroup per tile, of four waves (two workgroups to a CU) up to 16 pages, of eight above: with one
    // workgroup per CU four waves leave the CU's loads idle (80 pages, 256 tiles: 236 us against 149; 24 pages, 200
    // workgroups: 27.5 against 19.8), with few pages eight have too little each (12 pages, 320 tiles: 44.9 us against 43.3).
    // Where the tiles leave CUs idle the pages of a row are split over several workgroups and a second kernel merges the
    // partial results: worth it once the share of a CU's own stream that it saves (about 50 KB per us) exceeds that launch, its
    // place in the stream and the store of the partial results (100 tiles, 24 pages: 31.0 us unsplit, 20.1 + 5.0 in two; the launch
    // alone takes 4.8 to 5.0, and 7.0 dates from when it took 5.6 to 6.4: lower values are not measured).
    const int qtiles = (nflat + 31) / 32, tiles = qtiles * D.hkv * n_segs, wgs = std::max(1, seg_tiles * D.hkv), waves = max_pages > 16 ? 8 : 4;
    const double stream_us = max_pages * (D.hd * 512.0) / 50e3, combine_us = 7.0;
    int n_splits = std::min(std::min(256 / wgs, (max_pages + waves - 1) / waves), 16);
    while (n_splits > 1 && (size_t)tiles * n_splits * (64 + 32 * D.hd) > part_elems) --n_splits;
    if (n_splits < 1 || stream_us - stream_us / n_splits < combine_us) n_splits = 1;
    return {waves, n_splits};
}

void launch_attention(const Dev& D, const half_t* Q, u32x4* Apk, int layer, int mt_total, int max_seg_rows,
                      int seg_base, int n_segs, int max_pages, int seg_tiles, float* part, size_t part_elems, int wide, hipStream_t s) {
    const int nflat = max_seg_rows * (D.hq / D.hkv), qtiles = (nflat + 31) / 32;
    const AttentionPlan p = attention_plan(D, max_seg_rows, n_segs, max_pages, seg_tiles, part_elems);
    const int n_splits = p.n_splits;
    if (p.waves == 0) {
        dim3 grid(D.hkv, (nflat + 127) / 128, n_segs);
        if (D.hd == 128) attention_full_kernel<128><<<grid, 256, 0, s>>>(D, Q, Apk, layer, mt_total, seg_base, wide);
        else attention_full_kernel<64><<<grid, 256, 0, s>>>(D, Q, Apk, layer, mt_total, seg_base, wide);
        return;
    }
    dim3 grid(D.hkv, qtiles * n_splits, n_segs), cgrid(D.hkv, qtiles, n_segs);
#define ATT(HD_) do { \
        if (p.waves == 8) attention_kernel<HD_, 8><<<grid, 512, 0, s>>>(D, Q, Apk, layer, mt_total, seg_base, n_splits, part, wide); \
        else attention_kernel<HD_, 4><<<grid, 256, 0, s>>>(D, Q, Apk, layer, mt_total, seg_base, n_splits, part, wide); \
        if (n_splits > 1) attention_combine_kernel<HD_><<<cgrid, 256, 0, s>>>(D, part, Apk, mt_total, seg_base, n_splits, wide); \
    } while (0)
    if (D.hd == 128) ATT(128);
    else ATT(64);
#undef ATT
}
