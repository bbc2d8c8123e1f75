// Unrolling and schedule groups of the software-pipelined GEMM loops.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

// f(0), ..., f(N - 1) with the index as a constant of its own type
#define IC(v) std::integral_constant<int, (v)>{}
template <int N, int I = 0, class F> static __device__ __forceinline__ void unroll(F&& f) {
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); unroll<N, I + 1>(f); }
}

// sched_group_barrier masks
#define SG_MFMA 0x008
#define SG_VMEM 0x020
#define SG_DSR 0x100
#define SG_DSW 0x200
// One scheduling group per m-tile of a phase: NT MFMAs, then this group's share of the phase's LDS reads, LDS writes
// and global loads (dealt out as evenly as possible, larger shares first).  The builtin wants constants, hence
// templates.
template <int MASK, int N> static __device__ __forceinline__ void sgb() {
    if constexpr (N > 0) __builtin_amdgcn_sched_group_barrier(MASK, N, 0);
}
template <int GROUPS, int TOTAL, int I> constexpr int sg_share() { return TOTAL / GROUPS + (I < TOTAL % GROUPS ? 1 : 0); }
template <int GROUPS, int NT, int DSR_TOTAL, int DSW_TOTAL, int VMEM_TOTAL, int I = 0>
static __device__ __forceinline__ void sched_groups() {
    if constexpr (I < GROUPS) {
        sgb<SG_MFMA, NT>();
        sgb<SG_DSR, sg_share<GROUPS, DSR_TOTAL, I>()>();
        sgb<SG_DSW, sg_share<GROUPS, DSW_TOTAL, I>()>();
        sgb<SG_VMEM, sg_share<GROUPS, VMEM_TOTAL, I>()>();
        sched_groups<GROUPS, NT, DSR_TOTAL, DSW_TOTAL, VMEM_TOTAL, I + 1>();
    }
}
