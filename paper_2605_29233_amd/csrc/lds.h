// Direct-to-LDS loads, and the order of a wave's own LDS accesses.
#pragma once
#include <hip/hip_runtime.h>

// One 1 KiB fragment (64 lanes x 16 bytes) from src to the LDS byte offset dst without passing through registers; OFF is
// added on both sides.  Written as assembly because the compiler, where it knows of such loads, lets every LDS read
// wait for all outstanding ones: the waits for these loads are the explicit ones at the barriers.
// (The compiler warns that m0 is one of its own registers.  That is why it is told: what it keeps there is overwritten.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF> static __device__ __forceinline__ void load_to_lds(const char* src, unsigned lane16, unsigned dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                 ::"s"(dst), "v"(lane16), "s"(src), "n"(OFF) : "m0", "memory");
}
// The same if i < n only (a branch inside the assembly: one in the loop body would split the pipeline's block).
static __device__ __forceinline__ void load_to_lds_below(unsigned i, unsigned n, const char* src, unsigned lane16, unsigned dst) {
    asm volatile("s_cmp_ge_u32 %3, %4\n\ts_cbranch_scc1 1f\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n1:"
                 ::"s"(dst), "v"(lane16), "s"(src), "s"(i), "s"(n) : "m0", "scc", "memory");
}
#pragma clang diagnostic pop
// Between the stores and the loads by which the lanes of one wave exchange data through a slice of LDS that is theirs.  The
// LDS unit takes a wave's instructions in order, but seen per thread the addresses differ, so without this the compiler may
// move a load before the store of the lane it reads from.  Costs no instruction.
static __device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
static __device__ __forceinline__ unsigned lds_offset(const void* p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) const void*)p;
}
