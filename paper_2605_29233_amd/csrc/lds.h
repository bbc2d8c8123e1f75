// Direct-to-LDS loads.
#pragma once
#include <hip/hip_runtime.h>

// One 1 KiB fragment (64 lanes x 16 bytes) from src to the LDS byte offset dst without passing through registers; OFF is
// added on both sides.  Written as assembly because the compiler, where it knows of such loads, lets every LDS read
// wait for all outstanding ones: the waits for these loads are the explicit ones at the barriers.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF> static __device__ __forceinline__ void load_to_lds(const char* src, unsigned lane16, unsigned dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                 ::"s"(dst), "v"(lane16), "s"(src), "n"(OFF) : "m0", "memory");
}
// The same by the first N waves only (a branch inside the assembly: one in the loop body would split the pipeline's block).
template <int N> static __device__ __forceinline__ void load_to_lds_first(int wave, const char* src, unsigned lane16, unsigned dst) {
    asm volatile("s_cmp_ge_u32 %3, %4\n\ts_cbranch_scc1 1f\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n1:"
                 ::"s"(dst), "v"(lane16), "s"(src), "s"(wave), "n"(N) : "m0", "scc", "memory");
}
#pragma clang diagnostic pop
static __device__ __forceinline__ unsigned lds_offset(const void* p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) const void*)p;
}
