// What the block-scaled GEMM kernels share: vector types, direct global->LDS copies and their waits, BF16 rounding.
#pragma once
#include "moss_internal.h"

namespace moss {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// wave-wide direct global->LDS copy: every lane moves 16 bytes from base + off to
// lds_addr + 16 * lane (lds_addr is wave-uniform and goes through M0)
__device__ __forceinline__ void dma16(const uint8_t *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// the same to lds_addr + at, which is added in the move to M0 (`at` is a constant once loops are unrolled)
__device__ __forceinline__ void dma16_at(const uint8_t *base, uint32_t off, uint32_t lds_addr, int at)
{
    asm volatile("s_add_u32 m0, %2, %3\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(lds_addr), "i"(at) : "memory", "m0", "scc");
}

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

__device__ __forceinline__ void wait_lds_and_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two FP32 -> two BF16 (round to nearest even), a in the low half: one V_CVT_PK_BF16_F32
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// The block-scaled matrix instruction as volatile inline assembly: volatile asm statements keep
// their program order, which is what pins "one matrix instruction, one LDS read, one global->LDS
// copy" in the main loop (compiler scheduling hints did not survive: all 16 matrix instructions
// of a substep were emitted first and the memory instructions after them in one burst).
// SEL = 0 / 2 picks scale byte 0 / 2 of both scale registers.  Independent accumulators back to
// back need no wait states; the places where results are consumed add their own (see callers).
template <int SEL>
__device__ __forceinline__ void mfma_scaled(v16f &acc, const v8i &x, const v8i &y, int sx, int sy)
{
    if (SEL == 0)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0]"
                     : "+a"(acc) : "v"(x), "v"(y), "v"(sx), "v"(sy));
    else
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[1,1,0]"
                     : "+a"(acc) : "v"(x), "v"(y), "v"(sx), "v"(sy));
}
__device__ __forceinline__ void pin() { asm volatile("" ::: "memory"); }

}  // namespace moss
