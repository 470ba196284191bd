// What the block-scaled GEMM kernels share: vector types, direct global->LDS copies and their waits, BF16 rounding.
#pragma once
#include "moss_internal.h"

namespace moss {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// wave-wide direct global->LDS copy: every lane moves 16 bytes from base + off to
// lds_addr + 16 * lane (lds_addr is wave-uniform and goes through M0).  A copy into LDS that follows a scalar write of M0 needs
// one wait state in between, or it may go where M0 pointed before; the compiler, which puts it there itself elsewhere, does not
// look into an asm block.
__device__ __forceinline__ void dma16(const uint8_t *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// the same to lds_addr + at, which is added in the move to M0 (`at` is a constant once loops are unrolled)
__device__ __forceinline__ void dma16_at(const uint8_t *base, uint32_t off, uint32_t lds_addr, int at)
{
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
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

// Stores a 32 x 32 fragment of accumulators times `scale` without staging it.  Register v of lane (i32, h) is row i32, column
// 8 (v / 4) + 4 h + v % 4: four columns in a row, so that an FP32 output leaves in 16-byte pieces, 32 bytes of a row per
// instruction.  For BF16 the halves of the wave exchange every other group of four first and hold eight columns each.  The pieces
// of a line meet in the L2.  (2048 x 2048 x 512 in 128 x 128 tiles: 2.5 us to stage the
// tile in LDS and walk it and 2.0 to store it, 2.6 together this way, 10.7 -> 8.8; accumulating 17.3 -> 14.6.)  `row` is this lane's, `n` the fragment's first column.
__device__ __forceinline__ void store_fragment(const v16f &acc, float scale, void *out, int64_t ld, int64_t row, int64_t n, int h,
                                               int64_t M, int64_t N, int out_f32, int accumulate)
{
    float r[16];
#pragma unroll
    for (int v = 0; v < 16; v++) r[v] = acc[v] * scale;
    if (out_f32) {
        float *o = reinterpret_cast<float *>(out) + row * ld + n + 4 * h;
        if (n + 32 <= N && ld % 4 == 0) {            // (wave-uniform)
            if (row >= M) return;
            if (accumulate) {
                float4 q[4];
#pragma unroll
                for (int g = 0; g < 4; g++) q[g] = *reinterpret_cast<const float4 *>(o + 8 * g);
#pragma unroll
                for (int g = 0; g < 4; g++)
                    *reinterpret_cast<float4 *>(o + 8 * g) = make_float4(r[4 * g] + q[g].x, r[4 * g + 1] + q[g].y, r[4 * g + 2] + q[g].z, r[4 * g + 3] + q[g].w);
            } else {
#pragma unroll
                for (int g = 0; g < 4; g++) *reinterpret_cast<float4 *>(o + 8 * g) = make_float4(r[4 * g], r[4 * g + 1], r[4 * g + 2], r[4 * g + 3]);
            }
        } else if (row < M) {
            // the matrix ends inside the fragment, or its rows are not 16-byte aligned
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int64_t left = N - (n + 4 * h + 8 * g);
                if (left >= 4 && ld % 4 == 0) {
                    float4 v = make_float4(r[4 * g], r[4 * g + 1], r[4 * g + 2], r[4 * g + 3]);
                    if (accumulate) {
                        const float4 q = *reinterpret_cast<const float4 *>(o + 8 * g);
                        v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
                    }
                    *reinterpret_cast<float4 *>(o + 8 * g) = v;
                } else {
#pragma unroll
                    for (int x = 0; x < 4; x++)
                        if (x < left) o[8 * g + x] = accumulate ? r[4 * g + x] + o[8 * g + x] : r[4 * g + x];
                }
            }
        }
        return;
    }
    uint32_t w[8];
#pragma unroll
    for (int v = 0; v < 8; v++) w[v] = pack_bf16(r[2 * v], r[2 * v + 1]);
    uint16_t *o = reinterpret_cast<uint16_t *>(out) + row * ld + n;
    if (n + 32 <= N && ld % 8 == 0) {                // (wave-uniform)
#pragma unroll
        for (int g = 0; g < 2; g++) {
            // words 4 g .. : columns 16 g + 4 h + 0 .. 3 in the first two, 16 g + 8 + 4 h in the others
#pragma unroll
            for (int k = 0; k < 2; k++) {
                const auto both = __builtin_amdgcn_permlane32_swap(w[4 * g + k], w[4 * g + 2 + k], false, false);
                w[4 * g + k] = both[0];
                w[4 * g + 2 + k] = both[1];
            }
            if (row < M) *reinterpret_cast<uint4 *>(o + 16 * g + 8 * h) = make_uint4(w[4 * g], w[4 * g + 1], w[4 * g + 2], w[4 * g + 3]);
        }
    } else if (row < M) {
        // the matrix ends inside the fragment, or its rows are not 16-byte aligned
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const int at = 8 * g + 4 * h;
            const int64_t left = N - (n + at);
            if (left >= 4 && ld % 4 == 0) {
                *reinterpret_cast<uint2 *>(o + at) = make_uint2(w[2 * g], w[2 * g + 1]);
            } else {
#pragma unroll
                for (int x = 0; x < 4; x++)
                    if (x < left) o[at + x] = (uint16_t)(w[2 * g + x / 2] >> (16 * (x & 1)));
            }
        }
    }
}

}  // namespace moss
