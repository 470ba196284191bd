// SwiGLU forward and backward in BF16, each output with the maximum of its magnitudes: the producer
// in front of the quantizer of the down projection (forward) and of the gate / up projections' dY
// (backward).  The paper keeps the non-linear layers in BF16 (Sec. 4.1); what this adds is the tensor
// maximum of Sec. 3.1, Eq. 2 as a by-product of writing the tensor, so that the quantizer of these
// tensors (172 MiB each at LLaMA-7B sizes and 8192 tokens: too large to be kept on chip between a
// search for the maximum and the conversion) reads them once.
//
// Bound: HBM (2 or 3 BF16 tensors in, 1 or 2 out).  Every thread handles 16-byte chunks of eight
// elements; arithmetic in FP32 with the hardware's exp2 and reciprocal approximations (1 ulp each),
// one rounding to BF16 (round to nearest even) by V_CVT_PK_BF16_F32.  The maximum is taken over the
// bit patterns actually written (unsigned maximum of the 15 magnitude bits), folded per wave and per
// workgroup, and either left in slots that the last workgroup folds into the caller's word, or merged into it by
// one atomic per workgroup behind a one-thread kernel that clears it (callers without a workspace, captured
// calls; no memset, so the call can be captured into a graph).
#include "moss_internal.h"
#include "moss_producer.h"

namespace moss {
namespace {

constexpr int kSwThreads = 256;
typedef unsigned short sw_u16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 sw_bf16x2 __attribute__((ext_vector_type(2)));
typedef float sw_f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t sw_pk_max_u16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(sw_u16x2, a), __builtin_bit_cast(sw_u16x2, b)));
}
// two FP32 -> two BF16 (round to nearest even), a in the low half
__device__ __forceinline__ uint32_t sw_pack(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(sw_f32x2{a, b}, sw_bf16x2));
}
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// sig(g) = 1 / (1 + exp(-g)); exp(-g) = 2^(-g log2 e) overflows to +inf for g < -88.7, which gives 0
__device__ __forceinline__ float sigmoid(float g)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.44269504088896340736f));
}

__device__ __forceinline__ void fold_max(uint32_t m, uint32_t *word, int look, uint32_t *red)
{
    m = (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16);
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t seen = look_at_word(word, look);
        for (int i = 1; i < kSwThreads / kWave; i++) m = red[i] > m ? red[i] : m;
        merge_max_word(word, m, seen);
    }
    __syncthreads();
}

// maximum of the workgroup in thread 0 (red: a word per wave)
__device__ __forceinline__ uint32_t block_max(uint32_t m, uint32_t *red)
{
    m = (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16);
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < kSwThreads / kWave; i++) m = red[i] > m ? red[i] : m;
    return m;
}

__global__ void k_swiglu_clear(uint32_t *a, uint32_t *b)
{
    if (threadIdx.x == 0) {
        *a = 0;
        if (b) *b = 0;
    }
}

__device__ __forceinline__ int64_t chunk_offset(int64_t id, int chunks_per_row, int64_t ld, int dense)
{
    if (dense) return id * 8;
    const int64_t row = id / chunks_per_row;
    return row * ld + (id - row * chunks_per_row) * 8;
}

// CHUNKS: 16-byte chunks of every input per thread whose loads are on the way together (chunks_per_thread has the rule)
template <int CHUNKS>
__global__ __launch_bounds__(kSwThreads) void k_swiglu(const uint16_t *__restrict__ gate, const uint16_t *__restrict__ up,
                                                       int64_t n_chunks, int chunks_per_row, int64_t ld, int dense, int flags,
                                                       uint16_t *__restrict__ h, uint32_t *__restrict__ h_max, MaxSlots slots)
{
    __shared__ uint32_t red[kSwThreads / kWave];
    uint32_t m = 0;
    asm volatile("" ::"s"(slots.words), "s"(slots.call), "s"(slots.looks));      // (fetched here, not at the end in front of the slots)
    const int64_t stride = (int64_t)gridDim.x * kSwThreads * CHUNKS;
    for (int64_t id0 = (int64_t)blockIdx.x * kSwThreads * CHUNKS + threadIdx.x; id0 < n_chunks; id0 += stride) {
        uint4 g[CHUNKS], u[CHUNKS];
        int64_t off[CHUNKS];
#pragma unroll
        for (int k = 0; k < CHUNKS; k++) {
            const int64_t id = id0 + (int64_t)k * kSwThreads;
            off[k] = -1;
            if (id < n_chunks) {
                off[k] = chunk_offset(id, chunks_per_row, ld, dense);
                g[k] = ld_stream16(gate + off[k]);
                u[k] = ld_stream16(up + off[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < CHUNKS; k++) {
            if (off[k] < 0) continue;
            const uint32_t gw[4] = {g[k].x, g[k].y, g[k].z, g[k].w}, uw[4] = {u[k].x, u[k].y, u[k].z, u[k].w};
            uint32_t o[4];
#pragma unroll
            for (int w = 0; w < 4; w++) {
                const float g0 = lo_f32(gw[w]), g1 = hi_f32(gw[w]);
                o[w] = sw_pack((g0 * sigmoid(g0)) * lo_f32(uw[w]), (g1 * sigmoid(g1)) * hi_f32(uw[w]));
                m = sw_pk_max_u16(m, o[w] & 0x7FFF7FFFu);
            }
            st_producer16(h + off[k], make_uint4(o[0], o[1], o[2], o[3]), flags & kProducerStream);
        }
    }
    if (slots.call) {
        const uint32_t top[1] = {block_max(m, red)};
        uint32_t *const out[1] = {h_max};
        finish_max_in_slots<1, kSwThreads>(slots, top, out, red);
    } else {
        fold_max(m, h_max, flags & kProducerLook, red);
    }
}

template <int CHUNKS>
__global__ __launch_bounds__(kSwThreads) void k_swiglu_backward(const uint16_t *__restrict__ gate, const uint16_t *__restrict__ up,
                                                                const uint16_t *__restrict__ dh, int64_t n_chunks,
                                                                int chunks_per_row, int64_t ld, int dense, int flags,
                                                                uint16_t *__restrict__ d_gate, uint16_t *__restrict__ d_up,
                                                                uint32_t *__restrict__ dg_max, uint32_t *__restrict__ du_max,
                                                                MaxSlots slots)
{
    __shared__ uint32_t red[kSwThreads / kWave], red_u[kSwThreads / kWave], red_all[2 * kSwThreads / kWave];
    uint32_t mg = 0, mu = 0;
    asm volatile("" ::"s"(slots.words), "s"(slots.call), "s"(slots.looks));      // (fetched here, not at the end in front of the slots)
    const int64_t stride = (int64_t)gridDim.x * kSwThreads * CHUNKS;
    for (int64_t id0 = (int64_t)blockIdx.x * kSwThreads * CHUNKS + threadIdx.x; id0 < n_chunks; id0 += stride) {
        uint4 gc[CHUNKS], uc[CHUNKS], dc[CHUNKS];
        int64_t offs[CHUNKS];
#pragma unroll
        for (int k = 0; k < CHUNKS; k++) {
            const int64_t id = id0 + (int64_t)k * kSwThreads;
            offs[k] = -1;
            if (id < n_chunks) {
                offs[k] = chunk_offset(id, chunks_per_row, ld, dense);
                gc[k] = ld_stream16(gate + offs[k]);
                uc[k] = ld_stream16(up + offs[k]);
                dc[k] = ld_stream16(dh + offs[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < CHUNKS; k++) {
            const int64_t off = offs[k];
            if (off < 0) continue;
            const uint4 &g = gc[k], &u = uc[k], &d = dc[k];
            const uint32_t gw[4] = {g.x, g.y, g.z, g.w}, uw[4] = {u.x, u.y, u.z, u.w}, dw[4] = {d.x, d.y, d.z, d.w};
            uint32_t og[4], ou[4];
#pragma unroll
            for (int w = 0; w < 4; w++) {
                float rg[2], ru[2];
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    const float gv = e ? hi_f32(gw[w]) : lo_f32(gw[w]), uv = e ? hi_f32(uw[w]) : lo_f32(uw[w]);
                    const float dv = e ? hi_f32(dw[w]) : lo_f32(dw[w]);
                    const float sg = sigmoid(gv);
                    ru[e] = dv * (gv * sg);
                    rg[e] = (dv * uv) * (sg * (1.0f + gv * (1.0f - sg)));
                }
                og[w] = sw_pack(rg[0], rg[1]);
                ou[w] = sw_pack(ru[0], ru[1]);
                mg = sw_pk_max_u16(mg, og[w] & 0x7FFF7FFFu);
                mu = sw_pk_max_u16(mu, ou[w] & 0x7FFF7FFFu);
            }
            st_producer16(d_gate + off, make_uint4(og[0], og[1], og[2], og[3]), flags & kProducerStream);
            st_producer16(d_up + off, make_uint4(ou[0], ou[1], ou[2], ou[3]), flags & kProducerStream);
        }
    }
    if (slots.call) {
        const uint32_t top[2] = {block_max(mg, red), block_max(mu, red_u)};
        uint32_t *const out[2] = {dg_max, du_max};
        finish_max_in_slots<2, kSwThreads>(slots, top, out, red_all);
    } else {
        fold_max(mg, dg_max, flags & kProducerLook, red);
        fold_max(mu, du_max, flags & kProducerLook, red);
    }
}

int check_common(int64_t rows, int64_t cols, int64_t ld)
{
    if (rows <= 0 || cols <= 0 || cols % 8 || ld < cols) return MOSS_ERR_SHAPE;
    if (rows * (cols / 8) >= ((int64_t)1 << 40)) return MOSS_ERR_SHAPE;
    if (ld % 8) return MOSS_ERR_ALIGN;
    return MOSS_OK;
}

// Chunks per thread.  One leaves too little in flight where the memory's rate counts, four leave small tensors to few
// workgroups that each work through four chunks in a row.  Forward / backward alone, us, with 1, 2 and 4:
//   chunks   2^10 (128 x 64)    4.6  5.0  5.6   and   5.1  5.6  6.5
//            2^13               4.9  5.0  5.8         5.6  5.7  6.7
//            2^14 (512 x 256)   5.5  5.2  5.8         6.2  5.9  6.8
//            2^15               6.2  5.6  5.9         8.4  6.9  7.0
//            2^16 (512 x 1024)  8.9  7.0  6.6        13.2  9.5  8.4
//            2^18              19.9 12.8 10.1        34.5 21.1 15.0
// (1024 x 11008 forward + backward + three quantizers 142 us with 2 forward and 1 backward, 103 with 4 and 4; at the memory's
// rate, 4096 x 11008, 278 either way.)
int chunks_per_thread(int64_t n_chunks) { return n_chunks < (1 << 14) ? 1 : n_chunks < (1 << 16) ? 2 : 4; }

int grid_for(int64_t n_chunks)
{
    const int per_thread = chunks_per_thread(n_chunks);
    const int64_t want = (n_chunks + (int64_t)kSwThreads * per_thread - 1) / ((int64_t)kSwThreads * per_thread);
    int cus = moss_internal_cu_count();
    if (cus <= 0) cus = 256;
    // Eight workgroups per compute unit, grid-stride beyond, as many as have slots for their maxima (kMaxSlotBlocks).  Forward and backward
    // with the quantizers, us, 4 and 8: 1024 x 11008 86 and 87, 2048 x 11008 138 both, 4096 x 11008 253 and 254; merged into the caller's
    // words, 4 / 8 / 16: 2048 x 11008 143 / 144 / 163, 4096 x 11008 259 each.
    const int64_t cap = (int64_t)cus * 8;
    return (int)(want < cap ? want : cap);
}

// Look at the word before merging into it (merge_max_word) from 384 workgroups on.  Forward / backward (two words) alone, us,
// without and with the look, by the number of workgroups:
//     1 .. 63     5.2 / 6.0 and 5.4 / 6.6      64 .. 255   7.2 / 8.1 and 9.2 / 10.7
//   260           9.1 / 11.1 and 13.4 / 14.7     383      10.7 / 11.8 and 15.9 / 15.8
//   420          11.2 / 11.6 and 16.9 / 15.5     500      12.4 / 11.4 and 19.3 / 13.6
//   512 .. 1023  15.6 / 13.8 and 27.6 / 20.9     2048     41.4 / 34.9 and 80.3 / 61.6
// and with the quantizers behind, on inputs that no cache holds: 256 workgroups (1024 x 2048) 51.0 / 51.8, 344 (256 x 11008)
// 51.7 / 52.3, 512 (2048 x 2048) 64.1 / 60.0, 1024 (4096 x 2048) 88.9 / 74.4.
bool looks(int grid) { return grid >= 384; }

}  // namespace
}  // namespace moss

// what the two entry points below choose for a tensor (the tests hold the rules by it)
extern "C" int moss_internal_swiglu_looks(int64_t rows, int64_t cols) { return moss::looks(moss::grid_for(rows * (cols / 8))); }
extern "C" int moss_internal_swiglu_chunks(int64_t rows, int64_t cols) { return moss::chunks_per_thread(rows * (cols / 8)); }

extern "C" int moss_swiglu_bf16(const void *gate, const void *up, int64_t rows, int64_t cols, int64_t ld,
                                void *h, uint32_t *h_absmax_bits, void *stream)
{
    return moss_internal_swiglu_bf16(gate, up, rows, cols, ld, h, h_absmax_bits, nullptr, 0, stream);
}

extern "C" int moss_internal_swiglu_bf16(const void *gate, const void *up, int64_t rows, int64_t cols, int64_t ld, void *h,
                                         uint32_t *h_absmax_bits, void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace moss;
    if (!gate || !up || !h || !h_absmax_bits) return MOSS_ERR_NULL;
    int rc = check_common(rows, cols, ld);
    if (rc) return rc;
    if (!moss_aligned16(gate) || !moss_aligned16(up) || !moss_aligned16(h) || ((uintptr_t)h_absmax_bits & 3)) return MOSS_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const int chunks_per_row = (int)(cols / 8);
    const int64_t n_chunks = rows * chunks_per_row;
    const int grid = grid_for(n_chunks), per_thread = chunks_per_thread(n_chunks);
    const MaxSlots slots = max_slots(workspace, workspace_bytes, grid, 1, st);
    if (!slots.call) {
        hipLaunchKernelGGL(k_swiglu_clear, dim3(1), dim3(64), 0, st, h_absmax_bits, (uint32_t *)nullptr);
        MOSS_LAUNCH_CHECK();
    }
    const auto kern = per_thread == 1 ? k_swiglu<1> : per_thread == 2 ? k_swiglu<2> : k_swiglu<4>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kSwThreads), 0, st, (const uint16_t *)gate, (const uint16_t *)up, n_chunks,
                       chunks_per_row, ld, (int)(ld == cols), producer_flags(rows, cols, looks(grid)),
                       (uint16_t *)h, h_absmax_bits, slots);
    MOSS_LAUNCH_CHECK();
    return MOSS_OK;
}

extern "C" int moss_swiglu_bf16_backward(const void *gate, const void *up, const void *dh, int64_t rows, int64_t cols,
                                         int64_t ld, void *d_gate, void *d_up, uint32_t *d_gate_absmax_bits,
                                         uint32_t *d_up_absmax_bits, void *stream)
{
    return moss_internal_swiglu_bf16_backward(gate, up, dh, rows, cols, ld, d_gate, d_up, d_gate_absmax_bits, d_up_absmax_bits, nullptr, 0,
                                              stream);
}

extern "C" int moss_internal_swiglu_bf16_backward(const void *gate, const void *up, const void *dh, int64_t rows, int64_t cols,
                                                  int64_t ld, void *d_gate, void *d_up, uint32_t *d_gate_absmax_bits,
                                                  uint32_t *d_up_absmax_bits, void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace moss;
    if (!gate || !up || !dh || !d_gate || !d_up || !d_gate_absmax_bits || !d_up_absmax_bits) return MOSS_ERR_NULL;
    int rc = check_common(rows, cols, ld);
    if (rc) return rc;
    if (!moss_aligned16(gate) || !moss_aligned16(up) || !moss_aligned16(dh) || !moss_aligned16(d_gate) || !moss_aligned16(d_up))
        return MOSS_ERR_ALIGN;
    if (((uintptr_t)d_gate_absmax_bits & 3) || ((uintptr_t)d_up_absmax_bits & 3)) return MOSS_ERR_ALIGN;
    if (d_gate_absmax_bits == d_up_absmax_bits) return MOSS_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    const int chunks_per_row = (int)(cols / 8);
    const int64_t n_chunks = rows * chunks_per_row;
    const int grid = grid_for(n_chunks), per_thread = chunks_per_thread(n_chunks);
    const MaxSlots slots = max_slots(workspace, workspace_bytes, grid, 2, st);
    if (!slots.call) {
        hipLaunchKernelGGL(k_swiglu_clear, dim3(1), dim3(64), 0, st, d_gate_absmax_bits, d_up_absmax_bits);
        MOSS_LAUNCH_CHECK();
    }
    const auto kern = per_thread == 1 ? k_swiglu_backward<1> : per_thread == 2 ? k_swiglu_backward<2> : k_swiglu_backward<4>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kSwThreads), 0, st, (const uint16_t *)gate, (const uint16_t *)up,
                       (const uint16_t *)dh, n_chunks, chunks_per_row, ld, (int)(ld == cols),
                       producer_flags(rows, cols, looks(grid)), (uint16_t *)d_gate, (uint16_t *)d_up,
                       d_gate_absmax_bits, d_up_absmax_bits, slots);
    MOSS_LAUNCH_CHECK();
    return MOSS_OK;
}
