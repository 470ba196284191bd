// Internal helpers shared by the HIP translation units of libmoss_hip.so (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "moss.h"

#define MOSS_HIP_TRY(expr)                       \
    do {                                         \
        if ((expr) != hipSuccess) {              \
            (void)hipGetLastError();             \
            return MOSS_ERR_HIP;                 \
        }                                        \
    } while (0)

#define MOSS_LAUNCH_CHECK()                      \
    do {                                         \
        if (hipGetLastError() != hipSuccess) return MOSS_ERR_HIP; \
    } while (0)

static inline bool moss_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int moss_internal_cu_count();

// Numbers of calls, for words in a workspace of unknown contents that carry their own validity: a word that holds the number of
// the call in its upper 48 bits has been written by that call.  Never zero, never used again by this process.
uint64_t moss_next_call();
// A workgroup that looks for such words of others stops after so many looks (some milliseconds), or moss_quant_set_poll_limit's
// if that is less, and hands over what it waits for (moss::fold_is_ours): every kernel ends, whatever the others wait for.
constexpr uint32_t kMaxLooks = 1u << 12;
uint32_t moss_poll_limit();
static inline uint32_t moss_looks() { return moss_poll_limit() < kMaxLooks ? moss_poll_limit() : kMaxLooks; }
// false where a launch on the stream is being captured: a replay would use the number again, and find the words of the replay
// before it.
bool moss_may_number_calls(hipStream_t st);

// 256 x 256 tile fast path of the block-scaled GEMM; MOSS_ERR_UNSUPPORTED if the shape or
// operands do not qualify (the caller falls back to the general kernel).
int moss_internal_gemm_big(int64_t M, int64_t N, int64_t K, const uint8_t *a_q, const uint8_t *a_e, const float *a_s,
                           const uint8_t *b_q, const uint8_t *b_e, const float *b_s, void *out, int out_f32,
                           int64_t ld_out, int accumulate, hipStream_t st);
// whether the large-tile kernel takes the problem, and in half tiles (128 x 256)
bool moss_internal_gemm_big_ok(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, int64_t ld_out);
bool moss_internal_gemm_big_narrow(int64_t M, int64_t N);
// whether it can take a problem whose K is not a multiple of 128, and whether it should
bool moss_internal_gemm_big_ragged_ok(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, int64_t ld_out);
bool moss_internal_gemm_big_ragged(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, int accumulate,
                                   int64_t ld_out);

// small tiles and split K for problems that leave the large tiles idle, and ragged K: the kind of tiles, or -1 if another kernel
// is the better choice; MOSS_ERR_UNSUPPORTED if the device cannot launch them
int moss_internal_gemm_mid_kind(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, int accumulate,
                                bool large_ok);
int moss_internal_gemm_mid(int kind, int64_t M, int64_t N, int64_t K, const uint8_t *a_q, const uint8_t *a_e, const float *a_s,
                           const uint8_t *b_q, const uint8_t *b_e, const float *b_s, void *out, int out_f32, int64_t ld_out,
                           int accumulate, hipStream_t st);

namespace moss {

constexpr int kWave = 64;
constexpr int kGroup = 32;          // level-2 group size k2 (paper Sec. 3.1)
constexpr float kE4M3Max = 448.0f;  // Delta_max of E4M3 (paper Sec. 3.1)

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Streaming ("nontemporal") global accesses for data that is touched once per kernel: they
// do not allocate in the last-level cache, so a stream does not have to evict the dirty
// lines earlier kernels left there.  Measured on a cold 64-256 MB read: 5.1-6.5 TB/s against
// 2.7-3.0 TB/s with ordinary loads.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 ld_stream16(const void *p)
{
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ uint2 ld_stream8(const void *p)
{
    const u32x2 t = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p));
    return make_uint2(t.x, t.y);
}
__device__ __forceinline__ float4 ld_stream_f4(const void *p)
{
    const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void st_stream16(void *p, uint4 v)
{
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
}
__device__ __forceinline__ void st_stream8(void *p, uint2 v)
{
    __builtin_nontemporal_store(u32x2{v.x, v.y}, reinterpret_cast<u32x2 *>(p));
}
__device__ __forceinline__ void st_stream4(void *p, uint32_t v) { __builtin_nontemporal_store(v, reinterpret_cast<uint32_t *>(p)); }
__device__ __forceinline__ void st_stream_f4(void *p, float4 v)
{
    __builtin_nontemporal_store(f32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4 *>(p));
}

// How a producer stores BF16 tensors that the next kernel (its quantizer) reads: through the caches from 32 MiB a tensor,
// streaming below.  The eight L2s hold 32 MiB together and write what is dirty back when a kernel ends, which a small tensor
// pays for in full (1024 x 11008 SwiGLU with its quantizers: 141 us through the caches, 140 streaming; 2048 x 4096
// norm 90.5 and 89.4); a larger one leaves part of itself in the last-level cache (2048 x 11008: 189 and 196 us,
// 4096 x 11008: 277 and 298; norm 4096 x 4096: 112.6 both, 8192 x 4096: 166 and 177, 8192 x 8192: 305 and 317).
static inline int moss_stream_producer_stores(int64_t rows, int64_t cols) { return rows * cols <= ((int64_t)16 << 20); }

// One argument for both switches: the kernels hold it in a register for the stores, where an argument of its own for the
// look would be fetched at the end of the kernel, in front of it (1536 x 256 norm backward 14.1 instead of 12.9 us).
enum ProducerFlags { kProducerStream = 1, kProducerLook = 2 };
static inline int producer_flags(int64_t rows, int64_t cols, bool look)
{
    return (moss_stream_producer_stores(rows, cols) ? kProducerStream : 0) | (look ? kProducerLook : 0);
}

__device__ __forceinline__ void st_producer16(void *p, uint4 v, int stream)
{
    if (stream) st_stream16(p, v);
    else *reinterpret_cast<uint4 *>(p) = v;
}

// Merges a workgroup's maximum into a word that only grows while the kernel runs.  Atomics on one address are carried out
// one after the other, some 10 ns each: the 2048 of a norm of 2048 rows were 25 of its 30 us.  Looking first skips those that
// would change nothing (SwiGLU 4096 x 11008 with its quantizers 278 -> 260 us, 1024 x 11008 103 -> 92), but it is a trip to
// memory in front of the atomic, 0.4 to 0.9 us at the end of the kernel.  The launchers ask for it (`look`) from the number of
// workgroups on at which the queue of atomics takes longer; each gives both sides at its rule.
// The trip starts ahead of the workgroup's own reduction.
__device__ __forceinline__ uint32_t look_at_word(const uint32_t *word, int look)
{
    return look ? __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
}
__device__ __forceinline__ void merge_max_word(uint32_t *word, uint32_t m, uint32_t seen)
{
    if (m > seen) __hip_atomic_fetch_max(word, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Words of a call that one workgroup folds.  Each workgroup leaves its own, the last of the grid, which mostly starts last, looks
// for them all and folds them.  The others wait for nothing, but they may be kept off the machine for any time (the workgroups
// are dealt to the XCDs in turn, and another stream's kernel may fill some of them), so that the last stops looking after a
// while.  It then leaves a word that says so, `handed`, and looks once more; each of the others looks at that word behind its own
// words, and if it is there looks at all words once.  Of the words and `handed`, all written before their writers look, whoever
// wrote the last sees the others, so somebody finds all of them; the exchange makes that one workgroup.  Two calls that
// share the words by mistake may leave them unfolded, as words of each are missing; nobody waits for them.
//
// The looking wave: true if the fold is its own.  It has stored its workgroup's words itself.  all_there: looks once at this
// lane's share of the words.
__device__ __forceinline__ uint64_t look_at_call(const uint64_t *word)
{
    return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void leave_for_call(uint64_t *word, uint64_t call, uint32_t value)
{
    __hip_atomic_store(word, call << 16 | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename F>
__device__ __forceinline__ bool fold_is_ours(uint64_t *handed, uint64_t call, bool hand_over, F all_there)
{
    constexpr uint32_t kHanded = 1, kFolded = 2;
    const int lane = threadIdx.x & 63;
    if (hand_over && lane == 0) leave_for_call(handed, call, kHanded);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // what this wave has left is there for everyone
    if (!hand_over && !__any(look_at_call(handed) == (call << 16 | kHanded))) return false;
    if (!__all(all_there())) return false;
    uint64_t was = call << 16 | kHanded;
    return __any(lane == 0 && __hip_atomic_compare_exchange_strong(handed, &was, call << 16 | kFolded, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT));
}

// The same without the word: where the caller has memory to spare and calls may be numbered (moss_may_number_calls), each
// workgroup leaves its maxima (WORDS of them, BF16 magnitudes in thread 0) beside the number of the call in slots of its own,
// and the last of the grid, or whoever it hands over to, reads them all and writes the caller's words.  No launch to
// clear the words ahead, no queue of atomics, no look.  red: WORDS per wave.
struct MaxSlots {
    uint64_t *words;
    uint64_t call;           // 0: merge into the words, which a launch ahead has cleared
    uint32_t looks;
};
constexpr int kMaxSlotBlocks = 2048;

static inline MaxSlots max_slots(void *workspace, size_t bytes, int blocks, int words, hipStream_t st)
{
    const bool fits = workspace && moss_aligned16(workspace) && blocks <= kMaxSlotBlocks && bytes >= ((size_t)blocks * words + 1) * 8;
    return MaxSlots{(uint64_t *)workspace, fits && moss_may_number_calls(st) ? moss_next_call() : 0, moss_looks()};
}

template <int WORDS, int THREADS>
__device__ __forceinline__ void finish_max_in_slots(const MaxSlots &s, const uint32_t (&m)[WORDS], uint32_t *const (&out)[WORDS], uint32_t *red)
{
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < WORDS; w++) leave_for_call(s.words + (size_t)blockIdx.x * WORDS + w, s.call, m[w]);
    }
    constexpr int kLooks = 4;
    constexpr uint32_t kLate = ~0u;
    static_assert(THREADS % WORDS == 0 && kWave % WORDS == 0, "a thread's slots are all of one kind");
    const int n = (int)gridDim.x * WORDS;
    const bool last = blockIdx.x == gridDim.x - 1;
    auto write = [&](int w, uint32_t top) {
#pragma unroll
        for (int k = 0; k < WORDS; k++)
            if (w == k) *out[k] = top;
    };
    // the largest of each kind, in the first WORDS lanes of the wave
    auto largest = [&](uint32_t top) {
#pragma unroll
        for (int off = 32; off >= WORDS; off >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)top, off, 64);
            top = o > top ? o : top;
        }
        return top;
    };
    if (last) {
        uint32_t top = 0;
        for (int i0 = threadIdx.x; i0 < n; i0 += THREADS * kLooks) {
            uint64_t v[kLooks];
            bool there = false;
            for (uint32_t looks = 0; !there && looks < s.looks; looks++) {
                there = true;
#pragma unroll
                for (int u = 0; u < kLooks; u++) {
                    v[u] = s.call << 16;
                    if (i0 + u * THREADS < n) v[u] = look_at_call(s.words + i0 + u * THREADS);
                }
#pragma unroll
                for (int u = 0; u < kLooks; u++) there = there && (v[u] >> 16) == s.call;
                if (!there) __builtin_amdgcn_s_sleep(1);
            }
            if (!there) {
                top = kLate;
                break;
            }
#pragma unroll
            for (int u = 0; u < kLooks; u++) {
                const uint32_t x = (uint32_t)v[u] & 0xFFFFu;
                top = x > top ? x : top;
            }
        }
        top = largest(top);
        __syncthreads();             // (red is free: thread 0 has read what the workgroup's own reduction left)
        if ((threadIdx.x & 63) < WORDS) red[(threadIdx.x >> 6) * WORDS + (threadIdx.x & 63)] = top;
        __syncthreads();
        if (threadIdx.x >= kWave) return;
        top = 0;
        if (threadIdx.x < WORDS)
            for (int k = 0; k < THREADS / kWave; k++) {
                const uint32_t o = red[k * WORDS + threadIdx.x];
                top = o > top ? o : top;
            }
        if (!__any(top == kLate)) {
            if (threadIdx.x < WORDS) write((int)threadIdx.x, top);
            return;
        }
    }
    if (threadIdx.x >= kWave) return;
    uint32_t top = 0;
    const bool ours = fold_is_ours(s.words + n, s.call, last, [&]() {
        bool there = true;
        for (int i = threadIdx.x; i < n; i += kWave) {
            const uint64_t v = look_at_call(s.words + i);
            const uint32_t x = (uint32_t)v & 0xFFFFu;
            there = there && (v >> 16) == s.call;
            top = x > top ? x : top;
        }
        return there;
    });
    if (!ours) return;
    top = largest(top);
    if (threadIdx.x < WORDS) write((int)threadIdx.x, top);
}

// Two FP32 values -> two E4M3 bytes in the low half of the result.  The hardware
// converter rounds to nearest even; values are clamped to +-448 first so that the
// cast saturates instead of producing the NaN code.
__device__ __forceinline__ uint32_t cvt2_e4m3_sat(float a, float b)
{
    a = __builtin_amdgcn_fmed3f(a, kE4M3Max, -kE4M3Max);
    b = __builtin_amdgcn_fmed3f(b, kE4M3Max, -kE4M3Max);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false) & 0xFFFFu;
}

// Four FP32 values -> four E4M3 bytes (a in the lowest byte).
__device__ __forceinline__ uint32_t cvt4_e4m3_sat(float a, float b, float c, float d)
{
    a = __builtin_amdgcn_fmed3f(a, kE4M3Max, -kE4M3Max);
    b = __builtin_amdgcn_fmed3f(b, kE4M3Max, -kE4M3Max);
    c = __builtin_amdgcn_fmed3f(c, kE4M3Max, -kE4M3Max);
    d = __builtin_amdgcn_fmed3f(d, kE4M3Max, -kE4M3Max);
    int r = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, r, true);
    return (uint32_t)r;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        uint32_t o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ float wave_max_f32(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

}  // namespace moss
