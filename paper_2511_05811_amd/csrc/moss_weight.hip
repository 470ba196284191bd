// Per-tensor FP8 weights with automatic scaling for gfx950 (paper Sec. 3.2, Eq. 10;
// AdamW of Sec. 2.2 Eq. 1; App. C).
//
// The optimizer step is one streaming pass: each workgroup derives the predicted
// scale s_t = s_base + cum_lr/448 from the device-resident state (O(1), no
// max-reduction), applies AdamW to its slice, writes W, m, v and the E4M3 codes of the
// new weights, and leaves one partial amax / clipped-element count per workgroup in
// the workspace.  The pass's own last workgroup folds them into the state where they are few, else a one-workgroup
// kernel behind it.
// Partials instead of atomics keep the result independent of scheduling.
#include "moss_internal.h"

#pragma clang fp contract(off)

namespace moss {

constexpr int kWThreads = 256;
constexpr int kWMaxBlocks = 4096;   // grid cap of the flat (1-D) kernels
constexpr int kWTile = 128;         // tile edge of the 2-D kernel that also emits the transposed codes
// |y| <= 464 rounds to 448 by itself (464 is the midpoint to the next grid point, tie to
// even); beyond it the saturating cast changes the result: that is a clipped element.
constexpr float kClip = 464.0f;

struct WPartials {
    float *amax;      // [slots]
    uint32_t *over;   // [slots] elements outside 448 s
    uint32_t *clip;   // [slots] elements the saturation changed
};

// per-thread running by-products of a cast
struct WCounts {
    float amax = 0.0f;
    uint32_t over = 0, clip = 0;
};

// The scale is meant to keep |w| / s within 448 (Sec. 3.2, text under Eq. 10); an element is out of
// range when |w| > 448 s, compared exactly.  448 s has up to 27 significant bits, but for a single w
// "w > 448 s" is the same as "w > the largest single that does not exceed 448 s", so one
// double product per workgroup leaves a single-precision comparison per element.
__device__ __forceinline__ float range_limit(float s)
{
    const double exact = 448.0 * (double)s;
    float t = (float)exact;
    if ((double)t > exact) t = __uint_as_float(__float_as_uint(t) - 1u);
    return t;
}

__device__ __forceinline__ void count4(WCounts &c, const float4 &wv, float y0, float y1, float y2, float y3, float limit)
{
    c.over += (fabsf(wv.x) > limit) + (fabsf(wv.y) > limit) + (fabsf(wv.z) > limit) + (fabsf(wv.w) > limit);
    c.clip += (fabsf(y0) > kClip) + (fabsf(y1) > kClip) + (fabsf(y2) > kClip) + (fabsf(y3) > kClip);
}

// one slot per workgroup of the largest grid a call may launch
__host__ __device__ inline int64_t partial_slots(int64_t rows, int64_t cols)
{
    const int64_t tiles = ((rows + kWTile - 1) / kWTile) * ((cols + kWTile - 1) / kWTile);
    return tiles > kWMaxBlocks ? tiles : kWMaxBlocks;
}

__device__ __forceinline__ WPartials ws_partials(void *ws, int64_t slots)
{
    WPartials p;
    p.amax = reinterpret_cast<float *>(ws);
    p.over = reinterpret_cast<uint32_t *>(ws) + slots;
    p.clip = reinterpret_cast<uint32_t *>(ws) + 2 * slots;
    return p;
}

// Block-wide max / sums; the result is valid in thread 0 only.
template <int THREADS>
__device__ __forceinline__ void block_reduce(WCounts &c)
{
    __shared__ float r_amax[THREADS / kWave];
    __shared__ uint32_t r_over[THREADS / kWave], r_clip[THREADS / kWave];
    c.amax = wave_max_f32(c.amax);
    c.over = wave_sum_u32(c.over);
    c.clip = wave_sum_u32(c.clip);
    if ((threadIdx.x & 63) == 0) {
        r_amax[threadIdx.x >> 6] = c.amax;
        r_over[threadIdx.x >> 6] = c.over;
        r_clip[threadIdx.x >> 6] = c.clip;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < THREADS / kWave; i++) {
            c.amax = fmaxf(c.amax, r_amax[i]);
            c.over += r_over[i];
            c.clip += r_clip[i];
        }
    }
}

__device__ __forceinline__ void block_reduce_store(WCounts c, void *ws, int64_t slots)
{
    block_reduce<kWThreads>(c);
    if (threadIdx.x == 0) {
        WPartials p = ws_partials(ws, slots);
        const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
        p.amax[b] = c.amax;
        p.over[b] = c.over;
        p.clip[b] = c.clip;
    }
}

// the state after a step with scale prediction
__device__ __forceinline__ void advance_state(moss_wscale_state *st, const WCounts &c, double lr_term, int64_t step)
{
    if (st->step + 1 != step) st->flags |= MOSS_WSTATE_STEP_MISMATCH;
    const double cum = st->cum_lr + lr_term;
    st->cum_lr = cum;
    st->s_cur = (float)((double)st->s_base + cum / 448.0);
    st->step += 1;
    st->amax_seen = c.amax;
    st->overflow_count += c.over;
    st->clipped_count += c.clip;
}

// The fold inside the pass.  A workgroup leaves its partial as four 64-bit words, the number of the call in the upper 48 bits
// and in the others the maximum's lower and upper half and the two counts (it has fewer than 2^16 elements): a word that holds
// the number is this call's (see moss_next_call), so nothing has to be cleared or counted, and the words may arrive in any
// order.  The last workgroup of the grid, or whoever it hands over to (fold_is_ours), advances the state once all words are
// there; by then all workgroups have read the state.  The launch behind the pass that this replaces took 2 us on the
// device, with what lies between two kernels, and 2.3 on the host.  Steps back to back: 64 x 64 8.3 -> 6.7 us, 512 x 256 9.0 -> 7.2, 1024 x
// 1024 10.8 -> 9.5, 1792 x 1792 27.1 -> 24.6, 2048 x 2048 28.0 -> 26.5, 4096 x 4096 103.4 -> 101.9.
struct StepEnd {
    uint64_t call;            // 0: partials for the kernel behind
    int64_t step;
    double lr_term;
    uint32_t looks;
};
constexpr int kFoldWords = 4;
constexpr int kFoldBlocks = 1024;
static_assert((kFoldBlocks * kFoldWords + 1) * 8 <= kWMaxBlocks * 12, "the words, and one to hand over by, fit the smallest workspace");
static_assert(kFoldBlocks < kWMaxBlocks && kWTile * kWTile < 1 << 16, "a workgroup's elements (flat: 16 per thread below kWMaxBlocks)");

// one look at the partial of workgroup i, added to c if it is there
__device__ __forceinline__ bool take_partial(const uint64_t *words, int i, uint64_t call, WCounts &c)
{
    uint64_t w[kFoldWords];
    bool there = true;
#pragma unroll
    for (int j = 0; j < kFoldWords; j++) w[j] = look_at_call(words + i * kFoldWords + j);
#pragma unroll
    for (int j = 0; j < kFoldWords; j++) there = there && (w[j] >> 16) == call;
    if (!there) return false;
    c.amax = fmaxf(c.amax, __uint_as_float(((uint32_t)w[0] & 0xFFFFu) | (uint32_t)w[1] << 16));
    c.over += (uint32_t)w[2] & 0xFFFFu;
    c.clip += (uint32_t)w[3] & 0xFFFFu;
    return true;
}

__device__ __forceinline__ void block_reduce_end(WCounts c, void *ws, int64_t slots, moss_wscale_state *st, const StepEnd &end)
{
    if (end.call == 0) {
        block_reduce_store(c, ws, slots);
        return;
    }
    __shared__ uint32_t late;
    if (threadIdx.x == 0) late = 0;
    block_reduce<kWThreads>(c);
    uint64_t *words = reinterpret_cast<uint64_t *>(ws), *handed = words + kFoldBlocks * kFoldWords;
    const int n = (int)(gridDim.x * gridDim.y), mine = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (threadIdx.x < kWave) {
        const uint32_t amax = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(c.amax));
        const uint32_t over = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.over), clip = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.clip);
        const int j = threadIdx.x;
        if (j < kFoldWords) leave_for_call(words + mine * kFoldWords + j, end.call, j == 0 ? amax & 0xFFFFu : j == 1 ? amax >> 16 : j == 2 ? over : clip);
    }
    const bool last = mine == n - 1;
    WCounts all;
    if (last) {
        for (int i = threadIdx.x; i < n; i += kWThreads) {
            bool there = false;
            for (uint32_t looks = 0; !there && looks < end.looks; looks++) {
                there = take_partial(words, i, end.call, all);
                if (!there) __builtin_amdgcn_s_sleep(1);
            }
            if (!there) late = 1;
        }
        __syncthreads();             // (and thread 0 has read what the first reduction left)
        if (!late) {
            block_reduce<kWThreads>(all);
            if (threadIdx.x == 0) advance_state(st, all, end.lr_term, end.step);
            return;
        }
    }
    if (threadIdx.x >= kWave) return;
    const bool ours = fold_is_ours(handed, end.call, last, [&]() {
        bool there = true;
        all = WCounts();
        for (int i = threadIdx.x; i < n; i += kWave) there = take_partial(words, i, end.call, all) && there;
        return there;
    });
    if (!ours) return;
    all.amax = wave_max_f32(all.amax);
    all.over = wave_sum_u32(all.over);
    all.clip = wave_sum_u32(all.clip);
    if (threadIdx.x == 0) advance_state(st, all, end.lr_term, end.step);
}

__device__ __forceinline__ float4 load_as_f32x4(const void *p, int64_t i4, bool bf16)
{
    if (bf16) {
        uint2 r = ld_stream8(reinterpret_cast<const uint2 *>(p) + i4);
        return make_float4(bf16_bits_to_f32(r.x & 0xFFFFu), __uint_as_float(r.x & 0xFFFF0000u),
                           bf16_bits_to_f32(r.y & 0xFFFFu), __uint_as_float(r.y & 0xFFFF0000u));
    }
    return ld_stream_f4(reinterpret_cast<const float4 *>(p) + i4);
}

struct AdamW {
    float lr, beta1, beta2, eps, wd, omb1, omb2, bc1, bc2;
};

// One AdamW element update; every operation is a single correctly rounded FP32
// operation in the order of Eq. 1 of the paper (no FMA contraction; the build asks for
// IEEE division and square root).
__device__ __forceinline__ void adamw_elem(float &w, float &m, float &v, float g, const AdamW &a)
{
    float mi = a.beta1 * m + a.omb1 * g;
    float vi = a.beta2 * v + (a.omb2 * g) * g;
    float mhat = mi / a.bc1;
    float vhat = vi / a.bc2;
    float den = sqrtf(vhat) + a.eps;
    float u = mhat / den;
    float upd = a.lr * (u + a.wd * w);
    w = w - upd;
    m = mi;
    v = vi;
}

// Scale the cast of this call uses.  predict != 0: Eq. 10 from the state before the
// step; predict == 0: the scale already stored in the state (after init / re-base).
__device__ __forceinline__ float scale_for_cast(const moss_wscale_state *st, int predict, double lr_term)
{
    if (!predict) return st->s_cur;
    double cum = st->cum_lr + lr_term;
    return (float)((double)st->s_base + cum / 448.0);
}

// One vector of four elements in the AdamW pass.
struct StepVec {
    float4 w, m, v, g;
};

__device__ __forceinline__ void load_step(StepVec &t, const float *w, const float *m, const float *v, const void *g, int64_t i4,
                                          bool g_bf16)
{
    t.w = ld_stream_f4(reinterpret_cast<const float4 *>(w) + i4);
    t.m = ld_stream_f4(reinterpret_cast<const float4 *>(m) + i4);
    t.v = ld_stream_f4(reinterpret_cast<const float4 *>(v) + i4);
    t.g = load_as_f32x4(g, i4, g_bf16);
}

__device__ __forceinline__ void step_and_store(StepVec &t, const AdamW &a, float *w, float *m, float *v, int64_t i4)
{
    adamw_elem(t.w.x, t.m.x, t.v.x, t.g.x, a);
    adamw_elem(t.w.y, t.m.y, t.v.y, t.g.y, a);
    adamw_elem(t.w.z, t.m.z, t.v.z, t.g.z, a);
    adamw_elem(t.w.w, t.m.w, t.v.w, t.g.w, a);
    st_stream_f4(reinterpret_cast<float4 *>(w) + i4, t.w);
    st_stream_f4(reinterpret_cast<float4 *>(m) + i4, t.m);
    st_stream_f4(reinterpret_cast<float4 *>(v) + i4, t.v);
}

__device__ __forceinline__ float absmax4(const float4 &t)
{
    return fmaxf(fmaxf(fabsf(t.x), fabsf(t.y)), fmaxf(fabsf(t.z), fabsf(t.w)));
}

// Bound: HBM (four streams in, three or four out).  BATCH vectors per thread are loaded ahead of the first store: one at a time,
// a wave's loads queue behind its own stores and 11008 x 8192 with BF16 gradients took 572 us (4.2 TB/s); two at a time 492 us,
// four 457 us (5.3 TB/s, the rate of the tile kernel below and of a plain copy).  (Contiguous ranges per workgroup: 466 us;
// ordinary instead of streaming loads: 513 against 572 us with one vector, nothing on top of four.)  step_batch has the rule.
template <bool G_BF16, bool DO_CAST, int BATCH>
__global__ __launch_bounds__(kWThreads) void k_adamw_cast(float *__restrict__ w, float *__restrict__ m,
                                                          float *__restrict__ v, const void *__restrict__ g,
                                                          int64_t n4, AdamW a, StepEnd end,
                                                          moss_wscale_state *st,
                                                          uint8_t *__restrict__ wq, void *ws, int64_t slots)
{
    float inv_s = 0.0f, limit = 0.0f;
    if (DO_CAST) {
        float s = scale_for_cast(st, 1, end.lr_term);
        inv_s = s > 0.0f ? 1.0f / s : 0.0f;
        limit = range_limit(s);
    }
    WCounts cnt;
    auto finish = [&](StepVec &t, int64_t i) {
        step_and_store(t, a, w, m, v, i);
        cnt.amax = fmaxf(cnt.amax, absmax4(t.w));
        if (DO_CAST) {
            const float y0 = t.w.x * inv_s, y1 = t.w.y * inv_s, y2 = t.w.z * inv_s, y3 = t.w.w * inv_s;
            count4(cnt, t.w, y0, y1, y2, y3, limit);
            st_stream4(reinterpret_cast<uint32_t *>(wq) + i, cvt4_e4m3_sat(y0, y1, y2, y3));
        }
    };
    const int64_t stride = (int64_t)gridDim.x * kWThreads * BATCH;
    for (int64_t i0 = (int64_t)blockIdx.x * kWThreads * BATCH + threadIdx.x; i0 < n4; i0 += stride) {
        StepVec t[BATCH];
        if (BATCH == 1) {
            load_step(t[0], w, m, v, g, i0, G_BF16);
            finish(t[0], i0);
        } else {
#pragma unroll
            for (int u = 0; u < BATCH; u++) {
                const int64_t i = i0 + u * kWThreads;
                if (i < n4) load_step(t[u], w, m, v, g, i, G_BF16);
            }
#pragma unroll
            for (int u = 0; u < BATCH; u++) {
                const int64_t i = i0 + u * kWThreads;
                if (i < n4) finish(t[u], i);
            }
        }
    }
    block_reduce_end(cnt, ws, slots, st, end);
}

template <bool W_BF16>
__global__ __launch_bounds__(kWThreads) void k_weight_amax(const void *__restrict__ w, int64_t n4, void *ws, int64_t slots)
{
    WCounts cnt;
    const int64_t stride = (int64_t)gridDim.x * kWThreads;
    for (int64_t i = (int64_t)blockIdx.x * kWThreads + threadIdx.x; i < n4; i += stride) {
        float4 wv = load_as_f32x4(w, i, W_BF16);
        cnt.amax = fmaxf(cnt.amax, fmaxf(fmaxf(fabsf(wv.x), fabsf(wv.y)), fmaxf(fabsf(wv.z), fabsf(wv.w))));
    }
    block_reduce_store(cnt, ws, slots);
}

template <bool W_BF16>
__global__ __launch_bounds__(kWThreads) void k_weight_cast(const void *__restrict__ w, int64_t n4,
                                                           const moss_wscale_state *__restrict__ st,
                                                           uint8_t *__restrict__ wq, void *ws, int64_t slots)
{
    const float s = scale_for_cast(st, 0, 0.0);
    const float inv_s = s > 0.0f ? 1.0f / s : 0.0f;
    const float limit = range_limit(s);
    WCounts cnt;
    const int64_t stride = (int64_t)gridDim.x * kWThreads;
    for (int64_t i = (int64_t)blockIdx.x * kWThreads + threadIdx.x; i < n4; i += stride) {
        float4 wv = load_as_f32x4(w, i, W_BF16);
        cnt.amax = fmaxf(cnt.amax, fmaxf(fmaxf(fabsf(wv.x), fabsf(wv.y)), fmaxf(fabsf(wv.z), fabsf(wv.w))));
        float y0 = wv.x * inv_s, y1 = wv.y * inv_s, y2 = wv.z * inv_s, y3 = wv.w * inv_s;
        count4(cnt, wv, y0, y1, y2, y3, limit);
        st_stream4(reinterpret_cast<uint32_t *>(wq) + i, cvt4_e4m3_sat(y0, y1, y2, y3));
    }
    block_reduce_store(cnt, ws, slots);
}

// 2-D variant used when the transposed codes are wanted as well: a workgroup owns a
// ROWS x 128 tile, walks it 8 rows at a time (32 lanes x float4 = one 512-byte row piece),
// writes the codes row-major (128 bytes per row) and collects them transposed in LDS;
// at the end ROWS / 16 lanes write the ROWS bytes of each transposed row.  STEP: apply AdamW first
// (fused optimizer step), otherwise cast only, with the scale already in the state.
//
// ROWS = 128 leaves whole lines of the transposed codes.  A weight of few such tiles is bound by the chain of 16
// trips through memory of each workgroup, not by the rate: there ROWS = 32 has four times the workgroups with a
// quarter of the trips.  BATCH vectors are loaded ahead of the first store, as in the flat pass; see tile_form for the
// rule and what it measured.
template <bool STEP, bool SRC_BF16, int ROWS, int BATCH>
__global__ __launch_bounds__(kWThreads) void k_weight_tile(float *__restrict__ w, float *__restrict__ m,
                                                           float *__restrict__ v, const void *__restrict__ src,
                                                           int64_t rows, int64_t cols, AdamW a, StepEnd end,
                                                           moss_wscale_state *st,
                                                           uint8_t *__restrict__ wq, uint8_t *__restrict__ wq_t,
                                                           void *ws, int64_t slots)
{
    constexpr int kPitch = ROWS + 4;
    __shared__ __attribute__((aligned(16))) uint8_t tt[kWTile][kPitch];   // [column][row]
    const float s = scale_for_cast(st, STEP ? 1 : 0, end.lr_term);
    const float inv_s = s > 0.0f ? 1.0f / s : 0.0f;
    const float limit = range_limit(s);
    const int tid = threadIdx.x, rl = tid >> 5, c4 = (tid & 31) * 4;
    const int64_t r0 = (int64_t)blockIdx.y * ROWS, c0 = (int64_t)blockIdx.x * kWTile;
    const int64_t col = c0 + c4;
    WCounts cnt;
    // Casts the new weights of a vector and leaves the codes in the tile; 0 beyond the matrix.
    auto cast_vector = [&](const float4 &wv, int64_t i4) {
        cnt.amax = fmaxf(cnt.amax, absmax4(wv));
        const float y0 = wv.x * inv_s, y1 = wv.y * inv_s, y2 = wv.z * inv_s, y3 = wv.w * inv_s;
        count4(cnt, wv, y0, y1, y2, y3, limit);
        const uint32_t code = cvt4_e4m3_sat(y0, y1, y2, y3);
        st_stream4(reinterpret_cast<uint32_t *>(wq) + i4, code);
        return code;
    };
    auto transpose_codes = [&](int rr, uint32_t code) {
        tt[c4][rr] = (uint8_t)code;
        tt[c4 + 1][rr] = (uint8_t)(code >> 8);
        tt[c4 + 2][rr] = (uint8_t)(code >> 16);
        tt[c4 + 3][rr] = (uint8_t)(code >> 24);
    };
    auto load_vector = [&](StepVec &t, int64_t i4) {
        if (STEP) load_step(t, w, m, v, src, i4, SRC_BF16);
        else t.w = load_as_f32x4(src, i4, SRC_BF16);
    };
    // (cols % 4 == 0: a float4 is inside or outside as a whole)
    if (BATCH == 1) {
#pragma unroll 4
        for (int it = 0; it < ROWS / 8; it++) {
            const int rr = it * 8 + rl;
            const int64_t row = r0 + rr;
            uint32_t code = 0;
            if (row < rows && col < cols) {
                const int64_t i4 = (row * cols + col) >> 2;
                StepVec t;
                load_vector(t, i4);
                if (STEP) step_and_store(t, a, w, m, v, i4);
                code = cast_vector(t.w, i4);
            }
            transpose_codes(rr, code);
        }
    } else {
#pragma unroll 1
        for (int it0 = 0; it0 < ROWS / 8; it0 += BATCH) {
            StepVec t[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; u++) {
                const int64_t row = r0 + (it0 + u) * 8 + rl;
                if (row < rows && col < cols) load_vector(t[u], (row * cols + col) >> 2);
            }
#pragma unroll
            for (int u = 0; u < BATCH; u++) {
                const int rr = (it0 + u) * 8 + rl;
                const int64_t row = r0 + rr;
                uint32_t code = 0;
                if (row < rows && col < cols) {
                    const int64_t i4 = (row * cols + col) >> 2;
                    if (STEP) step_and_store(t[u], a, w, m, v, i4);
                    code = cast_vector(t[u].w, i4);
                }
                transpose_codes(rr, code);
            }
        }
    }
    __syncthreads();
    constexpr int kPieces = ROWS / 16;               // 16-byte pieces of a transposed row
#pragma unroll
    for (int k = 0; k < kWTile * kPieces / kWThreads; k++) {
        const int idx = tid + k * kWThreads, c = idx / kPieces, piece = idx % kPieces;
        if (c0 + c < cols && r0 + piece * 16 < rows) {   // rows % 16 == 0: a 16-row piece is whole
            const uint32_t *p = reinterpret_cast<const uint32_t *>(&tt[c][piece * 16]);
            st_stream16(wq_t + (c0 + c) * rows + r0 + piece * 16, make_uint4(p[0], p[1], p[2], p[3]));
        }
    }
    block_reduce_end(cnt, ws, slots, st, end);
}

enum FinalizeMode {
    kFinInit = 0,     // after k_weight_amax at initialisation: reset state, s_base = s_cur = amax/448
    kFinStep = 1,     // after a fused step: advance step / cum_lr / s_cur, record amax, add overflow
    kFinRebase = 2,   // after an AdamW-only pass on a re-scaling step: s_base = s_cur = amax/448
    kFinCastOnly = 3  // after a cast-only pass: record amax, add overflow
};

// `step`: the step number the caller says this call performs (only looked at by the two modes that
// advance the step count): a caller whose count has drifted from the state's is flagged in the state.
//
// One workgroup, bound by the latency of its loads.  THREADS = 1024 for the more than 1024 partials of a large weight (the flat
// pass leaves up to kWMaxBlocks, the tile pass one per tile), so that a few per thread are in flight together (130.2 -> 129.5 us
// for a flat step with 4096, BF16 gradients); fewer are folded by 256 threads, which start and meet sooner: 0.3 us per call, of
// 6.4 for 4 x 1024 and of 8.4 for 64 x 1024, twice that where the scale is re-based.
constexpr int kFinThreads = 1024;

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_weight_finalize(moss_wscale_state *st, void *ws, int64_t slots,
                                                             int n_partial, int mode, double lr_term, int64_t step)
{
    WPartials p = ws_partials(ws, slots);
    WCounts c;
#pragma unroll 4
    for (int i = threadIdx.x; i < n_partial; i += THREADS) {
        c.amax = fmaxf(c.amax, p.amax[i]);
        c.over += p.over[i];
        c.clip += p.clip[i];
    }
    block_reduce<THREADS>(c);
    if (threadIdx.x != 0) return;
    const float amax = c.amax;
    const uint32_t over = c.over, clip = c.clip;
    if (mode == kFinStep) {
        advance_state(st, c, lr_term, step);
        return;
    }
    if (mode == kFinRebase && st->step + 1 != step) st->flags |= MOSS_WSTATE_STEP_MISMATCH;
    if (mode == kFinInit) {
        st->s_base = amax / kE4M3Max;
        st->s_cur = st->s_base;
        st->cum_lr = 0.0;
        st->step = 0;
        st->last_rebase = 0;
        st->amax_seen = amax;
        st->overflow_count = 0;
        st->clipped_count = 0;
        st->flags = 0;
    } else if (mode == kFinRebase) {
        st->step += 1;
        st->s_base = amax / kE4M3Max;
        st->s_cur = st->s_base;
        st->cum_lr = 0.0;
        st->last_rebase = st->step;
        st->amax_seen = amax;
    } else {
        st->amax_seen = amax;
        st->overflow_count += over;
        st->clipped_count += clip;
    }
}

// Byte transpose [rows x cols] -> [cols x rows] through a padded LDS tile.
constexpr int kTT = 64;
__global__ __launch_bounds__(256) void k_transpose_u8(const uint8_t *__restrict__ src, int64_t rows, int64_t cols,
                                                      uint8_t *__restrict__ dst)
{
    __shared__ uint8_t tile[kTT][kTT + 4];
    const int64_t r0 = (int64_t)blockIdx.y * kTT, c0 = (int64_t)blockIdx.x * kTT;
    for (int i = threadIdx.x; i < kTT * kTT; i += 256) {
        int r = i / kTT, c = i % kTT;
        if (r0 + r < rows && c0 + c < cols) tile[r][c] = src[(r0 + r) * cols + c0 + c];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kTT * kTT; i += 256) {
        int c = i / kTT, r = i % kTT;
        if (r0 + r < rows && c0 + c < cols) dst[(c0 + c) * rows + r0 + r] = tile[r][c];
    }
}

static int grid_for(int64_t n4)
{
    int64_t per_block = (int64_t)kWThreads * 4;   // >= 4 vectors per thread before striding
    int64_t blocks = (n4 + per_block - 1) / per_block;
    if (blocks < 1) blocks = 1;
    return (int)(blocks < kWMaxBlocks ? blocks : kWMaxBlocks);
}

// BATCH of k_adamw_cast: four vectors from two vectors per thread of the largest grid on (8M elements), and for a step with its
// cast on up to one workgroup per compute unit.  Step alone, buffers that no cache holds, us, one vector and four:
//   0.25M elements 10.2 and 9.7 (re-base 15.2, 15.6)    0.75M 11.2 and 10.7 (16.7, 16.9)    1.5M 13.7 and 15.1 (20.0, 22.3)
//   2M 15.8 and 16.3    6M 40.0 and 41.5 (BF16 gradients 37.5, 40.0)    8M 52.0 and 51.7    12M 76.6 and 72.5    64M 401 and 361
// What reads the result next finds it in the L2 of the XCD that wrote it only if both give a vector to the same workgroup.  The
// cast behind a re-basing pass walks the grid-wide stride, as the pass does with one vector (64K elements 13.2, 14.5); the byte
// transpose behind a step (heights that the tile kernel does not take) walks 64 x 64 tiles, of which a workgroup of four writes
// whole ones if rows are narrow (1038 x 64 18.2, 13.4; 427 x 192 17.0, 15.3; wider than 256 0.4 us more with four).  Otherwise
// fewer than 32 workgroups are bound by the latency of their code, which is shorter with one.
constexpr int kStepBatch = 4;

enum StepNext { kNextNothing, kNextCast, kNextNarrowTranspose };

static int step_batch(int64_t n4, int grid, StepNext next)
{
    if (n4 >= 2 * (int64_t)kWMaxBlocks * kWThreads) return kStepBatch;
    int cus = moss_internal_cu_count();
    if (cus <= 0) cus = 256;
    return next != kNextCast && grid <= cus && (grid >= 32 || next == kNextNarrowTranspose) ? kStepBatch : 1;
}

static int launch_transpose(const uint8_t *src, int64_t rows, int64_t cols, uint8_t *dst, hipStream_t st)
{
    int64_t gx = (cols + kTT - 1) / kTT, gy = (rows + kTT - 1) / kTT;
    if (gy > 65535) return MOSS_ERR_SHAPE;
    hipLaunchKernelGGL(k_transpose_u8, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, st, src, rows, cols, dst);
    MOSS_LAUNCH_CHECK();
    return MOSS_OK;
}

}  // namespace moss

extern "C" size_t moss_weight_workspace_bytes(int64_t rows, int64_t cols)
{
    if (rows <= 0 || cols <= 0) return 0;
    return (size_t)moss::partial_slots(rows, cols) * (sizeof(float) + 2 * sizeof(uint32_t));
}

static int check_weight_common(int64_t rows, int64_t cols, const void *state, const void *wq, const void *wq_t,
                               const void *ws, size_t ws_bytes)
{
    if (!state || !wq) return MOSS_ERR_NULL;
    if (rows <= 0 || cols <= 0 || (rows * cols) % 4) return MOSS_ERR_SHAPE;
    if (!moss_aligned16(wq) || ((uintptr_t)state & 7)) return MOSS_ERR_ALIGN;
    if (wq_t && !moss_aligned16(wq_t)) return MOSS_ERR_ALIGN;
    if (!ws || ws_bytes < moss_weight_workspace_bytes(rows, cols)) return MOSS_ERR_WORKSPACE;
    if (!moss_aligned16(ws)) return MOSS_ERR_ALIGN;
    return MOSS_OK;
}

namespace moss {

// the 2-D kernel needs whole float4 per row and whole 16-row pieces per transposed row
static bool tile_path_ok(int64_t rows, int64_t cols) { return cols % 4 == 0 && rows % 16 == 0; }

// Form of k_weight_tile by the number of 128 x 128 tiles: step with FP32 gradients and transposed codes, in us,
//                                tiles  8 (512 x 256)   64 (1024^2)   256 (2048^2)   512 (4096 x 2048)   1024 (4096^2)   2752 (11008 x 4096)
//   32 rows, batches of 4               12.2            12.1          28.5           55.8                110
//   128 rows, one vector at a time      18.1            26.8          31.6           52                  104             273 (BF16 gradients 256)
//   128 rows, batches of 4              19.6            28.1          37.2           58                  104             264 (239)
// Batches raise the rate (5.0 -> 5.2 TB/s) once many rounds of workgroups overlap one's loads with another's stores.  Alone
// they cost nothing from 1024 tiles on, but behind the GEMM that has just written the gradient they do (4096^2 in a
// training step: + 5 us): from eight tiles per compute unit.
enum TileForm { kTile32, kTile128, kTile128Batched };

static TileForm tile_form(int64_t rows, int64_t cols)
{
    const int64_t tiles = ((rows + kWTile - 1) / kWTile) * ((cols + kWTile - 1) / kWTile);
    int64_t cus = moss_internal_cu_count();
    if (cus <= 0) cus = 256;
    if (tiles <= cus && tiles * 4 <= kWMaxBlocks) return kTile32;        // (four times the tiles have to fit the workspace)
    return tiles < 8 * cus ? kTile128 : kTile128Batched;
}

struct WLaunch {
    int64_t rows, cols, n4, slots;
    int grid1d;
    TileForm form;
    dim3 grid2d;
    hipStream_t st;
    void *ws;
    moss_wscale_state *state;
};

// (many workgroups are left to the kernel behind, whose time counts little there)
static bool folds_itself(int blocks) { return blocks <= kFoldBlocks; }

static int fold_threads(int n_partial) { return n_partial <= 4 * kWThreads ? kWThreads : kFinThreads; }

static int finalize(const WLaunch &L, int n_partial, int mode, double lr_term, int64_t step = 0)
{
    const int threads = fold_threads(n_partial);
    const auto kern = threads == kWThreads ? k_weight_finalize<kWThreads> : k_weight_finalize<kFinThreads>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(threads), 0, L.st, L.state, L.ws, L.slots, n_partial, mode, lr_term, step);
    MOSS_LAUNCH_CHECK();
    return MOSS_OK;
}

template <bool CAST>
static void launch_flat(const WLaunch &L, bool grad_bf16, float *w, float *m, float *v, const void *g, const AdamW &a, const StepEnd &end,
                        uint8_t *wq, StepNext next)
{
    const auto kern = step_batch(L.n4, L.grid1d, next) == 1
                          ? (grad_bf16 ? k_adamw_cast<true, CAST, 1> : k_adamw_cast<false, CAST, 1>)
                          : (grad_bf16 ? k_adamw_cast<true, CAST, kStepBatch> : k_adamw_cast<false, CAST, kStepBatch>);
    hipLaunchKernelGGL(kern, dim3(L.grid1d), dim3(kWThreads), 0, L.st, w, m, v, g, L.n4, a, end, L.state, wq, L.ws, L.slots);
}

template <bool STEP, bool SRC_BF16>
static void launch_tile_of(const WLaunch &L, float *w, float *m, float *v, const void *src, const AdamW &a, const StepEnd &end, uint8_t *wq,
                           uint8_t *wq_t)
{
    const auto kern = L.form == kTile32    ? k_weight_tile<STEP, SRC_BF16, 32, 4>
                      : L.form == kTile128 ? k_weight_tile<STEP, SRC_BF16, kWTile, 1>
                                           : k_weight_tile<STEP, SRC_BF16, kWTile, STEP ? 4 : 1>;   // (cast alone, 11008 x 4096: 61 us in batches, 54)
    hipLaunchKernelGGL(kern, L.grid2d, dim3(kWThreads), 0, L.st, w, m, v, src, L.rows, L.cols, a, end, L.state, wq, wq_t, L.ws,
                       L.slots);
}

template <bool STEP>
static void launch_tile(const WLaunch &L, bool src_bf16, float *w, float *m, float *v, const void *src, const AdamW &a, const StepEnd &end,
                        uint8_t *wq, uint8_t *wq_t)
{
    if (src_bf16) launch_tile_of<STEP, true>(L, w, m, v, src, a, end, wq, wq_t);
    else launch_tile_of<STEP, false>(L, w, m, v, src, a, end, wq, wq_t);
}

// cast (and transposed copy) of the weights under the scale stored in the state
static int cast_only(const WLaunch &L, const void *w, bool bf16, uint8_t *wq, uint8_t *wq_t)
{
    const AdamW none{};
    if (wq_t && tile_path_ok(L.rows, L.cols)) {
        launch_tile<false>(L, bf16, nullptr, nullptr, nullptr, w, none, StepEnd{}, wq, wq_t);
        MOSS_LAUNCH_CHECK();
        return finalize(L, (int)(L.grid2d.x * L.grid2d.y), kFinCastOnly, 0.0);
    }
    if (bf16)
        hipLaunchKernelGGL(k_weight_cast<true>, dim3(L.grid1d), dim3(kWThreads), 0, L.st, w, L.n4, L.state, wq, L.ws, L.slots);
    else
        hipLaunchKernelGGL(k_weight_cast<false>, dim3(L.grid1d), dim3(kWThreads), 0, L.st, w, L.n4, L.state, wq, L.ws, L.slots);
    MOSS_LAUNCH_CHECK();
    int rc = finalize(L, L.grid1d, kFinCastOnly, 0.0);
    if (rc) return rc;
    if (wq_t) return launch_transpose(wq, L.rows, L.cols, wq_t, L.st);
    return MOSS_OK;
}

static int make_launch(WLaunch &L, int64_t rows, int64_t cols, moss_wscale_state *state, void *ws, void *stream)
{
    L.rows = rows; L.cols = cols; L.n4 = rows * cols / 4; L.slots = partial_slots(rows, cols);
    L.grid1d = grid_for(L.n4);
    L.form = tile_form(rows, cols);
    const int64_t tile_rows = L.form == kTile32 ? 32 : kWTile;
    const int64_t gx = (cols + kWTile - 1) / kWTile, gy = (rows + tile_rows - 1) / tile_rows;
    if (gy > 65535 || gx > 0x7FFFFFFF) return MOSS_ERR_SHAPE;
    L.grid2d = dim3((unsigned)gx, (unsigned)gy);
    L.st = (hipStream_t)stream; L.ws = ws; L.state = state;
    return MOSS_OK;
}

}  // namespace moss

// what the launches below choose (the tests hold the rules by it)
extern "C" int moss_internal_weight_fold_threads(int64_t n_partial) { return moss::fold_threads((int)n_partial); }

extern "C" int moss_internal_weight_step_batch(int64_t rows, int64_t cols, int64_t next)
{
    return moss::step_batch(rows * cols / 4, moss::grid_for(rows * cols / 4), (moss::StepNext)next);
}

extern "C" int moss_weight_autoscale_init(const void *w, int w_dtype, int64_t rows, int64_t cols,
                                          moss_wscale_state *state, uint8_t *wq, uint8_t *wq_t,
                                          void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace moss;
    if (!w) return MOSS_ERR_NULL;
    if (w_dtype != MOSS_DT_F32 && w_dtype != MOSS_DT_BF16) return MOSS_ERR_UNSUPPORTED;
    int rc = check_weight_common(rows, cols, state, wq, wq_t, workspace, workspace_bytes);
    if (rc) return rc;
    if (!moss_aligned16(w)) return MOSS_ERR_ALIGN;
    WLaunch L;
    if ((rc = make_launch(L, rows, cols, state, workspace, stream))) return rc;
    const bool bf16 = w_dtype == MOSS_DT_BF16;
    if (bf16)
        hipLaunchKernelGGL(k_weight_amax<true>, dim3(L.grid1d), dim3(kWThreads), 0, L.st, w, L.n4, workspace, L.slots);
    else
        hipLaunchKernelGGL(k_weight_amax<false>, dim3(L.grid1d), dim3(kWThreads), 0, L.st, w, L.n4, workspace, L.slots);
    MOSS_LAUNCH_CHECK();
    if ((rc = finalize(L, L.grid1d, kFinInit, 0.0))) return rc;
    return cast_only(L, w, bf16, wq, wq_t);
}

extern "C" int moss_weight_autoscale_cast(float *w, float *m, float *v, const void *g, int g_dtype,
                                          int64_t rows, int64_t cols, const moss_adamw_args *args,
                                          moss_wscale_state *state, uint8_t *wq, uint8_t *wq_t,
                                          void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace moss;
    if (!w || !m || !v || !g || !args) return MOSS_ERR_NULL;
    if (g_dtype != MOSS_DT_F32 && g_dtype != MOSS_DT_BF16) return MOSS_ERR_UNSUPPORTED;
    int rc = check_weight_common(rows, cols, state, wq, wq_t, workspace, workspace_bytes);
    if (rc) return rc;
    if (!moss_aligned16(w) || !moss_aligned16(m) || !moss_aligned16(v) || ((uintptr_t)g & 7)) return MOSS_ERR_ALIGN;
    if (g_dtype == MOSS_DT_F32 && !moss_aligned16(g)) return MOSS_ERR_ALIGN;
    if (args->step < 1) return MOSS_ERR_SHAPE;

    WLaunch L;
    if ((rc = make_launch(L, rows, cols, state, workspace, stream))) return rc;
    AdamW a{args->lr, args->beta1, args->beta2, args->eps, args->weight_decay,
            args->one_minus_beta1, args->one_minus_beta2, args->bias_corr1, args->bias_corr2};
    const double lr_term = (double)args->margin * (double)args->lr;
    const bool rebase = args->interval > 0 && (args->step % args->interval) == 0;
    const bool gb = g_dtype == MOSS_DT_BF16;

    if (rebase) {
        // AdamW alone (it yields amax(W_new)), re-base the scale from it, then cast with the new scale
        launch_flat<false>(L, gb, w, m, v, g, a, StepEnd{0, 0, lr_term, 0}, wq, kNextCast);
        MOSS_LAUNCH_CHECK();
        if ((rc = finalize(L, L.grid1d, kFinRebase, lr_term, args->step))) return rc;
        return cast_only(L, w, false, wq, wq_t);
    }
    const bool tiled = wq_t && tile_path_ok(rows, cols);
    const int blocks = tiled ? (int)(L.grid2d.x * L.grid2d.y) : L.grid1d;
    const StepEnd end{folds_itself(blocks) && moss_may_number_calls(L.st) ? moss_next_call() : 0, args->step, lr_term, moss_looks()};
    if (tiled) launch_tile<true>(L, gb, w, m, v, g, a, end, wq, wq_t);
    else launch_flat<true>(L, gb, w, m, v, g, a, end, wq, wq_t && cols <= 256 ? kNextNarrowTranspose : kNextNothing);
    MOSS_LAUNCH_CHECK();
    if (end.call == 0 && (rc = finalize(L, blocks, kFinStep, lr_term, args->step))) return rc;
    if (tiled) return MOSS_OK;
    if (wq_t) return launch_transpose(wq, rows, cols, wq_t, L.st);
    return MOSS_OK;
}
