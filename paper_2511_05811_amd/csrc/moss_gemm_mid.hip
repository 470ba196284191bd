// Block-scaled FP8 GEMM for problems that do not fill the machine with 256-wide tiles, and for many that the 256-wide tiles
// cannot take, K % 128 != 0 above all (paper Sec. 3.1, Fig. 3b: only block-scaled matrix instructions in the main loop, the
// two FP32 scales once in the epilogue).
//
// What bounds these problems is not the matrix pipe but how much of the operands is in flight: a compute unit takes
// full 128-byte lines at about 62 B/clk, a miss takes some 2000 clocks, and with few tiles most compute units would
// idle.  Hence
//  * small tiles, so that there are enough workgroups, and the four waves of a workgroup split K as well (KS): each of
//    the KS groups of WM x WN waves multiplies a contiguous part of K for the whole tile, and the partial sums meet in
//    LDS at the end, in a fixed order.  A wave always computes (32 MI) x (32 NJ) outputs, so the LDS bytes read per
//    matrix instruction do not grow as the tile shrinks.
//  * SLOTS stages of K = 128 per group in flight as direct global->LDS copies of full lines.  A wave takes both
//    substeps' fragments of a stage into registers, hands the slot straight back to the copies of stage + SLOTS and
//    multiplies afterwards.  A group of one wave (WM = WN = 1) fills and reads slots of its own: its loop has no barrier.
//  * the exponent bytes of the tile are brought to LDS ahead of the loop, as one dword (four groups, K = 128) per row
//    and stage in [stage][row] order with a pitch of rows + 1 dwords, which neither the writes nor the reads find
//    conflicts in.  A K range too long for that area is walked in several pieces.
//  * K % 128 != 0: the copies of the last stage are clamped into the row, the missing part of the a fragments is zeroed
//    and its exponents are 127 (rows of K / 32 exponents are then not dword aligned: they are cut out of two dwords).
//
// Operand layout of V_MFMA_SCALE_F32_32X32X64_F8F6F4 and the LDS swizzle are those of the large-tile kernel.
#include <atomic>
#include <cmath>

#include "moss_gemm.h"

namespace moss {

extern __shared__ __attribute__((aligned(1024))) uint8_t mid_smem[];

constexpr int kMidThreads = 256;
constexpr int kMidK = 128;            // bytes of K per stage: one line per row

struct MidArgs {
    int64_t M, N, K;
    const uint8_t *a_q, *a_e;
    const float *a_s;
    const uint8_t *b_q, *b_e;
    const float *b_s;
    void *out;
    int64_t ld_out;
    int out_f32, accumulate;
    int tiles_m, tiles_n;
    int panel_stages;                 // stages whose exponents fit the LDS area
    int e_dwords;                     // exponent rows are dword aligned
};

template <int MI, int NJ, int WM, int WN, int KS, int SLOTS>
struct MidShape {
    static constexpr int kBM = 32 * MI * WM, kBN = 32 * NJ * WN;
    static constexpr int kRows = kBM + kBN;
    static constexpr int kGroupBytes = kRows * kMidK;                  // one group's stage: a rows, then b rows
    static constexpr int kSlot = KS * kGroupBytes;
    static constexpr int kPanel = SLOTS * kSlot;                       // byte offset of the exponent area
    static constexpr int kReduce = KS == 1 ? 0 : kBM * kBN * 4 * KS;   // partial sums (they reuse the slots and the area)
    static constexpr int kPA = kBM / 8 / (WM * WN), kPB = kBN / 8 / (WM * WN);   // 8-row copies of a, of b per wave and stage
    static constexpr int kPieces = kPA + kPB;
    static_assert(WM * WN * KS * 64 == kMidThreads, "four waves");
    static_assert(MI * NJ == 1 || MI * NJ % KS == 0, "whole fragments per wave");
    static_assert(kBM % (16 * WM * WN) == 0 && kBN % (16 * WM * WN) == 0, "an even number of whole copies per wave and operand");
};

template <int MI, int NJ, int WM, int WN, int KS, int SLOTS, bool HAS_BE>
__global__ __launch_bounds__(kMidThreads) void k_gemm_mx_mid(const MidArgs p)
{
    using S = MidShape<MI, NJ, WM, WN, KS, SLOTS>;
    constexpr int kBM = S::kBM, kBN = S::kBN, kPA = S::kPA, kPieces = S::kPieces;
    constexpr bool kAlone = WM * WN == 1;        // a group is one wave: nothing shared inside the loop
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave / (WM * WN), wg = wave % (WM * WN), wm = wg / WN, wn = wg % WN;
    const int i32 = lane & 31, h = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)mid_smem;
    const int64_t M = p.M, N = p.N, K = p.K;
    const int G = (int)(K >> 5);
    const int C = (int)((K + kMidK - 1) / kMidK);     // stages of the whole K range

    const float scale = (*p.a_s) * (*p.b_s);

    // Workgroups are dealt round-robin to the 8 XCDs: each XCD gets a contiguous range of tiles, in bands of 8 tile rows walked
    // column by column, so that the tiles it works on at a time form a block that shares rows of a and of b in its L2 (tile
    // rows to the end first: 4096 x 2048 x 4096 in 128 x 128 tiles 55 us, in bands 47; one band where there are fewer).
    int tm, tn;
    {
        const uint32_t total = (uint32_t)p.tiles_m * (uint32_t)p.tiles_n, q = total >> 3, r = total & 7;
        const uint32_t xcd = blockIdx.x & 7, pid = xcd * q + (xcd < r ? xcd : r) + (blockIdx.x >> 3);
        constexpr uint32_t kBand = 8;
        const uint32_t rows = (uint32_t)p.tiles_m, band = pid / (kBand * (uint32_t)p.tiles_n), rem = pid - band * kBand * (uint32_t)p.tiles_n;
        const uint32_t here = rows - band * kBand < kBand ? rows - band * kBand : kBand;
        tn = __builtin_amdgcn_readfirstlane((int)(rem / here));
        tm = __builtin_amdgcn_readfirstlane((int)(band * kBand + rem % here));
    }
    const int64_t m0 = (int64_t)tm * kBM, n0 = (int64_t)tn * kBN;
    const uint8_t *a_base = p.a_q + m0 * K, *b_base = p.b_q + n0 * K;
    const int last_a = (int)(M - m0 < kBM ? M - m0 : kBM) - 1, last_b = (int)(N - n0 < kBN ? N - n0 : kBN) - 1;

    // This lane's byte offsets of the wave's copies: piece x covers 8 rows of a (x < kPA) or of b, the lane fetches the 16-byte
    // chunk that its place in the swizzled row holds.  Rows beyond the matrix repeat the last row.
    uint32_t off[kPieces];
    uint32_t chunk[2];                           // (pieces of even and of odd number swizzle differently)
#pragma unroll
    for (int x = 0; x < 2; x++) chunk[x] = (uint32_t)((lane & 7) ^ ((x * 4 + (lane >> 4)) & 7)) * 16;
#pragma unroll
    for (int x = 0; x < kPieces; x++) {
        const int row = (x < kPA ? wg * kPA + x : wg * S::kPB + x - kPA) * 8 + (lane >> 3), last = x < kPA ? last_a : last_b;
        off[x] = (uint32_t)(row < last ? row : last) * (uint32_t)K + chunk[x & 1];
    }
    // Copies of a stage into a slot.  Stage C - 1 of a K that ends inside it is copied in one go, with offsets clamped into the
    // row.
    const uint32_t tail = (uint32_t)(K - (int64_t)(C - 1) * kMidK);      // bytes of the last stage that exist
    struct Bases {
        const uint8_t *a, *b;
        uint32_t dst_a, dst_b;
    };
    const uint32_t dst_a0 = lds0 + (uint32_t)(ks * S::kGroupBytes + wg * kPA * 1024);
    const uint32_t dst_b0 = lds0 + (uint32_t)(ks * S::kGroupBytes + kBM * kMidK + wg * S::kPB * 1024);
    auto bases = [&](int c, uint32_t slot_at) {
        return Bases{a_base + (int64_t)c * kMidK, b_base + (int64_t)c * kMidK, dst_a0 + slot_at, dst_b0 + slot_at};
    };
    auto copy_piece = [&](const Bases &t, int x) {
        if (x < kPA) dma16_at(t.a, off[x], t.dst_a, x * 1024);
        else dma16_at(t.b, off[x], t.dst_b, (x - kPA) * 1024);
    };
    auto copy_tail = [&](const Bases &t) {
#pragma unroll
        for (int x = 0; x < kPieces; x++) {
            const uint32_t o = chunk[x & 1] < tail ? off[x] : off[x] - chunk[x & 1];
            if (x < kPA) dma16_at(t.a, o, t.dst_a, x * 1024);
            else dma16_at(t.b, o, t.dst_b, (x - kPA) * 1024);
        }
    };
    auto is_tail = [&](int c) { return tail < (uint32_t)kMidK && c == C - 1; };

    // Exponents of stages [cb, cb + nc) into LDS: dword of (stage, row) at area[stage * (rows + 1) + row]
    uint32_t *area_a = reinterpret_cast<uint32_t *>(mid_smem + S::kPanel);
    uint32_t *area_b = area_a + p.panel_stages * (kBM + 1);
    auto load_exponents = [&](const uint8_t *e, uint32_t *area, int rows, int64_t row0, int last, int64_t limit, int cb, int nc) {
        const int per_row = kMidThreads / rows;              // threads that share a row (192 rows: one, and 64 are left over)
        const int r = tid / per_row;
        if (r >= rows) return;
        const int64_t at = (row0 + (r < last ? r : last)) * G + cb * 4;       // of this row's first dword, in bytes
        const int first = tid % per_row;
        constexpr int U = 8;
        if (!e) {
            for (int c = first; c < nc; c += per_row) area[c * (rows + 1) + r] = 0x7F7F7F7Fu;       // 2^0
        } else if (p.e_dwords) {
            const uint8_t *src = e + at;
            for (int c0 = first; c0 < nc; c0 += per_row * U) {
                uint32_t d[U];
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (c0 + u * per_row < nc) d[u] = *reinterpret_cast<const uint32_t *>(src + (c0 + u * per_row) * 4);
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (c0 + u * per_row < nc) area[(c0 + u * per_row) * (rows + 1) + r] = d[u];
            }
        } else {
            // rows that are not dword aligned (e itself is): cut out of two neighbouring dwords where both lie inside the
            // array, byte by byte at its end; 127 (2^0) beyond the row's end
            const int64_t safe = limit * G - 8;
            const int left = G - cb * 4, k = (int)(at & 3);
            const uint8_t *src = e + (at - k);
            constexpr int V = U / 2;
            for (int c0 = first; c0 < nc; c0 += per_row * V) {
                uint32_t lo[V], hi[V];
#pragma unroll
                for (int u = 0; u < V; u++) {
                    const int c = c0 + u * per_row;
                    lo[u] = hi[u] = 0;
                    if (c < nc && at - k + c * 4 <= safe) {
                        lo[u] = *reinterpret_cast<const uint32_t *>(src + c * 4);
                        hi[u] = *reinterpret_cast<const uint32_t *>(src + c * 4 + 4);
                    }
                }
#pragma unroll
                for (int u = 0; u < V; u++) {
                    const int c = c0 + u * per_row;
                    if (c >= nc) continue;
                    uint32_t d = __builtin_amdgcn_alignbyte(hi[u], lo[u], (uint32_t)k);
                    const int there = left - c * 4;          // bytes of this dword inside the row (at least one)
                    if (at - k + c * 4 > safe) {
                        d = 0;
                        for (int b = 0; b < 4 && b < there; b++) d |= (uint32_t)src[k + c * 4 + b] << (8 * b);
                    }
                    if (there < 4) d = (d & (0xFFFFFFFFu >> (32 - 8 * there))) | (0x7F7F7F7Fu << (8 * there));
                    area[c * (rows + 1) + r] = d;
                }
            }
        }
    };

    v16f acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < NJ; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;

    const int sw = (i32 >> 1) & 7;
    const uint8_t *frag_a = mid_smem + ks * S::kGroupBytes + (wm * 32 * MI + i32) * kMidK;
    const uint8_t *frag_b = mid_smem + ks * S::kGroupBytes + (kBM + wn * 32 * NJ + i32) * kMidK;
    struct Stage {
        v8i a[2][MI], b[2][NJ];
        int sa[MI], sb[NJ];
    };
    // The assembly form of the instruction needs accumulators that are not named again before it has retired: with one or
    // two accumulators the compiler pads the instructions instead.
    auto multiply = [&](int s, v16f &d, const v8i &x, const v8i &y, int sx, int sy) {
        if (MI * NJ >= 4) {
            if (s == 0) mfma_scaled<0>(d, x, y, sx, sy);
            else mfma_scaled<2>(d, x, y, sx, sy);
        } else {
            if (s == 0) d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, d, 0, 0, 0, sx, 0, sy);
            else d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, d, 0, 0, 2, sx, 2, sy);
            asm volatile("" : "+a"(d));          // (keeps the instruction here)
        }
    };
    // 16-byte read number x of a stage's fragments (both substeps; a, then b; low and high half)
    constexpr int kReads = 4 * (MI + NJ);
    auto read_piece = [&](Stage &f, int so, int x) {
        const int s = x / (2 * (MI + NJ)), fr = x % (2 * (MI + NJ)) / 2, half = x & 1;
        const uint8_t *row = fr < MI ? frag_a + fr * 32 * kMidK : frag_b + (fr - MI) * 32 * kMidK;
        const uint4 v = *reinterpret_cast<const uint4 *>(row + so + (((4 * s + 2 * half + h) ^ sw) << 4));
        v8i &dst = fr < MI ? f.a[s][fr] : f.b[s][fr - MI];
        dst[4 * half + 0] = (int)v.x; dst[4 * half + 1] = (int)v.y; dst[4 * half + 2] = (int)v.z; dst[4 * half + 3] = (int)v.w;
    };
    auto read_exponents = [&](uint32_t (&ra)[MI], uint32_t (&rb)[NJ], int c) {
#pragma unroll
        for (int i = 0; i < MI; i++) ra[i] = area_a[c * (kBM + 1) + wm * 32 * MI + i * 32 + i32];
#pragma unroll
        for (int j = 0; j < NJ; j++) rb[j] = HAS_BE ? area_b[c * (kBN + 1) + wn * 32 * NJ + j * 32 + i32] : 0x7F7F7F7Fu;
    };
    // byte 0 / 2 of a scale register = this lane's group in substep 0 / 1 (volatile: stays where it is put, away from
    // the matrix instructions that read the registers)
    const int sh8 = 8 * h;
    auto shift_exponents = [&](Stage &f, const uint32_t (&ra)[MI], const uint32_t (&rb)[NJ]) {
#pragma unroll
        for (int i = 0; i < MI; i++) asm volatile("v_lshrrev_b32 %0, %1, %2" : "=v"(f.sa[i]) : "v"(sh8), "v"(ra[i]));
#pragma unroll
        for (int j = 0; j < NJ; j++) asm volatile("v_lshrrev_b32 %0, %1, %2" : "=v"(f.sb[j]) : "v"(sh8), "v"(rb[j]));
    };

    // all but the copies of the wave's `newer` latest stages (at most SLOTS - 2 are in flight behind the one waited for)
    auto wait_newer = [&](int newer) {
        if (SLOTS > 3 && newer >= 2) wait_vmcnt<2 * kPieces>();
        else if (SLOTS > 2 && newer >= 1) wait_vmcnt<kPieces>();
        else wait_vmcnt<0>();
    };

    for (int cb = 0; cb < C; cb += p.panel_stages) {
        const int nc = C - cb < p.panel_stages ? C - cb : p.panel_stages;
        // this group's contiguous part of the piece; `per` iterations for everyone (barriers)
        const int per = (nc + KS - 1) / KS;
        const int c0 = ks * per < nc ? ks * per : nc;
        const int n = per < nc - c0 ? per : nc - c0;
        if (cb > 0) __syncthreads();             // slots and exponents of the last piece have been read
#pragma unroll
        for (int s = 0; s < SLOTS; s++)
            if (s < n) {
                const Bases t = bases(cb + c0 + s, s * S::kSlot);
                if (is_tail(cb + c0 + s)) {
                    copy_tail(t);
                } else {
#pragma unroll
                    for (int x = 0; x < kPieces; x++) copy_piece(t, x);
                }
            }
        load_exponents(p.a_e, area_a, kBM, m0, last_a, M, cb, nc);
        if (HAS_BE) load_exponents(p.b_e, area_b, kBN, n0, last_b, N, cb, nc);
        wait_vmcnt<0>();
        __syncthreads();

        // One barrier per stage.  At the top of iteration `it` the wave holds the fragments of its stage `it`: behind
        // the barrier every wave of the group does, so that stage's slot may be refilled, and everyone's part of stage
        // it + 1 has landed.  The reads of its fragments and the copies of stage it + SLOTS are dealt out between the
        // matrix instructions of stage `it`, the reads over the first three quarters of them, so that the last have arrived
        // at the next barrier.
        //
        // There are two copies of an iteration.  With one wave per SIMD whatever runs between two matrix instructions beyond
        // their 64 clocks leaves the matrix pipe idle, and with everything that can happen at either end of K asked
        // for on the way (a stage to refill with? which of the waits? the last stage?) that was as much again: 8 matrix
        // instructions of 128 x 128 took 0.44 us without any reads and copies, of which they themselves are 0.21.  So the
        // iterations in the middle, which always refill and never see the last stage, ask nothing.
        Stage f0, f1;
        uint32_t slot_at = 0;                     // byte offset of the slot of stage `it`
        constexpr uint32_t kEnd = SLOTS * S::kSlot;
        if (n > 0) {
            uint32_t ra[MI], rb[NJ];
            read_exponents(ra, rb, c0);
#pragma unroll
            for (int x = 0; x < kReads; x++) read_piece(f0, 0, x);
            shift_exponents(f0, ra, rb);
        }
        constexpr int kMat = 2 * MI * NJ, kReadMat = kMat - kMat / 4;
        // the matrix instructions of a stage, and between them what the next ones need
        auto stage = [&](Stage &f, Stage &next, const Bases &t, uint32_t next_at, const uint32_t (&ra)[MI], const uint32_t (&rb)[NJ], bool refill) {
#pragma unroll
            for (int q = 0; q < kMat; q++) {
                const int s = q / (MI * NJ), i = q % (MI * NJ) / NJ, j = q % NJ;
                multiply(s, acc[i][j], f.b[s][j], f.a[s][i], f.sb[j], f.sa[i]);
                if (q < kReadMat) {
#pragma unroll
                    for (int x = q * kReads / kReadMat; x < (q + 1) * kReads / kReadMat; x++) read_piece(next, (int)next_at, x);   // (behind the last stage: read and not used)
                }
#pragma unroll
                for (int x = q * kPieces / kMat; x < (q + 1) * kPieces / kMat; x++)
                    if (refill) copy_piece(t, x);
                if (q == kMat / 2) shift_exponents(next, ra, rb);
                pin();
            }
        };
        // iterations that refill a slot with a whole stage, an even number of them
        const bool ends_here = tail < (uint32_t)kMidK && cb + c0 + n == C;
        int middle = n - SLOTS - (ends_here ? 1 : 0);
        middle = middle > 0 ? middle & ~1 : 0;
        Bases t = bases(cb + c0 + SLOTS, 0);
        uint32_t at_a = (uint32_t)((c0 + 1) * (kBM + 1)), at_b = (uint32_t)((c0 + 1) * (kBN + 1));      // exponents of stage it + 1
        auto middle_step = [&](Stage &f, Stage &next) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wait_vmcnt<(SLOTS - 2) * kPieces>();
            if (!kAlone) {
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            uint32_t ra[MI], rb[NJ];
#pragma unroll
            for (int i = 0; i < MI; i++) ra[i] = area_a[at_a + wm * 32 * MI + i * 32 + i32];
#pragma unroll
            for (int j = 0; j < NJ; j++) rb[j] = HAS_BE ? area_b[at_b + wn * 32 * NJ + j * 32 + i32] : 0x7F7F7F7Fu;
            const uint32_t next_at = slot_at + S::kSlot == kEnd ? 0 : slot_at + S::kSlot;
            t.dst_a = dst_a0 + slot_at;
            t.dst_b = dst_b0 + slot_at;
            asm volatile("s_nop 4" ::: "memory");    // vector ALU write -> operand of a matrix instruction
            stage(f, next, t, next_at, ra, rb, true);
            t.a += kMidK;
            t.b += kMidK;
            at_a += kBM + 1;
            at_b += kBN + 1;
            slot_at = next_at;
        };
        int it = 0;
        for (; it < middle; it += 2) {
            middle_step(f0, f1);
            middle_step(f1, f0);
        }
        auto step = [&](Stage &f, Stage &next, int it) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wait_newer(n - 2 - it);              // stage it + 1 has landed
            if (!kAlone) {
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            const uint32_t next_at = slot_at + S::kSlot == kEnd ? 0 : slot_at + S::kSlot;
            if (it < n) {
                const int c = cb + c0 + it;
                if (is_tail(c)) {
#pragma unroll
                    for (int s = 0; s < 2; s++)
#pragma unroll
                        for (int half = 0; half < 2; half++)
                            if ((uint32_t)(4 * s + 2 * half + h) * 16 >= tail)
#pragma unroll
                                for (int i = 0; i < MI; i++)
#pragma unroll
                                    for (int v = 0; v < 4; v++) f.a[s][i][4 * half + v] = 0;
                }
                const bool last = it + SLOTS < n && is_tail(c + SLOTS), refill = it + SLOTS < n && !last;
                const Bases t = bases(c + SLOTS, slot_at);
                uint32_t ra[MI], rb[NJ];
                read_exponents(ra, rb, it + 1 < n ? c0 + it + 1 : c0);
                asm volatile("s_nop 4" ::: "memory");    // vector ALU write -> operand of a matrix instruction
                stage(f, next, t, next_at, ra, rb, refill);
                if (last) copy_tail(t);
            }
            slot_at = next_at;
        };
        for (; it < per; it += 2) {
            step(f0, f1, it);
            if (it + 1 < per) step(f1, f0, it + 1);
        }
    }

    // Epilogue with one K group: straight from the registers (see store_fragment)
    if (KS == 1) {
#pragma unroll
        for (int i = 0; i < MI; i++)
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[i][j]));   // the last matrix instructions retire
                store_fragment(acc[i][j], scale, p.out, p.ld_out, m0 + (wm * MI + i) * 32 + i32, n0 + (wn * NJ + j) * 32, h, M, N, p.out_f32,
                               p.accumulate);
            }
        return;
    }

    // Epilogue with several and more than one fragment per wave: the waves that computed the same outputs store an equal part of
    // their fragments each.  A wave leaves the others in LDS, register by register as they lie, takes the sums of the other
    // waves for its own, adds them in the order of the groups and stores from the registers.  (512 x 4096 x 512 in 64 x 128 tiles
    // 7.4 -> 6.7 us, 256 x 4096 x 4096 in 64 x 64 12.0 -> 11.7, against sums left in rows and walked as below; a single fragment,
    // a quarter of it per wave, took 0.2 us longer this way.)
    constexpr int kFrags = MI * NJ;
    if (kFrags > 1) {
        constexpr int kOwn = kFrags / KS;
        float4 *sums = reinterpret_cast<float4 *>(mid_smem);
#pragma unroll
        for (int f = 0; f < kFrags; f++) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[f / NJ][f % NJ]));   // the last matrix instructions retire
        __syncthreads();                         // slots and exponents have been read
#pragma unroll
        for (int f = 0; f < kFrags; f++)
            if (f / kOwn != ks)
#pragma unroll
                for (int qd = 0; qd < 4; qd++) {
                    const v16f &a = acc[f / NJ][f % NJ];
                    sums[((wave * kFrags + f) * 4 + qd) * kWave + lane] = make_float4(a[4 * qd], a[4 * qd + 1], a[4 * qd + 2], a[4 * qd + 3]);
                }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KS; k++) {
            if (k != ks) continue;               // (one part of the code per group: registers have no index)
#pragma unroll
            for (int f = k * kOwn; f < (k + 1) * kOwn; f++) {
                v16f &a = acc[f / NJ][f % NJ];
#pragma unroll
                for (int qd = 0; qd < 4; qd++) {
                    float4 t = make_float4(a[4 * qd], a[4 * qd + 1], a[4 * qd + 2], a[4 * qd + 3]);
                    const float4 own = t;
#pragma unroll
                    for (int g = 0; g < KS; g++) {
                        const float4 x = g == k ? own : sums[(((g * WM * WN + wg) * kFrags + f) * 4 + qd) * kWave + lane];
                        if (g == 0) t = x;
                        else { t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w; }
                    }
                    a[4 * qd] = t.x; a[4 * qd + 1] = t.y; a[4 * qd + 2] = t.z; a[4 * qd + 3] = t.w;
                }
                store_fragment(a, scale, p.out, p.ld_out, m0 + (wm * MI + f / NJ) * 32 + i32, n0 + (wn * NJ + f % NJ) * 32, h, M, N, p.out_f32,
                               p.accumulate);
            }
        }
        return;
    }

    // ... and a single fragment (32 x 32 tiles, a K group per wave): every wave leaves its sums in LDS (row pitch 32 floats, 16-byte
    // chunks XOR-swizzled by row), then a thread adds the KS parts of four columns of a row in order, scales and stores.
    // (accumulator register v of lane (i32, h): row i32, column 8 (v / 4) + 4 h + v % 4)
    if (kFrags == 1) {
        static_assert(kFrags > 1 || (WM * WN == 1 && S::kBM * S::kBN == 4 * kMidThreads), "four outputs per thread");
        constexpr int kPart = 32 * 32;               // floats per wave
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]));   // the last matrix instructions retire
        __syncthreads();                             // slots and exponents have been read
        float *part = reinterpret_cast<float *>(mid_smem);
#pragma unroll
        for (int qd = 0; qd < 4; qd++)
            *reinterpret_cast<float4 *>(part + wave * kPart + i32 * 32 + (((2 * qd + h) ^ (i32 & 7)) << 2)) =
                make_float4(acc[0][0][4 * qd], acc[0][0][4 * qd + 1], acc[0][0][4 * qd + 2], acc[0][0][4 * qd + 3]);
        __syncthreads();
        const bool vec_ok = p.ld_out % 4 == 0;
        const int row = tid / 8, c4 = tid % 8;
        const float *src = part + row * 32 + ((c4 ^ (row & 7)) << 2);
        float4 t = *reinterpret_cast<const float4 *>(src);
#pragma unroll
        for (int k = 1; k < KS; k++) {
            const float4 u = *reinterpret_cast<const float4 *>(src + k * kPart);
            t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
        }
        const int64_t m = m0 + row, nn = n0 + 4 * c4;
        if (m >= M || nn >= N) return;
        const float r[4] = {t.x * scale, t.y * scale, t.z * scale, t.w * scale};
        if (p.out_f32) {
            float *o = reinterpret_cast<float *>(p.out) + m * p.ld_out + nn;
            if (vec_ok && nn + 3 < N) {
                float4 v = make_float4(r[0], r[1], r[2], r[3]);
                if (p.accumulate) {
                    const float4 q = *reinterpret_cast<const float4 *>(o);
                    v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
                }
                *reinterpret_cast<float4 *>(o) = v;
            } else {
                for (int x = 0; x < 4 && nn + x < N; x++) o[x] = p.accumulate ? o[x] + r[x] : r[x];
            }
        } else {
            uint16_t *o = reinterpret_cast<uint16_t *>(p.out) + m * p.ld_out + nn;
            const uint32_t lo = pack_bf16(r[0], r[1]), hi = pack_bf16(r[2], r[3]);
            if (vec_ok && nn + 3 < N) {
                *reinterpret_cast<uint2 *>(o) = make_uint2(lo, hi);
            } else {
                for (int x = 0; x < 4 && nn + x < N; x++) o[x] = (uint16_t)((x & 2 ? hi : lo) >> (16 * (x & 1)));
            }
        }
    }
}

// LDS for the exponents: what is left of `budget` behind the slots
template <int MI, int NJ, int WM, int WN, int KS, int SLOTS>
static int launch_mid(MidArgs p, int budget, hipStream_t st)
{
    using S = MidShape<MI, NJ, WM, WN, KS, SLOTS>;
    const int64_t tiles_m = (p.M + S::kBM - 1) / S::kBM, tiles_n = (p.N + S::kBN - 1) / S::kBN;
    if (tiles_m * tiles_n > 0x7FFFFFF) return MOSS_ERR_UNSUPPORTED;
    const int stages = (int)((p.K + kMidK - 1) / kMidK);
    const int per_stage = 4 * ((S::kBM + 1) + (p.b_e ? S::kBN + 1 : 0));
    const int fit = (budget - S::kPanel) / per_stage;
    if (fit < 1) return MOSS_ERR_UNSUPPORTED;
    p.panel_stages = fit < stages ? fit : stages;
    p.tiles_m = (int)tiles_m;
    p.tiles_n = (int)tiles_n;
    int lds = S::kPanel + p.panel_stages * per_stage;
    if (lds < S::kReduce) lds = S::kReduce;
    const int be = p.b_e ? 1 : 0;
    const auto kern = be ? k_gemm_mx_mid<MI, NJ, WM, WN, KS, SLOTS, true> : k_gemm_mx_mid<MI, NJ, WM, WN, KS, SLOTS, false>;
    static std::atomic<bool> attr_set[64][2];    // per device and kernel: the LDS size it may ask for has been raised
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOSS_ERR_HIP;
    if (!attr_set[dev][be].load()) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
            (void)hipGetLastError();
            return MOSS_ERR_UNSUPPORTED;
        }
        attr_set[dev][be].store(true);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(kMidThreads), (size_t)lds, st, p);
    if (hipGetLastError() != hipSuccess) return MOSS_ERR_HIP;
    return MOSS_OK;
}

}  // namespace moss

// Time of a problem in the kernels that could take it, in microseconds: a launch, then per round of tiles over the compute
// units a fixed part (first latency, exponents, epilogue) and a part per iteration (stages of K = 128, dealt over the K groups
// of a tile), each with a share that grows with how full the rounds are.  The constants are fits to 2200 random problems (M 32 to
// 12000, N 256 to 12288, K 128 to 12288; calls back to back on two sets of operands, 256 compute units), each run in every
// kernel that can take it; the fits missed by 2 to 7 % (mean), 10 % at the 10th and 90th percentile.  K % 128 != 0: the rows no longer start on lines and
// the exponents are cut out of two dwords, so that a stage costs more.  "b" marks exponents of b, whose outputs are FP32.
// The fits are from before tiles of 64 x 128 and more, and FP32 outputs of the large ones, stored from the registers: a round of
// these takes up to 3 us less by now, of the large ones up to 5.  What the kernels take now:
//   tile        (M, N, K) measured / model
//   32 x 32     (256, 1024, 1024) 4.4 / 4.5    (17, 11008, 4096) 10.0 / 10.1
//   64 x 64     (1024, 1024, 1024) 6.3 / 7.0   (256, 4096, 4096) 12.0 / 12.3
//   64 x 128    (512, 4096, 1024) 7.8 / 8.9    (512, 4096, 4096) 14.7 / 16.3
//   128 x 128   (2048, 2048, 1024) 10.0 / 12.1 (2048, 2048, 4096) 22.6 / 24.0
//   128 x 192   (2048, 3072, 1024) 12.5 / 15.5 (2048, 3072, 7168) 43.4 / 44.6
//   large       (2048, 4096, 2048) 19.7 / 18.9 (4096, 4096, 4096) 60 / 58      (4096, 4096, 512) b 23.7 / 28.1
//   ... ragged  (11328, 3520, 2080) 105 / 105  (1336, 4096, 4128) 40.9 / 36.4  (2432, 6016, 2656) b 56.0 / 57.3
//   general     (4096, 4096, 2080) 66 / 62     (6321, 2424, 32) 14.8 / 15.9    (2528, 2912, 8032) b 128 / 131
namespace {

double rounds_of(double tiles, double cus) { return tiles <= cus ? 1.0 : std::ceil(tiles / cus); }
double tiles_of(int64_t M, int64_t N, int bm, int bn) { return (double)((M + bm - 1) / bm) * (double)((N + bn - 1) / bn); }

struct Cost {
    double round, round_full, it, it_full;      // per round, and per iteration in a round; their part that goes with its fill
};

double us_of(const Cost &c, double tiles, double cus, double iterations, double per_round = 0.0)
{
    const double n = rounds_of(tiles, cus), u = tiles / (n * cus);
    return 2.2 + n * (c.round + per_round + c.round_full * u + iterations * (c.it + c.it_full * u));
}

struct MidPlan {
    int kind;        // 0 .. 4: the tiles above, smallest first
    double us;
};

MidPlan plan_mid(int64_t M, int64_t N, int64_t K, bool b_exponents, bool accumulate, bool large_ok, double cus)
{
    // [kind 1 .. 4][K % 128 != 0][exponents of b]
    static const Cost cost[4][2][2] = {{{{2.43, 0.59, 0.704, 0.175}, {3.03, 0.63, 0.738, 0.253}}, {{2.38, 0.54, 0.953, 0.381}, {2.90, 0.45, 1.100, 0.565}}},
                                       {{{3.38, 0.86, 0.514, 0.101}, {3.84, 1.03, 0.700, 0.129}}, {{3.27, 0.94, 0.728, 0.210}, {3.82, 1.11, 1.009, 0.285}}},
                                       {{{4.76, 1.22, 0.354, 0.140}, {5.79, 1.68, 0.406, 0.150}}, {{4.78, 1.66, 0.510, 0.179}, {5.56, 1.95, 0.667, 0.206}}},
                                       {{{6.86, 1.59, 0.419, 0.187}, {8.05, 2.53, 0.622, 0.178}}, {{7.90, 2.23, 0.630, 0.205}, {7.67, 2.63, 0.960, 0.267}}}};
    // 32 x 32: one round; two workgroups fit a compute unit, so that more rounds cost less each
    static const double one[2][2][2] = {{{3.71, 0.407}, {4.27, 0.409}}, {{3.90, 0.490}, {4.26, 0.642}}};
    static const double more[2][2][2] = {{{0.95, 0.375}, {1.25, 0.400}}, {{0.95, 0.520}, {1.15, 0.630}}};
    const int r = K % 128 != 0, b = b_exponents;
    const int64_t C = (K + 127) / 128;
    const double it4 = (double)((C + 3) / 4), it2 = (double)((C + 1) / 2), t0 = tiles_of(M, N, 32, 32);
    // (an accumulating round of 128 rows is charged 3 or 5 us, which is also from before: 3520 x 1540 x 1184 with exponents of b 25.0 us in
    // 128 x 192 tiles, 29.1 in the general kernel, which has it)
    const double us[5] = {t0 <= cus ? one[r][b][0] + one[r][b][1] * it4 : 2.2 + rounds_of(t0, cus) * (more[r][b][0] + more[r][b][1] * it4),
                          us_of(cost[0][r][b], tiles_of(M, N, 64, 64), cus, it4), us_of(cost[1][r][b], tiles_of(M, N, 64, 128), cus, it2),
                          us_of(cost[2][r][b], tiles_of(M, N, 128, 128), cus, (double)C, accumulate ? 3.0 : 0.0),
                          us_of(cost[3][r][b], tiles_of(M, N, 128, 192), cus, (double)C, accumulate ? 5.0 : 0.0)};
    MidPlan best{0, us[0]};
    // (128 x 192 is left out where the large tiles can take the problem: they beat it before its loop became a quarter faster.  Since
    // then they do not always: 1333 x 4096 x 11008 69.6 us in half tiles, 62.8 in 128 x 192; 1492 x 3360 x 9344 57.5, 51.1; 2272 x 7712 x
    // 4992 116.0, 95.6; 1499 x 11168 x 3328 83.7, 67.2; but 2048 x 12288 x 4096 105.3, 109.8; 2048 x 4096 x 12288 89.6, 124.7;
    // 8192 x 4096 x 4096 117.0, 160.9.)
    for (int k = 1; k < (large_ok ? 4 : 5); k++)
        if (us[k] < 0.97 * best.us) best = MidPlan{k, us[k]};
    return best;
}

// k_gemm_mx_big, full or half tiles as it chooses them
double us_big(int64_t M, int64_t N, int64_t K, bool b_exponents, double cus)
{
    // [half tiles][K % 128 != 0][exponents of b]
    static const Cost cost[2][2][2] = {{{{8.83, 0.04, 0.832, 0.627}, {16.61, 3.47, 0.888, 0.566}}, {{9.93, 0.04, 0.824, 0.718}, {19.86, 0.0, 0.853, 0.878}}},
                                       {{{3.99, 0.65, 0.605, 0.147}, {5.30, 3.23, 0.667, 0.164}}, {{4.06, 0.05, 0.734, 0.260}, {5.48, 4.20, 0.865, 0.161}}}};
    const bool half = moss_internal_gemm_big_narrow(M, N);
    return us_of(cost[half][K % 128 != 0][b_exponents], tiles_of(M, N, half ? 128 : 256, 256), cus, (double)((K + 127) / 128));
}

// k_gemm: two workgroups run on a compute unit at a time, every stage waits for its own loads, every tile leaves at the
// memory's rate
double us_general(int64_t M, int64_t N, int64_t K, bool b_exponents, double cus)
{
    const double C = (double)((K + 127) / 128), w = tiles_of(M, N, 128, 128) / cus;       // tiles per compute unit
    const double rounds = w <= 2.0 ? 1.0 : std::ceil(w / 2.0), u = w < rounds ? w / rounds : 1.0;
    return b_exponents ? 5.4 + rounds * C * (1.25 + 0.65 * u) + 3.4 * w : 4.6 + rounds * C * (0.96 + 0.6 * u) + 2.2 * w;
}

double model_cus()
{
    const int cus = moss_internal_cu_count();
    return cus <= 0 ? 256 : cus;
}

// The small tiles if they are expected to take at most nine tenths of the time of the kernel that would have the problem
// otherwise (large_ok: k_gemm_mx_big, else k_gemm; three quarters where short K and FP32 outputs make the fits worse, seven
// tenths without exponents of a, which the fits have not seen), kind -1 and that kernel's time if not.
MidPlan plan_small_or_other(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, bool accumulate, bool large_ok)
{
    const double cus = model_cus(), other = large_ok ? us_big(M, N, K, b_e != nullptr, cus) : us_general(M, N, K, b_e != nullptr, cus);
    if (K > ((int64_t)1 << 22) || ((uintptr_t)a_e & 3) || ((uintptr_t)b_e & 3)) return MidPlan{-1, other};     // (32-bit offsets inside a tile)
    const MidPlan plan = plan_mid(M, N, K, b_e != nullptr, accumulate, large_ok, cus);
    const double margin = !a_e && plan.kind >= 3 ? 0.7 : b_e && plan.kind >= 3 && !large_ok && K <= 640 ? 0.75 : 0.9;
    return plan.us > margin * other ? MidPlan{-1, other} : plan;
}

}  // namespace

// The kind of tiles (0 .. 4), -1 to leave the problem to the kernel that would have it otherwise.  Over the 2200 problems, with the
// kernels as they were when fitted, the ones that this and the rule below choose took 0.5 % more than the fastest of each
// problem (mean).  With the kernels as they are now it is 1.3 % over 2000 other problems.
int moss_internal_gemm_mid_kind(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, int accumulate,
                                bool large_ok)
{
    return plan_small_or_other(M, N, K, a_e, b_e, accumulate != 0, large_ok).kind;
}

// Whether k_gemm_mx_big takes a problem with K % 128 != 0 from the kernel that has it by the rule above: where it is
// expected to be a fourteenth faster (a fifth for a short K with exponents of b, as above).  4096 x 4096 x 2080 66 -> 41 us, 11328 x 3520 x
// 2080 175 -> 105, 4160 x 4480 x 9824 287 -> 223, 2432 x 6016 x 2656 with exponents of b 105 -> 56.
bool moss_internal_gemm_big_ragged(int64_t M, int64_t N, int64_t K, const uint8_t *a_e, const uint8_t *b_e, int accumulate,
                                   int64_t ld_out)
{
    if (!moss_internal_gemm_big_ragged_ok(M, N, K, a_e, b_e, ld_out)) return false;
    const double other = plan_small_or_other(M, N, K, a_e, b_e, accumulate != 0, false).us;
    return us_big(M, N, K, b_e != nullptr, model_cus()) < (b_e && K < 1000 ? 0.8 : 0.93) * other;
}

int moss_internal_gemm_mid(int kind, int64_t M, int64_t N, int64_t K, const uint8_t *a_q, const uint8_t *a_e, const float *a_s,
                           const uint8_t *b_q, const uint8_t *b_e, const float *b_s, void *out, int out_f32, int64_t ld_out,
                           int accumulate, hipStream_t st)
{
    using namespace moss;
    MidArgs p{};
    p.M = M; p.N = N; p.K = K;
    p.a_q = a_q; p.a_e = a_e; p.a_s = a_s;
    p.b_q = b_q; p.b_e = b_e; p.b_s = b_s;
    p.out = out; p.ld_out = ld_out; p.out_f32 = out_f32; p.accumulate = accumulate;
    p.e_dwords = K % 128 == 0;
    switch (kind) {
        case 0: return launch_mid<1, 1, 1, 1, 4, 2>(p, 80 * 1024, st);       // two workgroups fit a compute unit
        case 1: return launch_mid<2, 2, 1, 1, 4, 2>(p, 160 * 1024, st);
        case 2: return launch_mid<2, 2, 1, 2, 2, 3>(p, 160 * 1024, st);
        case 3: return launch_mid<2, 2, 2, 2, 1, 4>(p, 160 * 1024, st);
        default: return launch_mid<2, 3, 2, 2, 1, 3>(p, 160 * 1024, st);
    }
}
