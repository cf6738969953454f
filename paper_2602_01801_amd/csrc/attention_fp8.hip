// Block-sparse attention over an 8-bit floating-point copy of the cache (E4M3 keys and values; Sec. 5.1, quantised
// search, and the appendix ablation on quantisation precision, applied to the attention itself), head dimension 128,
// blocks of 128 queries and 64 keys, and the kernel that keeps that copy up to date.
//
// Layout of the copy (per head): K8 [Cp, 128] bytes, rows as in K; V8T [Cp / 64, 128, 64] bytes, the values of every
// block of 64 slots transposed (Cp = C rounded up to a multiple of 64).  A selected key block is then two contiguous
// pieces of 8 KB, both products read their LDS operands with plain 16-byte loads (no transposing loads), and one
// matrix instruction (32x32x64, 8-bit floating-point operands) covers all 64 keys of a tile in the PV product:
//   S^T = K Q^T    A = 32 keys x 64 coordinates from LDS, B = the wavefront's 32 queries in registers (E4M3);
//                  key (32g + 16kb + 4q + e) sits in A row (8q + 4g + e) of half kb, so that a lane's 32 scores are
//                  the keys 32g .. 32g+31 in the order the next product wants them;
//   O^T = V^T P^T  A = 32 value coordinates x 64 keys from LDS, B = P rounded to E4M3, straight from the score registers;
//   l = 1^T P^T    the row sums, by a matrix instruction (16x16x128) on an operand of ones: numerator and denominator see
//                  the same rounded P, so the output stays a convex combination of the stored values.
// Softmax arithmetic as in the bf16 kernels: scores start from the keys' bias (log2 of the multiplicity, -inf for
// dead slots), exponent in one fma, lazily updated reference maximum.  E4M3 spans 2^-9 .. 448, so P is kept near the
// top of that range: P = 2^6 * exp2(score - reference) with the reference at most 2 octaves behind the running
// maximum (P <= 2^8); weights more than about 15 octaves below the row maximum fall out of the format and are dropped
// (the factor 2^6 cancels in O / l and is taken out of lse).
#include <type_traits>

#include <algorithm>

#include "common.hpp"

namespace fastar {

namespace f8 {

constexpr int D = 128;
constexpr int TK = 64;             // keys per tile = slots per block
constexpr int TILEB = TK * D;      // 8 KiB per tile and tensor
constexpr float LN2 = 0.6931471805599453f;
constexpr float F8_MAX = 448.0f;

typedef __attribute__((ext_vector_type(8))) int i32x8;
#define LDS_PTR8(T, p) ((__attribute__((address_space(3))) T *)(p))

// chunk (16 bytes) swizzles inside a tile, applied to the global address a lane fetches and to the LDS address it
// reads: 16 lanes of one operand read then hit 16 different 16-byte slots of a 256-byte bank line
__device__ __forceinline__ int sw_k(int row) { return ((row >> 1) & 1) | (((row >> 2) & 1) << 1) | (((row >> 5) & 1) << 2); }
__device__ __forceinline__ int sw_v(int row) { return (row >> 2) & 3; }

__device__ __forceinline__ unsigned pack_fp8x4(float a, float b, float c, float d) {
    int w = (int)__float_as_uint(a);   // both halves are written; a register that ends here anyway saves clearing one
    w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
    return (unsigned)w;
}
__device__ __forceinline__ float clamp_f8(float x) { return fminf(fmaxf(x, -F8_MAX), F8_MAX); }

// ---- the 8-bit copy of the cache ------------------------------------------------------------------------------
// A block of 64 slots that holds no live slot stamped >= stamp_lo is left alone; any other is rewritten whole: live slots with
// the codes of the stored rows, dead slots with zero.  What bounds it: the rows that are rewritten, and on a long cache, of
// which a frame leaves most alone, the starting of workgroups.  A workgroup looks at PER blocks, gridDim.x apart so that a run of
// slots that one frame wrote is spread over many, and rewrites its own one after the other.
template <bool BF16, int PER>
__global__ __launch_bounds__(256) void kv_to_fp8_kernel(const void *__restrict__ K, const void *__restrict__ V,
                                                        const int32_t *__restrict__ stamp, const int32_t *__restrict__ len,
                                                        int C, int n_blk, int stamp_lo, uint8_t *__restrict__ K8,
                                                        uint8_t *__restrict__ V8T) {
    __shared__ __attribute__((aligned(16))) uint8_t vt[D][TK + 16];   // transposed values of the block (padded rows)
    __shared__ unsigned dirty_of[4];                                   // per wavefront: its blocks that are to be rewritten
    const int h = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int L = min(len[h], C);
    if constexpr (PER == 1) {   // the first wavefront looks; the others, and most workgroups, are done at the barrier
        if (tid == 0) dirty_of[0] = 0u;
        __syncthreads();
        if (tid < TK) {
            const int slot = blockIdx.x * TK + tid;
            if (slot < L && stamp[(size_t)h * C + slot] >= stamp_lo) dirty_of[0] = 1u;
        }
    } else {
        constexpr int EACH = (PER + 3) / 4;   // a wavefront looks at blocks 4 e + wave of the workgroup's
        int st[EACH];
        bool live[EACH];
#pragma unroll
        for (int e = 0; e < EACH; ++e) {
            const int64_t slot = ((int64_t)blockIdx.x + (int64_t)(4 * e + wave) * gridDim.x) * TK + lane;
            live[e] = 4 * e + wave < PER && slot < L;
            st[e] = live[e] ? stamp[(size_t)h * C + slot] : INT_MIN;
        }
        unsigned mine = 0;
#pragma unroll
        for (int e = 0; e < EACH; ++e)
            if (__ballot(live[e] && st[e] >= stamp_lo)) mine |= 1u << (4 * e + wave);
        if (lane == 0) dirty_of[wave] = mine;
    }
    __syncthreads();
    for (unsigned dirty = PER == 1 ? dirty_of[0] : dirty_of[0] | dirty_of[1] | dirty_of[2] | dirty_of[3]; dirty; dirty &= dirty - 1u) {
        const int blk = PER == 1 ? (int)blockIdx.x : (int)blockIdx.x + (__ffs(dirty) - 1) * (int)gridDim.x;   // uniform
        const int j = tid >> 2, part = tid & 3;   // slot of the block, quarter of its row (32 coordinates)
        const int slot = blk * TK + j;
        const size_t Cp = (size_t)n_blk * TK;
        unsigned kw[8], vw[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) kw[w] = vw[w] = 0u;
        if (slot < L) {
            float kf[32], vf[32];
            if (BF16) {
                const unsigned short *kr = (const unsigned short *)K + ((size_t)h * C + slot) * D + 32 * part;
                const unsigned short *vr = (const unsigned short *)V + ((size_t)h * C + slot) * D + 32 * part;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32x4 a = *(const u32x4 *)(kr + 8 * q), b = *(const u32x4 *)(vr + 8 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        kf[8 * q + 2 * e] = bf16_lo(a[e]); kf[8 * q + 2 * e + 1] = bf16_hi(a[e]);
                        vf[8 * q + 2 * e] = bf16_lo(b[e]); vf[8 * q + 2 * e + 1] = bf16_hi(b[e]);
                    }
                }
            } else {
                const float *kr = (const float *)K + ((size_t)h * C + slot) * D + 32 * part;
                const float *vr = (const float *)V + ((size_t)h * C + slot) * D + 32 * part;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const f32x4 a = *(const f32x4 *)(kr + 4 * q), b = *(const f32x4 *)(vr + 4 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) { kf[4 * q + e] = a[e]; vf[4 * q + e] = b[e]; }
                }
            }
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                kw[w] = pack_fp8x4(clamp_f8(kf[4 * w]), clamp_f8(kf[4 * w + 1]), clamp_f8(kf[4 * w + 2]), clamp_f8(kf[4 * w + 3]));
                vw[w] = pack_fp8x4(clamp_f8(vf[4 * w]), clamp_f8(vf[4 * w + 1]), clamp_f8(vf[4 * w + 2]), clamp_f8(vf[4 * w + 3]));
            }
        }
        {
            uint8_t *dst = K8 + ((size_t)h * Cp + slot) * D + 32 * part;
            u32x4 lo = {kw[0], kw[1], kw[2], kw[3]}, hi = {kw[4], kw[5], kw[6], kw[7]};
            *(u32x4 *)dst = lo;
            *(u32x4 *)(dst + 16) = hi;
        }
#pragma unroll
        for (int w = 0; w < 8; ++w)
#pragma unroll
            for (int b = 0; b < 4; ++b) vt[32 * part + 4 * w + b][j] = (uint8_t)(vw[w] >> (8 * b));
        __syncthreads();
        {
            // 128 rows of 64 bytes: thread -> row tid/2, half tid%2 (32 bytes)
            const int row = tid >> 1, half = tid & 1;
            uint8_t *dst = V8T + (((size_t)h * n_blk + blk) * D + row) * TK + 32 * half;
            *(u32x4 *)dst = *(const u32x4 *)(&vt[row][32 * half]);
            *(u32x4 *)(dst + 16) = *(const u32x4 *)(&vt[row][32 * half + 16]);
        }
        if constexpr (PER == 1) return;
        __syncthreads();   // vt has been read
    }
}

// ---- attention ------------------------------------------------------------------------------------------------
// What bounds it: on a cache that L2 serves, the issue of one wavefront (per tile 9 matrix instructions, 33 exponentials, about
// 100 other vector instructions, 27 LDS reads and 50 scalar ones, one after the other: 1.0 us for a workgroup alone on a
// compute unit), which other wavefronts of the SIMD overlap; on a long cache, HBM.  So the kernel is held to 168 registers
// and three workgroups share a compute unit (two with 241 registers: 2.13 us per tile and three blocks, three: 1.77; gathered
// from a cache of 184320 slots x 32 heads 2.42 -> 2.12, 5.9 TB/s).  That takes what a lane keeps down to the accumulators,
// Q and half a dozen offsets: row sums from a 16x16x128 product (four accumulators, not sixteen), tile addresses in scalar
// registers, one copy of the loop's body (unrolled over the stages it spilt).  Launch at 40 heads x 3600 queries x 360 blocks of
// a 230400-slot cache 1.28 -> 1.13 ms.  Tiles in flight alone were not what it waited for: two workgroups per unit with three
// tiles each on their way instead of one took the same 1.29 ms; two each is what LDS leaves to three workgroups.
constexpr int NST = 3;                                        // stages of one K and one V tile
constexpr int LIST = 512;                                     // entries of the selection list held in LDS (a ring of two halves)
constexpr int OSTR = D + 8;                                   // bf16 elements per staged output row
constexpr int STAGE_BYTES = NST * 2 * TILEB;
constexpr int OUT_BYTES = 4 * 32 * OSTR * 2;                  // output staging of the four wavefronts
constexpr int LIST_OFF = OUT_BYTES > STAGE_BYTES ? OUT_BYTES : STAGE_BYTES;
constexpr int CNT_OFF = LIST_OFF + LIST * 4;                  // multiplicities as loaded, a row of TK per tile in flight
constexpr int BIAS_OFF = CNT_OFF + NST * TK * 4;              // log2 of them in units of raw scores, -inf when dead: two rows
constexpr int LDS_BYTES = BIAS_OFF + 2 * TK * 4;
static_assert(3 * LDS_BYTES <= 160 * 1024, "three workgroups per compute unit");

// Workgroup barrier that leaves the tile loads in flight (the fence of __syncthreads may drain them).
__device__ __forceinline__ void wg_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ i32x8 lds_read_32(const unsigned char *p0, const unsigned char *p1) {
    const i32x4 lo = *(const i32x4 *)p0, hi = *(const i32x4 *)p1;
    i32x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return r;
}
__device__ __forceinline__ f32x16 mfma_f8(i32x8 a, i32x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);   // both operands E4M3, no scales
}
__device__ __forceinline__ f32x4 mfma_row_sums(i32x8 ones, i32x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ones, b, c, 4, 0, 0, 0, 0, 0);   // E2M1 times E4M3, no scales
}
// max(x[l], x[l ^ 32]) on the vector ALU (the lane-swap instruction), without a trip through the LDS queue
__device__ __forceinline__ float max_across_halves(float x) {
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Query block b of head h over the entries t_begin <= t < t_end of its list (one entry = one tile).  part == nullptr:
// normalised output rows and lse are written (the range must then be the whole list).  part != nullptr: the unnormalised
// O^T accumulators ([wave][32-row block of d][register / 4][lane] of four), then the reference maxima and the row sums
// ([wave][lane] each): the fragment layout that the combination launch of the split bf16 kernel reads.
// All 256 threads of a workgroup; may be called again by the same workgroup for another block.
__device__ __forceinline__ void attend_item_fp8(
    const unsigned short *__restrict__ Q, const uint8_t *__restrict__ K8, const uint8_t *__restrict__ V8T,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int n_blk, int n_sel, int n_qb, float scale_log2,
    float inv_scale_log2, unsigned short *__restrict__ O, float *__restrict__ lse, unsigned char *lds, int h, int b,
    int t_begin, int t_end, float *__restrict__ part) {
    unsigned char *kbuf = lds;
    unsigned char *vbuf = lds + NST * TILEB;
    int *list = (int *)(lds + LIST_OFF);
    int *cnt_in = (int *)(lds + CNT_OFF);
    float *bias = (float *)(lds + BIAS_OFF);
    // opaque here and again at the end: the compiler would keep per-lane values of the epilogue, and of the loop over blocks
    // around this function, in registers through the loop over the tiles, and spill
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int L = min(len[h], C);
    const int n_live_blk = (L + TK - 1) / TK;
    const int nt_all = L > 0 ? min(nsel[(size_t)h * n_qb + b], n_sel) : 0;   // one selection entry = one tile
    const int nt = max(0, min(nt_all, t_end) - t_begin);                     // tiles of this call: entries t_begin .. t_begin + nt - 1
    const int32_t *sel_row = sel + ((size_t)h * n_qb + b) * n_sel + t_begin;
    const int32_t *cnt_h = cnt ? cnt + (size_t)h * C : nullptr;
    const uint8_t *Kh = K8 + (size_t)h * n_blk * TK * D;
    const uint8_t *Vh = V8T + (size_t)h * n_blk * TILEB;

    // queries of this wavefront as the B operand of the score product: lane (query col, half g) holds coordinates
    // 64s + 32g .. +31 of k-step s, rounded to E4M3
    const int q_idx = b * 128 + wave * 32 + col;
    i32x8 qf[2];
    {
        const unsigned short *qrow = Q + ((size_t)h * n_q + min(q_idx, n_q - 1)) * D;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const u32x4 w = *(const u32x4 *)(qrow + 64 * s + 32 * g + 8 * q);
                qf[s][2 * q] = (int)pack_fp8x4(clamp_f8(bf16_lo(w[0])), clamp_f8(bf16_hi(w[0])), clamp_f8(bf16_lo(w[1])),
                                               clamp_f8(bf16_hi(w[1])));
                qf[s][2 * q + 1] = (int)pack_fp8x4(clamp_f8(bf16_lo(w[2])), clamp_f8(bf16_hi(w[2])), clamp_f8(bf16_lo(w[3])),
                                                   clamp_f8(bf16_hi(w[3])));
            }
        }
    }
    f32x16 o_acc[D / 32];
    f32x4 l_acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) o_acc[db][v] = 0.0f;
    // The row sums come from a 16x16x128 product on the same P registers.  Lane l's weights (query l % 32, half l / 32 of the
    // keys) are there the k-slots 16 (l / 16) .. +15 and 64 + 16 (l / 16) .. +15 of column l % 16, so that queries below 16 own
    // the even sixteens of k and the others the odd ones.  Row i of the other operand is 1 on the sixteens of parity
    // (i / 4) % 2 and 0 on the others; lane l's first accumulator (row 4 (l / 16), column l % 16) is then the sum of query
    // l % 32.  That operand is in 4-bit floating point, whose lanes hold 32 k-slots in order: four registers.
    const bool odd16 = (lane >> 2) & 1;
    const int one_even = odd16 ? 0 : 0x22222222, one_odd = odd16 ? 0x22222222 : 0;
    i32x8 ones = {one_even, one_even, one_odd, one_odd, 0, 0, 0, 0};
    float m_ref = -INFINITY, neg_ms = 0.0f;
    constexpr float P_OFF = 6.0f;                  // P = 2^P_OFF * exp2(score - reference)
    const float tau_raw = 2.0f * inv_scale_log2;   // the reference may lag the true maximum by 2 octaves: P <= 2^8

    // Direct global -> LDS loads of one tile: eight 1-KiB instructions per tensor, two per wavefront.  The second of the two
    // reads and writes 1 KiB further on (its rows have the same swizzle), which the instruction's offset does for both.
    const unsigned ksrc = (8 * 2 * wave + (lane >> 3)) * D + (((lane & 7) ^ sw_k(16 * wave + (lane >> 3))) << 4);
    const unsigned vsrc = (16 * 2 * wave + (lane >> 2)) * TK + (((lane & 3) ^ sw_v(lane >> 2)) << 4);
    auto issue_loads = [&](int blk, int stage) {
        const uint8_t *kt = Kh + (size_t)blk * TILEB;   // uniform
        const uint8_t *vt = Vh + (size_t)blk * TILEB;
        unsigned char *kd = kbuf + stage * TILEB + wave * 2048, *vd = vbuf + stage * TILEB + wave * 2048;
        // buffer instructions: the tile's address stays in scalar registers, a lane adds its 32-bit offset
        const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void *)kt, 0, TILEB, 0x00020000);
        const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void *)vt, 0, TILEB, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, LDS_PTR8(unsigned, kd), 16, ksrc, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, LDS_PTR8(unsigned, kd), 16, ksrc, 0, 1024, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, LDS_PTR8(unsigned, vd), 16, vsrc, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, LDS_PTR8(unsigned, vd), 16, vsrc, 0, 1024, 0);
    };
    // the list by way of LDS, half a ring at a time: the block to load, or -1 (loads block 0, which is live, fully masked)
    auto load_list = [&](int from) {   // from: a multiple of LIST / 2
        static_assert(LIST / 2 == 256, "one entry per thread");
        if (from + tid < nt) {
            const int kb = sel_row[from + tid];
            list[(from + tid) % LIST] = kb >= 0 && kb < n_live_blk ? kb : -1;
        }
    };
    auto entry = [&](int tile) -> int { return __builtin_amdgcn_readfirstlane(list[tile % LIST]); };   // uniform
    // The first wavefront keeps the bias rows: multiplicities are loaded one tile ahead of the tile itself, straight to LDS,
    // and turned into the bias of a tile while the tile before it is worked on.
    const bool counts = wave == 0 && cnt_h != nullptr;   // uniform over the wavefront
    auto issue_counts = [&](int tile, int kb) {
        const int key = min(max(kb, 0) * TK + lane, L - 1);
        __builtin_amdgcn_global_load_lds(cnt_h + key, LDS_PTR8(unsigned, cnt_in + (tile % NST) * TK), 4, 0, 0);
    };
    auto fill_bias = [&](int tile, int kb, int n) {   // wavefront 0; n: the multiplicity read from cnt_in
        const bool live = kb >= 0 && lane < L - kb * TK;
        const float v = cnt_h ? __log2f((float)n) * inv_scale_log2 : 0.0f;
        bias[(tile & 1) * TK + lane] = live ? v : -INFINITY;
    };
    // Waits until this wavefront's share of tile t has landed (in the first: the multiplicities of tile t + 1, asked for
    // right behind it, too).  Loads complete in order; behind these there are NST - 2 tiles of four loads in flight, with one
    // load of multiplicities each, unless the list ends before.
    auto wait_tile = [&](bool ends) {   // ends: fewer than NST - 1 tiles are behind tile t
        constexpr int NEWER = 4 * (NST - 2), NEWER0 = 5 * (NST - 2);
        static_assert(NEWER0 < 16, "the counter's low bits alone");
        if (ends) __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
        else if (counts) __builtin_amdgcn_s_waitcnt(0x0F70 | NEWER0);
        else __builtin_amdgcn_s_waitcnt(0x0F70 | NEWER);
        asm volatile("" ::: "memory");
    };
    int kb_of[NST] = {};   // entries of tiles t + 1 .. t + NST (uniform)
    if (nt > 0) {
        load_list(0);
        __builtin_amdgcn_s_waitcnt(0x0F70);   // the counts in wait_tile start from nothing in flight
        __syncthreads();
        if (counts) issue_counts(0, entry(0));
#pragma unroll
        for (int i = 0; i < NST - 1; ++i) {
            if (i < nt) issue_loads(max(entry(i), 0), i);
            if (i + 1 < nt && counts) issue_counts(i + 1, entry(i + 1));
        }
#pragma unroll
        for (int i = 1; i < NST; ++i) kb_of[i - 1] = entry(min(i, nt - 1));
        wait_tile(NST - 1 >= nt);
        if (wave == 0) fill_bias(0, entry(0), cnt_in[lane]);
    }
    // Per-lane LDS offsets of the operand reads (tile-independent).  Rows 16 (K, second half of the keys) and 32 (V, next block
    // of coordinates) further on have the same swizzle, so everything but the 16-byte chunk is a constant on top.
    const int krow = 32 * ((col >> 2) & 1) + 4 * (col >> 3) + (col & 3);
    const unsigned koff = krow * D + (((2 * g) ^ sw_k(krow)) << 4);   // k-step s, second chunk: ^ 64 s, ^ 16
    const unsigned voff = col * TK + (((2 * g) ^ sw_v(col)) << 4);    // second chunk: ^ 16

    int stage = 0;
    for (int t = 0; t < nt; ++t) {
        wait_tile(t + NST - 1 >= nt);
        wg_barrier();   // everyone's share has landed, bias row t is written, tile t-1 is fully consumed
        const int stage_behind = stage == 0 ? NST - 1 : stage - 1;
        if (t + NST - 1 < nt) issue_loads(max(kb_of[NST - 2], 0), stage_behind);
        const int cnt_next = cnt_in[(stage == NST - 1 ? 0 : stage + 1) * TK + lane];   // wavefront 0 alone uses it
        if (t + NST < nt && (t + NST) % (LIST / 2) == 0) {   // half a ring of the list; its other half is still in use
            load_list(t + NST);
            __syncthreads();
        }
        const float *bt = bias + (t & 1) * TK;
        const unsigned ka0 = koff + stage * TILEB, va0 = voff + stage * TILEB;
        // The reads of an operand are issued well before its product (the scheduling fences keep them there): a wavefront
        // waits about 130 cycles for a read that it has just issued.
        // Scores start from the keys' bias: register 4q+e of half kb is key 32g + 16kb + 4q + e.
        f32x16 s_acc[2];
        auto read_bias = [&](int kb) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 bv = *(const f32x4 *)(&bt[32 * g + 16 * kb + 4 * q4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) s_acc[kb][4 * q4 + e] = bv[e];
            }
        };
        auto k_operand = [&](int kb, int s) {
            return lds_read_32(kbuf + (ka0 ^ (64u * s)) + 16 * kb * D, kbuf + (ka0 ^ (64u * s) ^ 16u) + 16 * kb * D);
        };
        auto v_operand = [&](int db) { return lds_read_32(vbuf + va0 + 32 * db * TK, vbuf + (va0 ^ 16u) + 32 * db * TK); };
        i32x8 ka[2][2], va[D / 32];
        read_bias(0);
        ka[0][0] = k_operand(0, 0);
        ka[0][1] = k_operand(0, 1);
        ka[1][0] = k_operand(1, 0);
        __builtin_amdgcn_sched_barrier(0);
        s_acc[0] = mfma_f8(ka[0][0], qf[0], s_acc[0]);
        read_bias(1);
        ka[1][1] = k_operand(1, 1);
        __builtin_amdgcn_sched_barrier(0);
        s_acc[0] = mfma_f8(ka[0][1], qf[1], s_acc[0]);
        s_acc[1] = mfma_f8(ka[1][0], qf[0], s_acc[1]);
        s_acc[1] = mfma_f8(ka[1][1], qf[1], s_acc[1]);
        const int kb_raw = list[(t + NST) % LIST];   // not used beyond the end of the list
        constexpr int VE = 1, VM = 1;   // blocks of V^T read before the row maximum, and after half of the weights
#pragma unroll
        for (int db = 0; db < VE; ++db) va[db] = v_operand(db);
        __builtin_amdgcn_sched_barrier(0);
        float mx = s_acc[0][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s_acc[0][v]);
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s_acc[1][v]);
        mx = max_across_halves(mx);
        if (__any(mx > m_ref + tau_raw)) {   // wave-uniform
            const float m_new = fmaxf(m_ref, mx);
            const float alpha = m_ref == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_ref - m_new) * scale_log2);
            m_ref = m_new;
            neg_ms = m_new == -INFINITY ? 0.0f : P_OFF - m_new * scale_log2;
            l_acc[0] *= alpha;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o_acc[db][v] *= alpha;
        }
        i32x8 pf;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                float p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(s_acc[kb][4 * q4 + e], scale_log2, neg_ms));
                pf[4 * kb + q4] = (int)pack_fp8x4(p[0], p[1], p[2], p[3]);
            }
            if (kb == 0) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int db = VE; db < VE + VM; ++db) va[db] = v_operand(db);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int db = VE + VM; db < D / 32; ++db) va[db] = v_operand(db);
        kb_of[NST - 1] = __builtin_amdgcn_readfirstlane(kb_raw);
        l_acc = mfma_row_sums(ones, pf, l_acc);
#pragma unroll
        for (int db = 0; db < D / 32; ++db) o_acc[db] = mfma_f8(va[db], pf, o_acc[db]);
        if (wave == 0) {   // multiplicities that were asked for with the tile before t + 1 (see wait_tile)
            if (t + 1 < nt) fill_bias(t + 1, kb_of[0], cnt_next);
            if (t + NST < nt && counts) issue_counts(t + NST, kb_of[NST - 1]);
        }
#pragma unroll
        for (int i = 0; i + 1 < NST; ++i) kb_of[i] = kb_of[i + 1];
        stage = stage == NST - 1 ? 0 : stage + 1;
    }

    int etid = threadIdx.x;
    asm volatile("" : "+v"(etid));
    const int elane = etid & 63, ecol = elane & 31, eg = elane >> 5, e_idx = b * 128 + wave * 32 + ecol;
    const float l_tot = l_acc[0];
    if (part) {   // a fragment: the combination launch normalises
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 w = {o_acc[db][4 * q4], o_acc[db][4 * q4 + 1], o_acc[db][4 * q4 + 2], o_acc[db][4 * q4 + 3]};
                ((f32x4 *)part)[((wave * (D / 32) + db) * 4 + q4) * 64 + elane] = w;
            }
        part[4 * ATTN_PART_O_FLOATS + wave * 64 + elane] = m_ref;
        part[4 * ATTN_PART_O_FLOATS + 4 * 64 + wave * 64 + elane] = l_tot;
        __syncthreads();   // the tile stages and the bookkeeping are free for the next block
        return;
    }
    // epilogue: normalise, transpose through LDS, store rows coalesced
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    __syncthreads();
    unsigned short *Os = (unsigned short *)lds + (size_t)wave * 32 * OSTR;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(o_acc[db][4 * q4 + e] * inv);
            *(bf16x4 *)(Os + ecol * OSTR + 32 * db + 8 * q4 + 4 * eg) = w;
        }
    __syncthreads();
    {
        const int rr = elane >> 4, cc = elane & 15;
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int r = it * 4 + rr;
            const int qi = b * 128 + wave * 32 + r;
            if (qi < n_q) *(u32x4 *)(O + ((size_t)h * n_q + qi) * D + cc * 8) = *(const u32x4 *)(Os + r * OSTR + cc * 8);
        }
    }
    if (lse && eg == 0 && e_idx < n_q)
        lse[(size_t)h * n_q + e_idx] = l_tot > 0.0f ? (m_ref * scale_log2 - 6.0f + __log2f(l_tot)) * LN2 : -INFINITY;
    __syncthreads();   // the staged output rows have been read: the tile stages are free for the next block
}

// One query block per workgroup; three workgroups per CU, started as slots free up.
__global__ __launch_bounds__(256, 3) void attn_fp8_d128_kernel(
    const unsigned short *__restrict__ Q, const uint8_t *__restrict__ K8, const uint8_t *__restrict__ V8T,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int n_blk, int n_sel, int n_qb, int H, float scale_log2,
    float inv_scale_log2, unsigned short *__restrict__ O, float *__restrict__ lse) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    // workgroup -> (head, query block): each XCD gets a contiguous range of (head, block) pairs
    const int total = n_qb * H;
    const int wg = blockIdx.x;
    const int per = (total + 7) / 8;
    const int item = (wg & 7) * per + (wg >> 3);
    if (item >= total) return;
    attend_item_fp8(Q, K8, V8T, cnt, len, sel, nsel, n_q, C, n_blk, n_sel, n_qb, scale_log2, inv_scale_log2, O, lse, lds,
                    item / n_qb, item % n_qb, 0, INT_MAX, nullptr);
}

// The split launch (see the bf16 kernel of the same structure in attention_d128.hip): the first n_plain workgroups take one
// whole query block each, in the plain kernel's order; the others take equal shares of the tiles of the blocks left over.
__global__ __launch_bounds__(256, 3) void attn_fp8_d128_sk_kernel(
    const unsigned short *__restrict__ Q, const uint8_t *__restrict__ K8, const uint8_t *__restrict__ V8T,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int n_blk, int n_sel, int n_qb, TailMap tm, int n_plain, int NT,
    float scale_log2, float inv_scale_log2, unsigned short *__restrict__ O, float *__restrict__ lse, float *__restrict__ ws) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int P = (int)gridDim.x - n_plain;                        // a multiple of 8
    const int wg = (int)blockIdx.x - n_plain;
    const int i = (wg & 7) * (P >> 3) + (wg >> 3);                 // neighbouring shares on one XCD: those of its own range
    const int direct = wg < 0 ? ((int)blockIdx.x & 7) * tm.per + ((int)blockIdx.x >> 3) : -1;
    const long long W = tm.tiles(NT);
    long long v = wg < 0 ? 0 : i * W / P;
    const long long v_end = wg < 0 ? NT : (i + 1) * W / P;
    while (v < v_end) {
        const int vi = (int)(v / NT);
        const int t_begin = (int)(v - (long long)vi * NT);
        const int t_end = (int)min((long long)NT, v_end - (long long)vi * NT);
        const int item = direct >= 0 ? direct : tm.item(vi);
        if (item < tm.total) {   // uniform over the workgroup
            float *part = nullptr;
            if (t_begin > 0 || t_end < NT) part = ws + ((size_t)i * 2 + (t_begin > 0 ? 0 : 1)) * ATTN_PART_FLOATS;
            attend_item_fp8(Q, K8, V8T, cnt, len, sel, nsel, n_q, C, n_blk, n_sel, n_qb, scale_log2, inv_scale_log2, O, lse,
                            lds, item / n_qb, item % n_qb, t_begin, t_end, part);
        }
        v = (long long)vi * NT + t_end;
    }
}

// Few query blocks: n_parts workgroups per block, each an equal run of its entries, which leave fragments for
// attn_combine_parts_kernel (attention_d128.hip).
__global__ __launch_bounds__(256, 3) void attn_fp8_d128_parts_kernel(
    const unsigned short *__restrict__ Q, const uint8_t *__restrict__ K8, const uint8_t *__restrict__ V8T,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int n_blk, int n_sel, int n_qb, int H, int n_parts, float scale_log2,
    float inv_scale_log2, float *__restrict__ frag) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int units = n_qb * H * n_parts, per = (units + 7) / 8;
    const int unit = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);   // neighbouring units on one XCD
    if (unit >= units) return;
    const int item = unit / n_parts, part = unit - item * n_parts;
    const int n_listed = min(nsel[item], n_sel);
    const int tb = (int)((long long)n_listed * part / n_parts), te = (int)((long long)n_listed * (part + 1) / n_parts);
    attend_item_fp8(Q, K8, V8T, cnt, len, sel, nsel, n_q, C, n_blk, n_sel, n_qb, scale_log2, inv_scale_log2, nullptr, nullptr,
                    lds, item / n_qb, item % n_qb, tb, te, frag + (size_t)unit * ATTN_PART_FLOATS);
}

// Whether a launch of n_items pairs with n_tiles tiles each is split, and how many pairs per XCD range are taken whole then
// (0: not split).  An XCD holds 96 of these workgroups.  Us per launch, lists from a cache of 37440 slots (pairs per XCD;
// unsplit / 64 or a multiple taken whole / 96 or a multiple):
//   up to 96 a single round, which the split can only make fuller: 65 of 90 tiles 162 / 211 (230400 slots 183 / 272), of 180
//     304 / 325; 70 of 90 164 / 171, of 180 311 / 295, of 360 602 / 537; 93 of 180 341 / 381;
//   98 of 90 tiles 239 / 219 / 251, of 135 345 / 297 / 334, of 360 877 / 717 / 737; 109 of 135 350 / 333 / 303; 125 of 135
//     358 / 392 / 365, of 360 906 / 1007 / 908; 132 of 90 281 / 300 / 275, of 180 537 / 525 / 483, of 360 1041 / 971 / 930;
//   145 of 90 288 / 301 / 311, of 180 548 / 558 / 541, of 360 1072 / 992 / 1059; 240 of 135 651 / 689 / 680.
static int split_full_per(int n_items, int n_tiles) {
    const int per_xcd = (n_items + 7) / 8, tail96 = per_xcd % 96, tail64 = per_xcd % 64;
    if (per_xcd > 96 && tail96 > 0 && ((tail96 <= 24 && n_tiles >= 120) || (tail96 <= 40 && n_tiles >= 150))) return per_xcd - tail96;
    if (per_xcd > 64 && tail64 >= 5 && tail64 <= 24 && n_tiles >= 150) return per_xcd - tail64;
    return 0;
}

}  // namespace f8

int attn_fp8_setup() {
    static DeviceOnce once;
    return once.run([](int) {
        return hipFuncSetAttribute((const void *)f8::attn_fp8_d128_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   f8::LDS_BYTES) == hipSuccess &&
                       hipFuncSetAttribute((const void *)f8::attn_fp8_d128_sk_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, f8::LDS_BYTES) == hipSuccess &&
                       hipFuncSetAttribute((const void *)f8::attn_fp8_d128_parts_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, f8::LDS_BYTES) == hipSuccess
                   ? FASTAR_OK
                   : FASTAR_ERR_HIP;
    });
}

}  // namespace fastar

using namespace fastar;

extern "C" int fastar_kv_to_fp8(const fastar_cache *cache, int32_t stamp_lo, uint8_t *K8, uint8_t *V8T, void *stream) {
    if (!cache || !K8 || !V8T) return FASTAR_ERR_INVALID_ARG;
    if (!cache->K || !cache->V || !cache->stamp || !cache->len) return FASTAR_ERR_INVALID_ARG;
    const int H = cache->H, C = cache->C;
    if (H <= 0 || C <= 0) return FASTAR_ERR_INVALID_ARG;
    if (cache->dtype != FASTAR_F32 && cache->dtype != FASTAR_BF16) return FASTAR_ERR_INVALID_ARG;
    if (cache->d != 128) return FASTAR_ERR_UNSUPPORTED;
    if (((uintptr_t)cache->K & 15) || ((uintptr_t)cache->V & 15) || ((uintptr_t)K8 & 15) || ((uintptr_t)V8T & 15))
        return FASTAR_ERR_INVALID_ARG;
    const int n_blk = (C + f8::TK - 1) / f8::TK;
    // Blocks per workgroup: one while there are few workgroups to start (or all blocks are to be rewritten), then as many as
    // keep the grid at 16384 or more.  Us per call by 1 / 2 / 4 / 8 / 16 blocks after a frame with 4/5 of its tokens merged:
    // 40 heads x 230400 slots (144000 blocks) 136 / 127 / 112 / 106 / 106, 40 x 115200 126 / 126 / 124 / 127 / 127, 40 x 57600
    // 60 / 60 / 57 / 59 / 60, 12 x 37440 13 / 14 / 15 / 17 / 18, 5 x 28000 7 / 8 / 8 / 11 / 11; all blocks of 40 x 230400
    // 1265 / 1280 / 1303 / 1329 / 1350, of 5 x 28000 18 / 19 / 22 / 25 / 32.
    const int64_t blocks = (int64_t)n_blk * H;
    const int per = stamp_lo == INT_MIN ? 1 : blocks >= 8 * 16384 ? 8 : blocks >= 4 * 16384 ? 4 : blocks >= 2 * 16384 ? 2 : 1;
#define FASTAR_KV8(BF, PER)                                                                                                 \
    hipLaunchKernelGGL((f8::kv_to_fp8_kernel<BF, PER>), dim3((n_blk + PER - 1) / PER, H), dim3(256), 0, (hipStream_t)stream, \
                       cache->K, cache->V, cache->stamp, cache->len, C, n_blk, stamp_lo, K8, V8T)
#define FASTAR_KV8_PER(BF)                   \
    do {                                     \
        if (per == 8) FASTAR_KV8(BF, 8);     \
        else if (per == 4) FASTAR_KV8(BF, 4); \
        else if (per == 2) FASTAR_KV8(BF, 2); \
        else FASTAR_KV8(BF, 1);              \
    } while (0)
    if (cache->dtype == FASTAR_BF16) FASTAR_KV8_PER(true);
    else FASTAR_KV8_PER(false);
#undef FASTAR_KV8_PER
#undef FASTAR_KV8
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

static int sparse_attn_fp8_impl(const void *Q, int n_q, const uint8_t *K8, const uint8_t *V8T, const int32_t *cnt,
                                const int32_t *len, int H, int C, int d, const int32_t *sel, const int32_t *nsel, int BQ,
                                int BK, int n_sel, float scale, void *O, float *lse, void *ws, void *stream);

extern "C" int sparse_attn_fwd_fp8(const void *Q, int n_q, const uint8_t *K8, const uint8_t *V8T, const int32_t *cnt,
                                   const int32_t *len, int H, int C, int d, const int32_t *sel, const int32_t *nsel,
                                   int BQ, int BK, int n_sel, float scale, void *O, float *lse, void *stream) {
    return sparse_attn_fp8_impl(Q, n_q, K8, V8T, cnt, len, H, C, d, sel, nsel, BQ, BK, n_sel, scale, O, lse, nullptr, stream);
}

extern "C" int sparse_attn_fwd_fp8_ws(const void *Q, int n_q, const uint8_t *K8, const uint8_t *V8T, const int32_t *cnt,
                                      const int32_t *len, int H, int C, int d, const int32_t *sel, const int32_t *nsel,
                                      int BQ, int BK, int n_sel, float scale, void *O, float *lse, void *ws,
                                      size_t ws_bytes, void *stream) {
    if (!ws || ((uintptr_t)ws & 255)) return FASTAR_ERR_INVALID_ARG;
    if (ws_bytes < (size_t)ATTN_SHARE_WORKGROUPS * 2 * ATTN_PART_FLOATS * sizeof(float)) return FASTAR_ERR_WORKSPACE;
    return sparse_attn_fp8_impl(Q, n_q, K8, V8T, cnt, len, H, C, d, sel, nsel, BQ, BK, n_sel, scale, O, lse, ws, stream);
}

static int sparse_attn_fp8_impl(const void *Q, int n_q, const uint8_t *K8, const uint8_t *V8T, const int32_t *cnt,
                                const int32_t *len, int H, int C, int d, const int32_t *sel, const int32_t *nsel, int BQ,
                                int BK, int n_sel, float scale, void *O, float *lse, void *ws, void *stream) {
    if (!Q || !K8 || !V8T || !len || !sel || !nsel || !O) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || C <= 0 || n_sel <= 0) return FASTAR_ERR_INVALID_ARG;
    if (!(scale > 0.0f) || !(scale < INFINITY)) return FASTAR_ERR_INVALID_ARG;
    if (((uintptr_t)Q & 15) || ((uintptr_t)K8 & 15) || ((uintptr_t)V8T & 15) || ((uintptr_t)O & 15))
        return FASTAR_ERR_INVALID_ARG;
    if (d != 128 || BQ != 128 || BK != 64) return FASTAR_ERR_UNSUPPORTED;
    if (const int rc = attn_fp8_setup(); rc != FASTAR_OK) return rc;
    const int n_qb = (n_q + 127) / 128;
    const int n_blk = (C + f8::TK - 1) / f8::TK;
    // |q.k| <= 128 * 448^2 < 2^25: below that least scale a score counts for nothing beside the bias either way
    const float scale_log2 = std::max(scale * 1.4426950408889634f, ATTN_LEAST_SCALE_LOG2);
    // with a workspace, a launch that would end in a short last round of workgroups is split (one entry = one tile)
    const int full_per = ws ? f8::split_full_per(n_qb * H, n_sel) : 0;
    if (full_per > 0) {
        const TailMap tm = {(n_qb * H + 7) / 8, full_per, n_qb * H};
        const int n_plain = 8 * full_per;
        hipLaunchKernelGGL(f8::attn_fp8_d128_sk_kernel, dim3(n_plain + tm.shares(n_sel)), dim3(256), f8::LDS_BYTES,
                           (hipStream_t)stream, (const unsigned short *)Q, K8, V8T, cnt, len, sel, nsel, n_q, C, n_blk,
                           n_sel, n_qb, tm, n_plain, n_sel, scale_log2, 1.0f / scale_log2, (unsigned short *)O, lse,
                           (float *)ws);
        FASTAR_LAUNCH_CHECK();
        return launch_attn_combine(ws, n_q, n_qb, tm, n_sel, scale_log2, -6.0f, O, lse, (hipStream_t)stream);
    }
    // at most one block per compute unit: several workgroups per block where that pays (4 blocks of 96 tiles 97 -> 19 us, 156
    // of 48 tiles 55 -> 41; 156 of 24 tiles 31 either way, of 3 tiles 9: then one workgroup).  Over 1 to 256 blocks of 3 to 192
    // tiles the number chosen is within 2 us or 9 % of the best one.
    const int n_parts = ws && n_qb * H <= 256 ? attn_parts(n_qb * H, n_sel, 1, 0.97f, 1.35f) : 1;
    if (n_parts > 1) {
        const int units = n_qb * H * n_parts;
        hipLaunchKernelGGL(f8::attn_fp8_d128_parts_kernel, dim3((unsigned)(((units + 7) / 8) * 8)), dim3(256), f8::LDS_BYTES,
                           (hipStream_t)stream, (const unsigned short *)Q, K8, V8T, cnt, len, sel, nsel, n_q, C, n_blk,
                           n_sel, n_qb, H, n_parts, scale_log2, 1.0f / scale_log2, (float *)ws);
        FASTAR_LAUNCH_CHECK();
        return launch_attn_combine_parts(ws, n_parts, n_q, n_qb, H, scale_log2, -6.0f, O, lse, (hipStream_t)stream);
    }
    const dim3 grid((unsigned)(((n_qb * H + 7) / 8) * 8));
    hipLaunchKernelGGL(f8::attn_fp8_d128_kernel, grid, dim3(256), f8::LDS_BYTES, (hipStream_t)stream,
                       (const unsigned short *)Q, K8, V8T, cnt, len, sel, nsel, n_q, C, n_blk, n_sel, n_qb, H, scale_log2,
                       1.0f / scale_log2, (unsigned short *)O, lse);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}
