// ANN selection (Sec. 5.1 goal "keys with the largest dot products"; Sec. 5.4 AnnSA; Sec. 5.3 AnnCA).
//
// Three stages, all on exact integer scores so that the selected sets are reproducible bit for bit:
//   rep_kernel          mean codes that summarise each query block (AnnSA only)
//   score_*_kernel      int8 matrix-core scoring of summaries x key codes, reduced on the fly to one
//                       int32 per (query block, key block) [AnnSA] or per (query block, prompt token)
//                       [AnnCA]; HBM-bound: every key code is streamed exactly once
//   topk                exact top-n_sel per row, ties to the lowest index, written in ascending order
//                       (topk_dev.hpp; a kernel of its own for AnnSA, the tail of the scoring kernel for
//                       AnnCA, where one workgroup owns a whole row)
// Short caches: all three in one launch (select_short_kernel).
#include <limits.h>

#include <algorithm>

#include "common.hpp"
#include "topk_dev.hpp"

namespace fastar {

constexpr int KB_PER_WG = 4;      // key blocks scored by one workgroup of score_self_kernel
// Key blocks over all heads from which the streaming kernel pays, by the summaries' column blocks of 32 (it holds four): never for
// up to three and for 64-entry codes, where the other one keeps more wavefronts in flight.  Call, streaming / the other, us:
// 4: 10 heads x 64000 slots (10000) 17.4 / 17.6, 13 x 103000 (20930) 27.9 / 28.6, 20 x 150000 41 / 46, 40 x 150000 62 / 73, 40 x 230400
// 108 / 115; 3: 10 x 64000 18.3 / 16.6, 20 x 150000 41.1 / 39.6, 40 x 110000 (68760) 49.4 / 48.1, 40 x 230400 95.3 / 94.7, 64 x 230400 157 / 146;
// 2: 40 x 230400 88 / 82, 24 x 200000 49.6 / 45.6, 40 x 115200 45 / 41; 64 entries: 4: 10 x 64000 33 / 22, 40 x 110000 95 / 93, 3: 20 x 230400
// 95 / 84, 2: 40 x 115200 86 / 61.
// Codes of 2 and 4 bits keep one line.
constexpr size_t LONG_CACHE_BLOCKS = 16 * 4096, LONG_CACHE_BLOCKS_4 = 20000;
static bool streams(int r, int bits, int n_cb, size_t blocks) {
    if (n_cb > 4 || r != 32) return false;
    if (bits != 8) return blocks >= LONG_CACHE_BLOCKS;
    return n_cb == 4 && blocks >= LONG_CACHE_BLOCKS_4;
}
// Slots per head up to which one workgroup per query block scores them all (select_short_kernel); three launches against
// one, us: r = 32, 2 x 2 query blocks, 4096 slots 9.3 -> 6.6, 9360 9.3 -> 8.9, 12288 9.6 -> 9.3; 12 x 21, 4096 11.1 -> 7.4,
// 9360 11.7 -> 10.2, 12288 11.7 -> 12.2; r = 64, 6 x 21, 1024 11.7 -> 7.0, 4096 11.7 -> 9.3, 8192 11.8 -> 13.1.
constexpr int short_keys(int r) { return r == 32 ? 10240 : 4096; }
// What it reads from beyond L2: the blocks of a head lie on as many XCDs, which fetch the head's codes each (three launches against
// one, us): 8 heads x 32 query blocks x 10240 slots (20 MB) 11.5 -> 10.1, 40 x 3 x 10240 (37 MB) 12.5 -> 11.0, 16 x 16 x 8192
// (32 MB) 10.9 -> 9.5, x 10240 (40 MB) 11.2 -> 12.7, 24 x 8 x 8192 (48 MB) 10.8 -> 12.6, 32 x 8 x 10240 (80 MB) 11.5 -> 16.7.
constexpr int64_t SHORT_BYTES = 38 << 20;
constexpr int SHORT_WGS = 256;     // its workgroups: no more than compute units (a second round: 11 us like the launches it replaces)

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- codes narrower than a byte -----------------------------------------------------------------------
// Codes of BITS (2, 4 or 8) bits per entry, packed from the low end of each byte (appendix, "Quantization precision for
// ANN matching").  Key codes stay packed in memory and are widened in registers, as the matrix operand of one lane half
// (16 entries): an entry is moved to the TOP bits of its byte, i.e. multiplied by 2^(8-BITS) - the same factor on every
// score of a call, so no ranking changes - which needs one shift and one mask per four entries and no sign extension.
// Byte i of output word t then holds entry (8/BITS) * i' + t of its word; the summaries are stored in the same order.
template <int BITS>
__device__ __forceinline__ i32x4 load_key_codes(const int8_t *p) {   // p: the lane half's 16 * BITS / 8 bytes
    i32x4 a;
    if constexpr (BITS == 8) {
        a = *(const i32x4 *)p;
    } else if constexpr (BITS == 4) {
        const u32x2 w = *(const u32x2 *)p;
        a[0] = (int)((w[0] << 4) & 0xF0F0F0F0u);
        a[1] = (int)(w[0] & 0xF0F0F0F0u);
        a[2] = (int)((w[1] << 4) & 0xF0F0F0F0u);
        a[3] = (int)(w[1] & 0xF0F0F0F0u);
    } else {
        const unsigned w = *(const unsigned *)p;
        a[0] = (int)((w << 6) & 0xC0C0C0C0u);
        a[1] = (int)((w << 4) & 0xC0C0C0C0u);
        a[2] = (int)((w << 2) & 0xC0C0C0C0u);
        a[3] = (int)(w & 0xC0C0C0C0u);
    }
    return a;
}
// position, inside its group of 16, at which entry e of a summary is stored so that it meets the widened key entries
template <int BITS>
__device__ __forceinline__ int summary_slot(int e) {
    if constexpr (BITS == 8) return e;
    else if constexpr (BITS == 4) return (e & 8) + ((e & 1) << 2) + ((e & 7) >> 1);
    else return ((e & 3) << 2) + (e >> 2);
}

// ---- query-block summaries ------------------------------------------------------------------------
// rep[h][b*n_rep + u][j] = floor((sum over the u-th run of g queries of block b of qcode[.][j] + g/2) / g)
template <int BITS>
__global__ void rep_kernel(const int8_t *__restrict__ qcode, int n_q, int r, int BQ, int n_rep, int n_qb,
                           int8_t *__restrict__ rep) {
    const int b = blockIdx.x, h = blockIdx.y;
    const int g = BQ / n_rep;
    constexpr int PER = 8 / BITS;
    const int rb = r / PER;   // bytes per query row
    for (int t = threadIdx.x; t < n_rep * r; t += blockDim.x) {
        const int u = t / r, j = t % r;
        const int q0 = b * BQ + u * g;
        const int q1 = min(q0 + g, n_q);
        int s = 0;
        const int8_t *col = qcode + ((size_t)h * n_q + q0) * rb + j / PER;
        const int up = 32 - BITS * (j % PER + 1);   // shift that puts the entry at the top of a word, then arithmetic shift down
        const int n = q1 - q0;
        int q = 0;
        for (; q + 32 <= n; q += 32) {   // the usual run whole: a load costs a microsecond behind the launch that wrote it
            int v[32];
#pragma unroll
            for (int e = 0; e < 32; ++e) v[e] = col[(size_t)(q + e) * rb];
#pragma unroll
            for (int e = 0; e < 32; ++e) s += BITS == 8 ? v[e] : ((int)((unsigned)v[e] << up) >> (32 - BITS));
        }
        for (; q + 8 <= n; q += 8) {   // eight independent loads in flight
            int v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = col[(size_t)(q + e) * rb];
#pragma unroll
            for (int e = 0; e < 8; ++e) s += BITS == 8 ? v[e] : ((int)((unsigned)v[e] << up) >> (32 - BITS));
        }
        for (; q < n; ++q) {
            const int v = col[(size_t)q * rb];
            s += BITS == 8 ? v : ((int)((unsigned)v << up) >> (32 - BITS));
        }
        s += g / 2;
        int m = s / g;
        if (s % g != 0 && s < 0) m -= 1;
        rep[((size_t)h * n_qb * n_rep + (size_t)b * n_rep + u) * r + (j & ~15) + summary_slot<BITS>(j & 15)] = (int8_t)m;
    }
}

// Lane exchanges of the scoring epilogue without a trip through LDS.
__device__ __forceinline__ int max_across_halves_i32(int x) {   // max with lane ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    return max((int)r[0], (int)r[1]);
}
__device__ __forceinline__ int max_over_quad_i32(int x) {       // max over the four lanes 4k .. 4k+3
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    return max(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
}
// max over the n_rep (a power of two up to 32) neighbouring lanes that hold the summaries of one query block
__device__ __forceinline__ int max_over_reps_i32(int x, int n_rep) {
    if (n_rep >= 2) x = max(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
    if (n_rep >= 4) x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
    if (n_rep >= 8) x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false));   // row_half_mirror
    if (n_rep >= 16) x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false));  // row_mirror
    if (n_rep >= 32) x = max(x, shfl_xor(x, 16));
    return x;
}

// ---- AnnSA scoring -----------------------------------------------------------------------------------
// out[h][b][kb] = max over the summaries u of block b (whose run holds a query) and the live keys k of
// key block kb of rep[b,u] . kcode[k].   D = A x B with A rows = 32 keys, B columns = 32 summaries.
// COL_CHUNK: summary column blocks (of 32) per pass; their operands are registers, so it is what the call's equal passes need,
// from two to eight: what bounds the launch is the codes' latency, and it wants wavefronts in flight.  Calls in us, eight at every
// size / as many as the call has: one block of columns, 12 heads x 37440 slots 12.7 / 11.6; three 14.3 / 13.1, 20 x 100000 34.3 / 30.3,
// 64-entry codes 47.8 / 38.8; five 16.6 / 16.0; six 17.7 / 17.5, 40 x 57600 with 64-entry codes 70.3 / 59.3; seven 18.8 / 18.6, 40 x 115200
// with 64-entry codes 158 / 141; twice seven, 12 x 60000 with 64-entry codes 52.3 / 45.9.  Codes of 2 and 4 bits have two, four, five and
// eight: with the others as well, 60 KB more code, the launches of this file took 0.2 to 0.4 us longer (12 x 4680 x 37440).
template <int R, int BITS, int COL_CHUNK>
__global__ __launch_bounds__(256) void score_self_kernel(const int8_t *__restrict__ kcode, const int32_t *__restrict__ len,
                                                         const int8_t *__restrict__ rep, int C, int n_q, int BQ,
                                                         int n_rep, int BK, int n_qb, int n_kb_cap,
                                                         int32_t *__restrict__ out) {
    constexpr int KS = R / 32;
    extern __shared__ int32_t tile[];  // [n_qb][KB_PER_WG]
    const int h = blockIdx.y;
    const int L = min(len[h], C);
    const int n_kb = (L + BK - 1) / BK;
    const int kb0 = blockIdx.x * KB_PER_WG;
    if (kb0 >= n_kb) return;  // whole workgroup beyond the live cache (uniform)
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int col = lane & 31, g2 = lane >> 5;
    const int NR = n_qb * n_rep;
    const int NCB = (NR + 31) / 32;
    const int rep_shift = __ffs(n_rep) - 1;   // n_rep is a power of two
    const int g = BQ >> rep_shift;
    constexpr int RB = R * BITS / 8;   // bytes per key row
    const int8_t *kc = kcode + (size_t)h * C * RB;
    const int8_t *rp = rep + (size_t)h * NR * R;

    for (int cb0 = 0; cb0 < NCB; cb0 += COL_CHUNK) {
        i32x4 bfrag[COL_CHUNK][KS];
#pragma unroll
        for (int c = 0; c < COL_CHUNK; ++c) {
            if (cb0 + c >= NCB) continue;   // uniform
            const int rc = min((cb0 + c) * 32 + col, NR - 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) bfrag[c][ks] = *(const i32x4 *)(rp + (size_t)rc * R + ks * 32 + 16 * g2);
        }
        for (int kl = wave; kl < KB_PER_WG; kl += 4) {
            const int kb = kb0 + kl;
            if (kb >= n_kb) break;
            int best[COL_CHUNK];
#pragma unroll
            for (int c = 0; c < COL_CHUNK; ++c) best[c] = INT_MIN;
            // two groups of 32 keys per round: both loads are issued before the first product waits
            for (int sg0 = 0; sg0 < BK; sg0 += 64) {
                if (kb * BK + sg0 >= L) break;
                i32x4 afrag[2][KS];
                bool have[2], partial[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int sg = sg0 + 32 * q;
                    const int kbase = kb * BK + sg;
                    have[q] = sg < BK && kbase < L;
                    partial[q] = kbase + 32 > L || sg + 32 > BK;
                    const int krow = min(kbase + col, C - 1);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        i32x4 a = {0, 0, 0, 0};
                        if (have[q]) a = load_key_codes<BITS>(kc + (size_t)krow * RB + (ks * 32 + 16 * g2) * BITS / 8);
                        afrag[q][ks] = a;
                    }
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (!have[q]) continue;   // uniform
                    const int sg = sg0 + 32 * q;
                    const int kbase = kb * BK + sg;
#pragma unroll
                    for (int c = 0; c < COL_CHUNK; ++c) {
                        if (cb0 + c < NCB) {
                            i32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                            for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(afrag[q][ks], bfrag[c][ks], acc);
                            int m = best[c];
                            if (partial[q]) {
#pragma unroll
                                for (int v = 0; v < 16; ++v) {
                                    const int kloc = 8 * (v >> 2) + 4 * g2 + (v & 3);
                                    if (kbase + kloc < L && sg + kloc < BK) m = max(m, acc[v]);
                                }
                            } else {
#pragma unroll
                                for (int v = 0; v < 16; ++v) m = max(m, acc[v]);
                            }
                            best[c] = m;
                        }
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < COL_CHUNK; ++c) {
                if (cb0 + c < NCB) {
                    int m = max_across_halves_i32(best[c]);
                    const int rc = (cb0 + c) * 32 + col;
                    const int b = rc >> rep_shift, u = rc & (n_rep - 1);
                    if (rc >= NR || b * BQ + u * g >= n_q) m = INT_MIN;
                    m = max_over_reps_i32(m, n_rep);
                    if (g2 == 0 && u == 0 && rc < NR) tile[b * KB_PER_WG + kl] = m;
                }
            }
        }
    }
    __syncthreads();
    const int n_here = min(KB_PER_WG, n_kb - kb0);
    for (int t = threadIdx.x; t < n_qb * KB_PER_WG; t += blockDim.x) {
        const int b = t / KB_PER_WG, kl = t % KB_PER_WG;
        if (kl < n_here) out[((size_t)h * n_qb + b) * n_kb_cap + kb0 + kl] = tile[t];
    }
}

// The same scores for long caches.  What bounds this kernel is how the memory system is addressed: workgroups that
// each own a contiguous run of key blocks read at large, equal strides from each other and reach only about
// 2.8 TB/s on this chip, whatever they compute; workgroups that together sweep a dense window reach 5 TB/s and more.
// So the grid walks the head's key blocks in steps: in step s workgroup x takes blocks 4(sG + x) .. +3, one per
// wavefront, G = gridDim.x; a wavefront keeps the codes of its next three rounds in flight while it scores the current
// one (four operand buffers in an unrolled rotation: copying a buffer would wait for its loads) and writes its block's
// scores straight to the rows of the score matrix.  CC: summary column blocks (of 32) kept in registers at a time.
template <int R, int CC, int BITS>
__global__ __launch_bounds__(256, 3) void score_self_stream_kernel(const int8_t *__restrict__ kcode, const int32_t *__restrict__ len,
                                                         const int8_t *__restrict__ rep, int C, int n_q, int BQ,
                                                         int n_rep, int BK, int n_qb, int n_kb_cap,
                                                         int32_t *__restrict__ out) {
    constexpr int KS = R / 32;
    constexpr int RB = R * BITS / 8;   // bytes per key row
    const int h = blockIdx.y;
    const int L = min(len[h], C);
    const int n_kb = (L + BK - 1) / BK;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, kept in a scalar register
    const int col = lane & 31, g2 = lane >> 5;
    const int NR = n_qb * n_rep;
    const int NCB = (NR + 31) / 32;
    const int g = BQ / n_rep;
    const int rep_shift = __ffs(n_rep) - 1;   // n_rep is a power of two
    const int8_t *kc = kcode + (size_t)h * C * RB;
    const int8_t *rp = rep + (size_t)h * NR * R;
    const int first = blockIdx.x * 4 + wave;          // this wavefront's first key block
    const int stride = gridDim.x * 4;                 // ... and the distance to its next one
    if (first >= n_kb) return;                        // nothing for this wavefront (no barrier follows)
    // rounds of 64 keys (two groups of 32): key block first + stride * (it / rpk), keys 64 * (it % rpk) .. of it
    const int rpk = (BK + 63) / 64;
    const int n_it = ((n_kb - first + stride - 1) / stride) * rpk;
    auto load_round = [&](int it, i32x4 (&a)[2][KS]) __attribute__((always_inline)) {
        it = min(it, n_it - 1);   // rounds past the wavefront's share re-read its last one (cache hits), never other blocks
        const int kb = first + stride * (it / rpk), sg0 = 64 * (it % rpk);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int sg = sg0 + 32 * q;
            const int kbase = kb * BK + sg;
            // always loaded, from a clamped row: the number of loads in flight is then the same on every path and
            // the compiler can wait for exactly the buffer it needs; rows past the block or the cache are never scored
            const int krow = min(kbase + col, C - 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[q][ks] = load_key_codes<BITS>(kc + (size_t)krow * RB + (ks * 32 + 16 * g2) * BITS / 8);
        }
    };

    for (int cb0 = 0; cb0 < NCB; cb0 += CC) {
        i32x4 bfrag[CC][KS];
#pragma unroll
        for (int c = 0; c < CC; ++c) {
            const int rc = min((cb0 + c) * 32 + col, NR - 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) bfrag[c][ks] = *(const i32x4 *)(rp + (size_t)rc * R + ks * 32 + 16 * g2);
        }
        int best[CC];
        // what this lane's summary column of every column block stands for: its score row and whether it is the
        // block's first summary; columns past the summaries or of a run without a query never count
        int32_t *col_out[CC];
        bool col_ok[CC], col_first[CC];
#pragma unroll
        for (int c = 0; c < CC; ++c) {
            const int rc = (cb0 + c) * 32 + col;
            const int b = rc >> rep_shift;
            const int u = rc & (n_rep - 1);
            col_ok[c] = rc < NR && b * BQ + u * g < n_q;
            col_first[c] = rc < NR && u == 0 && g2 == 0;
            col_out[c] = out + ((size_t)h * n_qb + min(b, n_qb - 1)) * n_kb_cap;
        }
        const bool full_cols = cb0 + CC <= NCB;
        auto score_round = [&](int it, const i32x4 (&cur)[2][KS]) __attribute__((always_inline)) {
            if (it >= n_it) return;   // uniform
            const int kb = first + stride * (it / rpk), sg0 = 64 * (it % rpk);
            if (sg0 == 0) {
#pragma unroll
                for (int c = 0; c < CC; ++c) best[c] = INT_MIN;
            }
            if (full_cols && kb * BK + sg0 + 64 <= L && sg0 + 64 <= BK) {
                // the common round, straight line: 64 live keys, every column block in use
#pragma unroll
                for (int c = 0; c < CC; ++c) {
                    i32x16 acc0 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                    i32x16 acc1 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        acc0 = mfma_i8_32x32x32(cur[0][ks], bfrag[c][ks], acc0);
                        acc1 = mfma_i8_32x32x32(cur[1][ks], bfrag[c][ks], acc1);
                    }
                    int m = best[c];
#pragma unroll
                    for (int v = 0; v < 16; ++v) m = max(max(m, acc0[v]), acc1[v]);   // one three-operand maximum each
                    best[c] = m;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int sg = sg0 + 32 * q;
                    const int kbase = kb * BK + sg;
                    if (!(sg < BK && kbase < L)) continue;   // uniform
                    const bool partial = kbase + 32 > L || sg + 32 > BK;
#pragma unroll
                    for (int c = 0; c < CC; ++c) {
                        if (cb0 + c < NCB) {
                            i32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                            for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(cur[q][ks], bfrag[c][ks], acc);
                            int m = best[c];
                            if (partial) {
#pragma unroll
                                for (int v = 0; v < 16; ++v) {
                                    const int kloc = 8 * (v >> 2) + 4 * g2 + (v & 3);
                                    if (kbase + kloc < L && sg + kloc < BK) m = max(m, acc[v]);
                                }
                            } else {
#pragma unroll
                                for (int v = 0; v < 16; ++v) m = max(m, acc[v]);
                            }
                            best[c] = m;
                        }
                    }
                }
            }
            if (it % rpk == rpk - 1) {   // the key block is complete
#pragma unroll
                for (int c = 0; c < CC; ++c) {
                    if (cb0 + c < NCB) {
                        int m = max_across_halves_i32(best[c]);
                        if (!col_ok[c]) m = INT_MIN;
                        if (n_rep == 4) m = max_over_quad_i32(m);   // uniform
                        else for (int off = 1; off < n_rep; off <<= 1) m = max(m, shfl_xor(m, off));
                        if (col_first[c]) col_out[c][kb] = m;
                    }
                }
            }
        };
        i32x4 b0[2][KS], b1[2][KS], b2[2][KS], b3[2][KS];
        load_round(0, b0);
        load_round(1, b1);
        load_round(2, b2);
        for (int it = 0; it < n_it; it += 4) {
            load_round(it + 3, b3);
            score_round(it, b0);
            load_round(it + 4, b0);
            score_round(it + 1, b1);
            load_round(it + 5, b1);
            score_round(it + 2, b2);
            load_round(it + 6, b2);
            score_round(it + 3, b3);
        }
    }
}

// ---- AnnCA scoring -----------------------------------------------------------------------------------
// score[p] = max over the queries q of block b of qcode[q] . pcode[p], kept in LDS, then the top n_sel of the row.
// D = A x B with A rows = 32 queries, B columns = 32 prompt tokens.

// Maximum of m and the 16 results, three levels deep.
__device__ __forceinline__ int max_of_16(int m, const i32x16 &a) {
    const int t0 = max(max(a[0], a[1]), a[2]), t1 = max(max(a[3], a[4]), a[5]), t2 = max(max(a[6], a[7]), a[8]);
    const int t3 = max(max(a[9], a[10]), a[11]), t4 = max(max(a[12], a[13]), a[14]);
    return max(max(m, max(max(t0, t1), a[15])), max(max(t2, t3), t4));
}

// smax[p] = max over the queries of block b of qcode[q] . pcode[p], for all n_p prompt tokens; whole workgroup.
// A wavefront takes every fourth group of 32 prompt tokens against all queries, 128 at a time: a token's codes are read once
// and its maximum over four products stays in registers, without atomics.  (Every wavefront a quarter of the queries
// against all tokens, maxima met in LDS: 5.4 us for 128 queries x 512 tokens, 13.6 x 2048; 3.9 and 8.0 this way.)
// What bounds it is the issue of the wavefront: a product's result is there 64 cycles after it was asked for, so the next product
// is under way while the maxima of one are taken, without branches between them (one after the other, each waited for: launch
// for 2 x 256 queries x 2048 tokens 8.5 us, now 7.4; 1 x 128 x 12000 68.7, 60.7).
// in_flight() is called once, behind the first loads: what it asks for does not hold the scores up (loads come back in order).
// Queries q0 .. q_end (at most 32 QG; rows beyond repeat the last one, which changes no maximum) against all tokens.
template <int R, int QG, typename F>
__device__ __forceinline__ void score_cross_queries(const int8_t *__restrict__ qc, const int8_t *__restrict__ pc, int n_p, int q0,
                                                    int q_end, bool first, int32_t *smax, F &&in_flight) {
    constexpr int KS = R / 32;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, g2 = lane >> 5;
    const int n_groups = (n_p + 31) / 32;
    constexpr int PB = 4;   // groups of tokens in flight: the codes of a group four further on replace those just used
    i32x4 afrag[QG][KS], bfrag[PB][KS];
    auto load = [&](int u, int group) {
        const int prow = min(group * 32 + col, n_p - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bfrag[u][ks] = *(const i32x4 *)(pc + (size_t)prow * R + ks * 32 + 16 * g2);
    };
#pragma unroll
    for (int u = 0; u < QG; ++u) {
        const int qrow = min(q0 + 32 * u + col, q_end - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) afrag[u][ks] = *(const i32x4 *)(qc + (size_t)qrow * R + ks * 32 + 16 * g2);
    }
#pragma unroll
    for (int u = 0; u < PB; ++u) load(u, wave + 4 * u);
    __builtin_amdgcn_sched_barrier(0);
    in_flight();
    __builtin_amdgcn_sched_barrier(0);
    auto product = [&](int qg, int u) {
        i32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(afrag[qg][ks], bfrag[u][ks], acc);
        return acc;
    };
    i32x16 acc[2];
    // the tokens of slot u; leaves the first product of slot `next` under way
    auto score = [&](int u, int next, int group) {
        static_assert(QG % 2 == 0, "two sets of results in turn");
        const int p = group * 32 + col;
        int m = INT_MIN;
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
            acc[(qg + 1) & 1] = qg + 1 < QG ? product(qg + 1, u) : product(0, next);
            __builtin_amdgcn_sched_barrier(0);
            m = max_of_16(m, acc[qg & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        const auto halves = __builtin_amdgcn_permlane32_swap((unsigned)m, (unsigned)m, false, false);
        m = max((int)halves[0], (int)halves[1]);
        if (g2 == 0 && p < n_p) smax[p] = first ? m : max(smax[p], m);   // the same lane every time
    };
    acc[0] = product(0, 0);
    int t0 = wave;
    for (; t0 + 4 * PB < n_groups; t0 += 4 * PB) {
#pragma unroll
        for (int u = 0; u < PB; ++u) {   // whole groups of four: t0 + 4 u + 4 < n_groups
            score(u, (u + 1) % PB, t0 + 4 * u);
            load(u, t0 + 4 * (PB + u));
        }
    }
#pragma unroll
    for (int u = 0; u < PB; ++u) {
        if (t0 + 4 * u >= n_groups) break;   // uniform
        score(u, (u + 1) % PB, t0 + 4 * u);
    }
}

template <int R>
__global__ __launch_bounds__(256) void score_cross_kernel(const int8_t *__restrict__ qcode, const int8_t *__restrict__ pcode,
                                                          int n_q, int n_p, int BQ, int n_qb, int n_sel,
                                                          int32_t *__restrict__ sel, int32_t *__restrict__ nsel) {
    extern __shared__ int32_t smax[];  // [n_p]
    __shared__ __attribute__((aligned(16))) unsigned scratch[TOPK_SCRATCH];
    const int b = blockIdx.x, h = blockIdx.y;
    const int8_t *qc = qcode + (size_t)h * n_q * R, *pc = pcode + (size_t)h * n_p * R;
    const int q_end = min((b + 1) * BQ, n_q);
    for (int q0 = b * BQ; q0 < q_end; q0 += 128) {   // uniform
        if (q_end - q0 > 64) score_cross_queries<R, 4>(qc, pc, n_p, q0, q_end, q0 == b * BQ, smax, [] {});
        else score_cross_queries<R, 2>(qc, pc, n_p, q0, q_end, q0 == b * BQ, smax, [] {});
    }
    __syncthreads();
    // the workgroup owns the whole row: select from LDS right away
    topk_row(smax, n_p, n_sel, sel + ((size_t)h * n_qb + b) * n_sel, nsel + (size_t)h * n_qb + b, nullptr, scratch);
}

// ---- AnnCA in one launch: selection and the attention over it (bf16, d = 128, blocks of 128 queries, up to 64 tokens) --
// One workgroup = one query block: scores and exact top-n_sel as above (the list also goes to sel / nsel), then the
// selected prompt rows are gathered into LDS once and the four wavefronts (32 queries each) attend to them:
// S^T = K Q^T, softmax over the at most 64 tokens in one piece (no running maximum), O^T = V^T P^T.  V is stored
// in rows like K and transposed by the LDS reads, which take the tokens of each 16 in the order the score accumulators hold
// them, so that the accumulators, converted to bf16, are the second product's operand as they are.
namespace fused {
constexpr int D = 128, TK = 64;
constexpr int KROW = D * 2 + 16;          // bytes per staged K row (padded: 16 consecutive rows hit 16 different bank groups)
constexpr int VROW = D * 2 + 64;          // bytes per staged V row (the four rows of a transposing read lie in different quarters of the banks)
constexpr int TILE_BYTES = TK * KROW + TK * VROW;
static_assert(TOPK_SCRATCH * 4 <= TILE_BYTES, "the selection's scratch does, too");
__host__ __device__ inline size_t lds_bytes(int n_p) { return ((size_t)n_p * 4 + 15) / 16 * 16 + TK * 4 + 16 + TILE_BYTES; }
}  // namespace fused

template <int R>
__global__ __launch_bounds__(256) void cross_fused_kernel(const unsigned short *__restrict__ Q, const int8_t *__restrict__ qcode,
                                                          const unsigned short *__restrict__ Kp,
                                                          const unsigned short *__restrict__ Vp,
                                                          const int8_t *__restrict__ pcode, int n_q, int n_p, int n_qb,
                                                          int n_sel, float scale_log2, int32_t *__restrict__ sel,
                                                          int32_t *__restrict__ nsel, unsigned short *__restrict__ O) {
    using namespace fused;
    extern __shared__ __attribute__((aligned(16))) unsigned char flds[];
    int32_t *smax = (int32_t *)flds;
    int32_t *lsel = (int32_t *)(flds + ((size_t)n_p * 4 + 15) / 16 * 16);   // [TK] selected tokens, ascending
    int32_t *lcnt = lsel + TK;                                              // [1] how many
    unsigned char *ktile = (unsigned char *)(lcnt + 4);
    unsigned char *vtile = ktile + TK * KROW;
    const int b = blockIdx.x, h = blockIdx.y;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int col = lane & 31, g = lane >> 5;
    // this lane's query row as the second operand of K Q^T: in flight during the scoring and the selection
    const int q_idx = b * 128 + wave * 32 + col;
    bf16x8 qf[D / 16];
    score_cross_queries<R, 4>(qcode + (size_t)h * n_q * R, pcode + (size_t)h * n_p * R, n_p, b * 128, min((b + 1) * 128, n_q), true, smax, [&] {
        const unsigned short *qrow = Q + ((size_t)h * n_q + min(q_idx, n_q - 1)) * D;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) qf[s] = *(const bf16x8 *)(qrow + 16 * s + 8 * g);
    });
    __syncthreads();
    topk_row(smax, n_p, n_sel, lsel, lcnt, nullptr, (unsigned *)ktile);   // the tile's memory is free until the gather
    __syncthreads();
    const int k = __builtin_amdgcn_readfirstlane(lcnt[0]);
    if (tid < n_sel) sel[((size_t)h * n_qb + b) * n_sel + tid] = lsel[tid];
    if (tid == 0) nsel[(size_t)h * n_qb + b] = k;
    // gather: slot p of the tiles holds the rows of token lsel[p], zeros from k to the end of the last block of 32 in use
    const unsigned short *Kh = Kp + (size_t)h * n_p * D, *Vh = Vp + (size_t)h * n_p * D;
    const bool two = k > 32;   // uniform
    {
        u32x4 kv[4], vv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (16 * e >= k) break;   // uniform
            const int idx = e * 256 + tid, p = idx >> 4, c = idx & 15;
            const int tok = p < k ? lsel[p] : 0;
            kv[e] = *(const u32x4 *)(Kh + (size_t)tok * D + 8 * c);
            vv[e] = *(const u32x4 *)(Vh + (size_t)tok * D + 8 * c);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (e >= 2 && !two) break;   // uniform
            const int idx = e * 256 + tid, p = idx >> 4, c = idx & 15;
            if (16 * e + 16 > k) {   // uniform
                const u32x4 none = {0u, 0u, 0u, 0u};
                kv[e] = p < k ? kv[e] : none;
                vv[e] = p < k ? vv[e] : none;
            }
            *(u32x4 *)(ktile + p * KROW + c * 16) = kv[e];
            *(u32x4 *)(vtile + p * VROW + c * 16) = vv[e];
        }
    }
    __syncthreads();
    // S^T = K Q^T: rows = token slots (two blocks of 32, the second where there are so many), columns = this wavefront's 32 queries.
    // Softmax over the k live slots in one piece: register v of block kb is slot 32 kb + 8 (v / 4) + 4 g + v % 4.
    f32x16 s_acc[2];
    auto scores = [&](int kb) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s_acc[kb][v] = 0.0f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            const bf16x8 a = *(const bf16x8 *)(ktile + (32 * kb + col) * KROW + (16 * s + 8 * g) * 2);
            s_acc[kb] = mfma_bf16_32x32x16(a, qf[s], s_acc[kb]);
        }
    };
    auto mask = [&](int kb) {
        if (k >= 32 * kb + 32) return;   // uniform
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (32 * kb + 8 * (v >> 2) + 4 * g + (v & 3) >= k) s_acc[kb][v] = -INFINITY;
    };
    scores(0);
    if (two) scores(1);
    mask(0);
    float mx = s_acc[0][0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s_acc[0][v]);
    if (two) {
        mask(1);
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s_acc[1][v]);
    }
    {
        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
    }
    const float neg_ms = mx == -INFINITY ? 0.0f : -mx * scale_log2;
    float l = 0.0f;
    f32x16 o_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o_acc[db][v] = 0.0f;
    // O^T += V^T P^T of one block: rows = 32 of the d coordinates per block, columns = queries
    auto weigh = [&](int kb) {
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            bf16x8 pf;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                pf[j] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s_acc[kb][8 * st + j], scale_log2, neg_ms));
                l += (float)pf[j];   // the sum takes the rounded P, the values the second product sees
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
                // tokens in the order the score accumulators hold them: 4 g .. + 3 and 8 + 4 g .. + 3 of the 16; lane i of 16
                // gets coordinate i of the four rows that the lanes 4 j + q address
                const unsigned char *vp = vtile + (32 * kb + 16 * st + 4 * g + ((lane & 15) >> 2)) * VROW +
                                          (32 * db + (lane & 16) + 4 * (lane & 3)) * 2;
                const bf16x4 lo = ds_read_tr16(vp), hi = ds_read_tr16(vp + 8 * VROW);
                const bf16x8 a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                o_acc[db] = mfma_bf16_32x32x16(a, pf, o_acc[db]);
            }
        }
    };
    weigh(0);
    if (two) weigh(1);
    {
        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        l = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
    }
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    // A lane holds four of every eight coordinates of its query; the halves of the wavefront trade theirs, so that a lane has
    // eight neighbours for one store.  (By way of LDS, for whole rows: 1.5 us, with the rounding in software.)
    if (q_idx < n_q) {
        unsigned short *orow = O + ((size_t)h * n_q + q_idx) * D + 8 * g;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                unsigned x[2], y[2];
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    x[w] = cvt_bf16x2(o_acc[db][8 * a + 2 * w] * inv, o_acc[db][8 * a + 2 * w + 1] * inv);
                    y[w] = cvt_bf16x2(o_acc[db][8 * a + 4 + 2 * w] * inv, o_acc[db][8 * a + 4 + 2 * w + 1] * inv);
                }
                u32x4 o;
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const auto t = __builtin_amdgcn_permlane32_swap(x[w], y[w], false, false);
                    o[w] = t[0];
                    o[2 + w] = t[1];
                }
                *(u32x4 *)(orow + 32 * db + 16 * a) = o;
            }
    }
}

// Row (h, b) of `score` holds n entries (n = ceil(len[h]/BK) when len is given, else n_fixed).  ALONE: rows of up to
// TOPK_WAVE_MAX entries, a wavefront each; otherwise four.
template <bool ALONE>
__global__ __launch_bounds__(ALONE ? 64 : 256) void topk_kernel(const int32_t *__restrict__ score, int row_stride,
                                                   const int32_t *__restrict__ len, int len_cap, int BK, int n_fixed,
                                                   int n_qb, int n_sel, int32_t *__restrict__ sel,
                                                   int32_t *__restrict__ nsel, int n_sink, int n_local, int cand_min) {
    // staging of the row's keys: min(row_stride, TOPK_LDS_CAP) words of dynamic LDS (a static array of the full size
    // would hold the kernel to four workgroups per compute unit whatever the row length)
    extern __shared__ unsigned keys[];
    const int b = blockIdx.x, h = blockIdx.y;
    int n = n_fixed;
    if (len) n = (min(len[h], len_cap) + BK - 1) / BK;
    n = min(n, row_stride);
    const int32_t *row = score + ((size_t)h * n_qb + b) * row_stride;
    int32_t *out = sel + ((size_t)h * n_qb + b) * n_sel, *n_out = nsel + (size_t)h * n_qb + b;
    if constexpr (ALONE) {
        __shared__ __attribute__((aligned(16))) unsigned hist[TOPK_WAVE_BINS];
        topk_row_wave<TOPK_WAVE_MAX>(row, n, n_sel, out, n_out, hist, n_sink, n_local, cand_min);
    } else {
        __shared__ __attribute__((aligned(16))) unsigned scratch[TOPK_SCRATCH];
        topk_row(row, n, n_sel, out, n_out, keys, scratch, n_sink, n_local, cand_min);
    }
}

static void launch_topk(const int32_t *score, int n_kb_cap, const int32_t *len, int C, int BK, int n_qb, int H, int n_sel, int32_t *sel,
                        int32_t *nsel, int n_sink, int n_local, int cand_min, hipStream_t s) {
    const dim3 grid(n_qb, H);
    if (n_kb_cap <= TOPK_WAVE_MAX)
        hipLaunchKernelGGL(topk_kernel<true>, grid, dim3(64), 0, s, score, n_kb_cap, len, C, BK, 0, n_qb, n_sel, sel, nsel, n_sink,
                           n_local, cand_min);
    else
        hipLaunchKernelGGL(topk_kernel<false>, grid, dim3(256), (size_t)std::min(n_kb_cap, TOPK_LDS_CAP) * 4, s, score, n_kb_cap, len, C,
                           BK, 0, n_qb, n_sel, sel, nsel, n_sink, n_local, cand_min);
}

// ---- AnnSA selection in one launch, short caches -------------------------------------------------------
// One workgroup = one query block: its summaries, the scores of every live key block and the top-k of the row, which
// never leaves LDS.  The summaries are the rows of the products (row i: summary i mod n_rep, so eight rows hold them all)
// and the keys the columns, so a lane keeps four of its sixteen results.  Nothing is masked: a run without queries is
// replaced by the block's first one, and keys beyond the live ones by the last of them, which lies in the same key block.
// What bounds it: a chain of latencies (keys and queries, summaries, a round of keys per 4096 of them, top-k) in place of
// three launches; 4 heads x 780 queries x 4096 slots 9.9 -> 6.9 us, x 9360 10.2 -> 9.3; 5.2 and 8.3 since the sums of the summaries
// are split over lanes and one wavefront selects.
constexpr int SHORT_THREADS = 1024;
constexpr int SHORT_BLOCKS = 512;   // key blocks: at least 32 slots each
static_assert(SHORT_BLOCKS * 32 >= short_keys(32) && SHORT_BLOCKS * 32 >= short_keys(64), "one wavefront selects from the row");
template <int R>
__global__ __launch_bounds__(SHORT_THREADS) void select_short_kernel(
    const int8_t *__restrict__ qcode, int n_q, const int8_t *__restrict__ kcode, const int32_t *__restrict__ len, int C, int BQ,
    int n_rep, int BK, int n_qb, int n_kb_cap, int n_sel, int32_t *__restrict__ sel, int32_t *__restrict__ nsel, int n_sink,
    int n_local) {
    constexpr int KS = R / 32, WAVES = SHORT_THREADS / 64;
    constexpr int KB = R == 32 ? 4 : 2;   // key blocks in flight per wavefront (four rows of 64 bytes: 16 registers spilled)
    extern __shared__ __attribute__((aligned(16))) unsigned char slds[];
    int32_t *smax = (int32_t *)slds;                              // [n_kb_cap]
    unsigned *qrow = (unsigned *)(slds + ((size_t)n_kb_cap * 4 + 15) / 16 * 16);   // [BQ][R] bytes
    __shared__ __attribute__((aligned(16))) int8_t srep[8 * R];
    __shared__ __attribute__((aligned(16))) unsigned hist[TOPK_WAVE_BINS];
    const int b = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g2 = lane >> 5;
    const int g = BQ / n_rep;
    const int q_lo = b * BQ, n_here = min(BQ, n_q - q_lo);
    const unsigned *qc = (const unsigned *)(qcode + ((size_t)h * n_q + q_lo) * R);
    for (int t = tid; t < n_here * (R / 4); t += SHORT_THREADS) qrow[t] = qc[t];
    const int L = min(len[h], C);
    const int n_kb = (L + BK - 1) / BK;
    const int8_t *kc = kcode + (size_t)h * C * R;
    i32x4 kf[KB][2][KS];
    // two groups of 32 keys of each of the wavefront's next key blocks; the last group again where there is no second one
    auto load = [&](int kb0, int sg0) {
#pragma unroll
        for (int q = 0; q < KB; ++q)
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int k = min((kb0 + q * WAVES) * BK + min(sg0 + 32 * w, BK - 32) + col, L - 1);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) kf[q][w][ks] = *(const i32x4 *)(kc + (size_t)k * R + ks * 32 + 16 * g2);
            }
    };
    if (wave < n_kb) load(wave, 0);
    __syncthreads();
    // As rep_kernel, eight neighbouring lanes a sum (32 reads one after the other took 1.0 to 1.7 us).
    const bool pow2 = (g & (g - 1)) == 0;   // uniform
    const int g_shift = 31 - __clz(g);
    for (int t0 = 0; t0 < n_rep * R * 8; t0 += SHORT_THREADS) {   // n_rep * R * 8 is a multiple of 256: whole wavefronts
        const int t = (t0 + tid) >> 3, part = tid & 7;
        if (t >= n_rep * R) break;
        const int u = t / R, j = t % R;
        const int q0 = u * g, q1 = min(q0 + g, n_here);
        const int8_t *qb = (const int8_t *)qrow + j;
        int s = 0, q = q0 + part;
        for (; q + 24 < q1; q += 32) s += (qb[q * R] + qb[(q + 8) * R]) + (qb[(q + 16) * R] + qb[(q + 24) * R]);
        for (; q < q1; q += 8) s += qb[q * R];
        s += (int)lane_of_eight<0>((unsigned)s);
        s += (int)lane_of_eight<1>((unsigned)s);
        s += (int)lane_of_eight<2>((unsigned)s);
        s += g / 2;
        int m;   // floor(s / g)
        if (pow2) {
            m = s >> g_shift;
        } else {
            m = s / g;
            if (s % g != 0 && s < 0) m -= 1;
        }
        if (part == 0) srep[t] = (int8_t)m;
    }
    __syncthreads();
    int u = col & (n_rep - 1);
    if (u * g >= n_here) u = 0;
    i32x4 rf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rf[ks] = *(const i32x4 *)(srep + u * R + ks * 32 + 16 * g2);
    constexpr int BIAS = 1 << 21;   // |score| <= 64 * 127 * 127
    for (int kb0 = wave; kb0 < n_kb; kb0 += KB * WAVES) {
        int best[KB];
#pragma unroll
        for (int q = 0; q < KB; ++q) best[q] = INT_MIN;
        for (int sg0 = 0; sg0 < BK; sg0 += 64) {
            if (kb0 != wave || sg0 != 0) load(kb0, sg0);
#pragma unroll
            for (int q = 0; q < KB; ++q)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    i32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(rf[ks], kf[q][w][ks], acc);
#pragma unroll
                    for (int v = 0; v < 4; ++v) best[q] = max(best[q], acc[v]);   // rows 4 g2 + v
                }
        }
#pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int m = (int)wave_max_last((unsigned)(best[q] + BIAS)) - BIAS;
            if (lane == 63 && kb0 + q * WAVES < n_kb) smax[kb0 + q * WAVES] = m;
        }
    }
    __syncthreads();
    if (wave > 0) return;
    topk_row_wave<SHORT_BLOCKS>(smax, n_kb, n_sel, sel + ((size_t)h * n_qb + b) * n_sel, nsel + (size_t)h * n_qb + b, hist, n_sink,
                                n_local);
}

// ---- selection on sign codes (LSH family) -------------------------------------------------------------
// Summaries: bit j of the summary of a run of g queries = majority of the run's bits (2 * ones >= queries).
// One workgroup per (query block, head), one thread per hash bit of a run, as many runs at a time as fit the workgroup
// (one at a time: 7.5 us for 12 x 4680 queries of 128 bits, now 4.8); a wavefront's ballot is two words.
__global__ __launch_bounds__(256) void lsh_summary_kernel(const uint32_t *__restrict__ qbits, int n_q, int W, int BQ,
                                                          int n_rep, int n_qb, uint32_t *__restrict__ rep) {
    extern __shared__ uint32_t qw[];  // the query block's codes, [BQ][W]
    const int b = blockIdx.x, h = blockIdx.y, j = threadIdx.x;
    const int g = BQ / n_rep;
    const int lane = lane_id();
    // a run's bits take 32 * W threads; the workgroup counts blockDim / (32 * W) runs at a time
    const int bit = j & (32 * W - 1), wave = bit >> 6, run0 = j / (32 * W), runs = blockDim.x / (32 * W);
    const int q_lo = b * BQ, q_hi = min(q_lo + BQ, n_q);
    // one round of loads for the whole block, then the votes are counted from LDS
    for (int t = j; t < (q_hi - q_lo) * W; t += blockDim.x) qw[t] = qbits[((size_t)h * n_q + q_lo) * W + t];
    __syncthreads();
    for (int u = run0; u < n_rep; u += runs) {
        const int q0 = q_lo + u * g, q1 = min(q0 + g, n_q);
        int ones = 0;
#pragma unroll 8
        for (int q = q0; q < q1; ++q) ones += (int)((qw[(q - q_lo) * W + (bit >> 5)] >> (bit & 31)) & 1u);
        const unsigned long long m = __ballot(q1 > q0 && 2 * ones >= q1 - q0);
        uint32_t *out = rep + ((size_t)h * n_qb * n_rep + (size_t)b * n_rep + u) * W;
        if (lane == 0) {
            out[2 * wave] = (uint32_t)m;
            out[2 * wave + 1] = (uint32_t)(m >> 32);
        }
    }
}

// out[h][b][kb] = max over the summaries u of block b (whose run holds a query) and the live keys k of key block
// kb of the number of equal bits.  A lane owns one key (its W words in registers) and walks all summaries (the
// same for every lane: scalar loads); the maximum over a key block is a reduction over BK lanes (BK a power of two
// <= 64) or over several 64-key rounds of a wavefront (BK a multiple of 64).
constexpr int LSH_QB = 8;  // query blocks whose scores a lane carries at a time

// Score of one 32-bit word of a (summary, key) pair, d = summary ^ key.
// BAND = 0: equal bits.  BAND in {4, 8, 16, 32}: the word holds 32/BAND hash tables (bands); a table counts when the
// two buckets differ in at most `radius` bits (0: same bucket; more: the neighbouring buckets are probed too).  Bits
// set per band by the usual pairwise sums, then one add per word whose carry into each band's top bit says "more than
// radius"; rc = that addend (see lsh_radius_addend).
template <int BAND>
__device__ __forceinline__ int lsh_word_score(unsigned d, unsigned rc, int radius) {
    if constexpr (BAND == 0) {
        return __popc(~d);
    } else {
        unsigned c = d - ((d >> 1) & 0x55555555u);
        c = (c & 0x33333333u) + ((c >> 2) & 0x33333333u);
        if constexpr (BAND == 4) return 8 - __popc((c + rc) & 0x88888888u);
        c = (c + (c >> 4)) & 0x0F0F0F0Fu;
        if constexpr (BAND == 8) return 4 - __popc((c + rc) & 0x80808080u);
        c = (c + (c >> 8)) & 0x00FF00FFu;
        if constexpr (BAND == 16) return 2 - __popc((c + rc) & 0x80008000u);
        c = (c + (c >> 16)) & 0xFFFFu;
        return (int)c <= radius ? 1 : 0;
    }
}
static inline unsigned lsh_radius_addend(int band, int radius) {
    if (band == 4) return (unsigned)(7 - radius) * 0x11111111u;
    if (band == 8) return (unsigned)(0x7F - radius) * 0x01010101u;
    if (band == 16) return (unsigned)(0x7FFF - radius) * 0x00010001u;
    return 0u;
}

template <int W, int BAND>
__global__ __launch_bounds__(256) void lsh_score_kernel(const uint32_t *__restrict__ kbits, const int32_t *__restrict__ len,
                                                        const uint32_t *__restrict__ rep, int C, int n_q, int BQ,
                                                        int n_rep, int BK, int n_qb, int n_kb_cap, int lds_words,
                                                        unsigned rc, int radius, int32_t *__restrict__ out) {
    const int h = blockIdx.y;
    const int L = min(len[h], C);
    const int n_kb = (L + BK - 1) / BK;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int g = BQ / n_rep;
    const uint32_t *kb_h = kbits + (size_t)h * C * W;
    const uint32_t *rp = rep + (size_t)h * n_qb * n_rep * W;
    // the head's summaries are staged in LDS when they fit (lds_words > 0): every lane reads the same word
    extern __shared__ uint32_t srep[];
    if (lds_words > 0) {
        for (int t = threadIdx.x; t < lds_words; t += blockDim.x) srep[t] = rp[t];
        __syncthreads();
        rp = srep;
    }
    const int rounds = BK > 64 ? BK / 64 : 1;             // 64-key rounds per key block
    const int kb_per_round = BK >= 64 ? 1 : 64 / BK;      // key blocks covered by one round of 64 lanes
    // unit = one round-set: kb_per_round key blocks (BK < 64) or one key block (BK >= 64)
    const int n_units = (n_kb + kb_per_round - 1) / kb_per_round;
    for (int unit = blockIdx.x * 4 + wave; unit < n_units; unit += gridDim.x * 4) {
        uint32_t kw[W];   // this lane's key when a key block fits one round (re-read per round otherwise)
        bool live = false;
        if (rounds == 1) {
            const int key = BK >= 64 ? unit * BK + lane : unit * 64 + lane;
            live = key < L;
#pragma unroll
            for (int w = 0; w < W; ++w) kw[w] = live ? kb_h[(size_t)key * W + w] : 0u;
        }
        // query blocks in batches of LSH_QB: the lane-exchange reductions of a batch are independent of each other
        for (int b0 = 0; b0 < n_qb; b0 += LSH_QB) {
            int best[LSH_QB];
#pragma unroll
            for (int i = 0; i < LSH_QB; ++i) best[i] = -1;
            for (int rd = 0; rd < rounds; ++rd) {
                if (rounds > 1) {
                    const int key = unit * BK + rd * 64 + lane;
                    live = key < L;
#pragma unroll
                    for (int w = 0; w < W; ++w) kw[w] = live ? kb_h[(size_t)key * W + w] : 0u;
                }
#pragma unroll
                for (int i = 0; i < LSH_QB; ++i) {
                    const int b = b0 + i;
                    if (b >= n_qb) break;  // uniform
                    for (int u = 0; u < n_rep; ++u) {
                        if (b * BQ + u * g >= n_q) break;  // uniform: this run and the later ones hold no query
                        const uint32_t *r = rp + ((size_t)b * n_rep + u) * W;
                        int eq = 0;
#pragma unroll
                        for (int w = 0; w < W; ++w) eq += lsh_word_score<BAND>(r[w] ^ kw[w], rc, radius);
                        if (live) best[i] = max(best[i], eq);
                    }
                }
            }
            // maximum over the lanes of a key block
            const int span = BK >= 64 ? 64 : BK;
            for (int off = 1; off < span; off <<= 1) {
#pragma unroll
                for (int i = 0; i < LSH_QB; ++i) best[i] = max(best[i], shfl_xor(best[i], off));
            }
            const int kb = BK >= 64 ? unit : unit * kb_per_round + lane / BK;
            if ((lane & (span - 1)) == 0 && kb < n_kb) {
#pragma unroll
                for (int i = 0; i < LSH_QB; ++i)
                    if (b0 + i < n_qb) out[((size_t)h * n_qb + b0 + i) * n_kb_cap + kb] = best[i];
            }
        }
    }
}

// Equal-bit ranking on the int8 matrix cores.  With the key's bits as 0 / 1 and the summary's as -1 / +1,
// equal bits = product + number of the summary's zero bits, a constant per summary that is added after the maximum.  The
// vector ALU form above needs 2 W + 1 instructions per (summary, 64 keys); here 32 x 32 pairs take W matrix instructions
// and 16 maxima, the bits of a key are spread over bytes once (8 instructions per word) and the summaries once per
// workgroup, as operand fragments in LDS (slot i of half g2 of a word: bits 4 g2 + i + 8 * {0..3} on both sides).
// A workgroup takes up to LSH_MM_KB / W column blocks of 32 summaries (blockIdx.z), a wavefront a key block at a time.
// 148 summaries of 128 bits against 12 x 37440 keys: 51.2 us on the vector ALU, 15.5 here (1.7 key blocks per wavefront,
// so set-up and the first rows' latency weigh most).
constexpr int LSH_MM_KB = 32;   // LDS for summary fragments per workgroup, in KB: several workgroups fit a compute unit
__device__ __forceinline__ i32x4 lsh_spread(unsigned w) {
    const unsigned m = 0x01010101u;
    return i32x4{(int)(w & m), (int)((w >> 1) & m), (int)((w >> 2) & m), (int)((w >> 3) & m)};
}
template <int W>
__global__ __launch_bounds__(256) void lsh_score_mm_kernel(const uint32_t *__restrict__ kbits, const int32_t *__restrict__ len,
                                                           const uint32_t *__restrict__ rep, int C, int n_q, int BQ, int n_rep,
                                                           int BK, int n_qb, int n_kb_cap, int32_t *__restrict__ out) {
    constexpr int CC = LSH_MM_KB / W;
    typedef unsigned __attribute__((ext_vector_type(W > 4 ? 4 : W), aligned(4))) key_words;   // rows are 4-byte aligned
    constexpr int KW = W > 4 ? 4 : W;
    __shared__ i32x4 frag[CC][W][64];
    __shared__ int zeros[CC * 32];
    const int h = blockIdx.y;
    const int L = min(len[h], C);
    const int n_kb = (L + BK - 1) / BK;
    if ((int)blockIdx.x * 4 >= n_kb) return;   // uniform for the workgroup
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, g2 = lane >> 5;
    const int NR = n_qb * n_rep, g = BQ / n_rep;
    const int cb0 = blockIdx.z * CC;
    const int ncb = min(CC, (NR + 31) / 32 - cb0);
    const uint32_t *kb_h = kbits + (size_t)h * C * W;
    const uint32_t *rp = rep + (size_t)h * NR * W;
    // one thread per (summary, word): both halves' fragments
    for (int t = threadIdx.x; t < ncb * 32 * W; t += blockDim.x) {
        const int w = t % W, c = t / W;
        const unsigned bits = rp[(size_t)min(cb0 * 32 + c, NR - 1) * W + w];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            i32x4 f = lsh_spread(bits >> (4 * half));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned z = (unsigned)f[i] ^ 0x01010101u;   // bytes that become -1
                f[i] = (int)(((z << 8) - z) | (unsigned)f[i]);
            }
            frag[c >> 5][w][half * 32 + (c & 31)] = f;
        }
    }
    for (int c = threadIdx.x; c < ncb * 32; c += blockDim.x) {
        const int rc = cb0 * 32 + c;
        // columns past the summaries or of a run without a query never count
        int z = -(1 << 20);
        if (rc < NR && (rc / n_rep) * BQ + (rc % n_rep) * g < n_q) {
            z = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) z += __popc(~rp[(size_t)rc * W + w]);
        }
        zeros[c] = z;
    }
    __syncthreads();
    for (int kb = blockIdx.x * 4 + wave; kb < n_kb; kb += gridDim.x * 4) {
        int best[CC];
#pragma unroll
        for (int c = 0; c < CC; ++c) best[c] = -(1 << 20);
        const int k_end = min(kb * BK + BK, L);
        for (int k0 = kb * BK; k0 < k_end; k0 += 64) {
            i32x4 a[2][W];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t *row = kb_h + (size_t)min(k0 + 32 * q + col, C - 1) * W;
#pragma unroll
                for (int p = 0; p < W / KW; ++p) {
                    const key_words kw = *(const key_words *)(row + p * KW);
#pragma unroll
                    for (int w = 0; w < KW; ++w) a[q][p * KW + w] = lsh_spread(kw[w] >> (4 * g2));
                }
            }
            const bool whole = k0 + 64 <= k_end;   // uniform
#pragma unroll
            for (int c = 0; c < CC; ++c) {
                if (c < ncb) {   // uniform
                    i32x16 acc0 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                    i32x16 acc1 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const i32x4 b = frag[c][w][lane];
                        acc0 = mfma_i8_32x32x32(a[0][w], b, acc0);
                        acc1 = mfma_i8_32x32x32(a[1][w], b, acc1);
                    }
                    int m = best[c];
                    if (whole) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) m = max(max(m, acc0[v]), acc1[v]);
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int key = k0 + 8 * (v >> 2) + 4 * g2 + (v & 3);
                            if (key < k_end) m = max(m, acc0[v]);
                            if (key + 32 < k_end) m = max(m, acc1[v]);
                        }
                    }
                    best[c] = m;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CC; ++c) {
            if (c < ncb) {
                int m = max_across_halves_i32(best[c]) + zeros[c * 32 + col];
                if (n_rep == 4) m = max_over_quad_i32(m);   // uniform
                else for (int off = 1; off < n_rep; off <<= 1) m = max(m, shfl_xor(m, off));
                const int rc = (cb0 + c) * 32 + col;
                if (g2 == 0 && (col & (n_rep - 1)) == 0 && rc < NR)
                    out[((size_t)h * n_qb + rc / n_rep) * n_kb_cap + kb] = m;
            }
        }
    }
}

struct LshWs {
    size_t rep_off, score_off, total;
};
static LshWs lsh_ws(int H, int n_q, int C, int n_bits, int BQ, int BK, int n_rep) {
    const int n_qb = (n_q + BQ - 1) / BQ;
    const int n_kb_cap = (C + BK - 1) / BK;
    LshWs w;
    w.rep_off = 0;
    w.score_off = align256((size_t)H * n_qb * n_rep * (n_bits / 8));
    w.total = w.score_off + align256((size_t)H * n_qb * n_kb_cap * sizeof(int32_t));
    return w;
}
size_t select_lsh_ws_bytes(int H, int n_q, int C, int n_bits, int BQ, int BK, int n_rep) {
    if (H <= 0 || n_q <= 0 || C <= 0 || n_bits <= 0 || BQ <= 0 || BK <= 0 || n_rep <= 0) return 0;
    return lsh_ws(H, n_q, C, n_bits, BQ, BK, n_rep).total;
}

static bool pow2_le32(int v) { return v >= 1 && v <= 32 && (v & (v - 1)) == 0; }

struct SelfWs {
    size_t rep_off, score_off, total;
};
static SelfWs self_ws(int H, int n_q, int C, int r, int BQ, int BK, int n_rep) {
    const int n_qb = (n_q + BQ - 1) / BQ;
    const int n_kb_cap = (C + BK - 1) / BK;
    SelfWs w;
    w.rep_off = 0;
    w.score_off = align256((size_t)H * n_qb * n_rep * r);
    w.total = w.score_off + align256((size_t)H * n_qb * n_kb_cap * sizeof(int32_t));
    return w;
}

size_t select_self_ws_bytes(int H, int n_q, int C, int r, int BQ, int BK, int n_rep) {
    if (H <= 0 || n_q <= 0 || C <= 0 || r <= 0 || BQ <= 0 || BK <= 0 || n_rep <= 0) return 0;
    return self_ws(H, n_q, C, r, BQ, BK, n_rep).total;
}
size_t select_cross_ws_bytes(int H, int n_q, int n_p, int BQ) {
    if (H <= 0 || n_q <= 0 || n_p <= 0 || BQ <= 0) return 0;
    const int n_qb = (n_q + BQ - 1) / BQ;
    return align256((size_t)H * n_qb * n_p * sizeof(int32_t));
}

int static_scratch_setup();

// more than 64 KB of LDS (long prompts) has to be allowed once per kernel and device; fastar_init also resolves the
// static scratch through this
int select_setup() {
    if (const int rc = static_scratch_setup(); rc != FASTAR_OK) return rc;
    static DeviceOnce once;
    return once.run([](int) {
        if (hipFuncSetAttribute((const void *)cross_fused_kernel<32>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)fused::lds_bytes(12288)) != hipSuccess ||
            hipFuncSetAttribute((const void *)cross_fused_kernel<64>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)fused::lds_bytes(12288)) != hipSuccess)
            return FASTAR_ERR_HIP;
        return FASTAR_OK;
    });
}

}  // namespace fastar

using namespace fastar;

static int select_self_impl(const int8_t *qcode, int n_q, const int8_t *kcode, const int32_t *len, int H, int C, int r,
                            int BQ, int n_rep, int BK, int n_sel, int32_t *sel, int32_t *nsel, void *ws,
                            size_t ws_bytes, void *stream, int n_sink = 0, int n_local = 0, int bits = 8) {
    if (!qcode || !kcode || !len || !sel || !nsel || !ws) return FASTAR_ERR_INVALID_ARG;
    if (n_sink < 0 || n_local < 0 || n_sink + n_local > n_sel) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || C <= 0 || BQ <= 0 || n_rep <= 0 || BK <= 0 || n_sel <= 0) return FASTAR_ERR_INVALID_ARG;
    if (BQ % n_rep != 0) return FASTAR_ERR_INVALID_ARG;
    if (((uintptr_t)qcode & 15) || ((uintptr_t)kcode & 15) || ((uintptr_t)ws & 255)) return FASTAR_ERR_INVALID_ARG;
    if ((r != 32 && r != 64) || !pow2_le32(n_rep) || BK % 32 != 0) return FASTAR_ERR_UNSUPPORTED;
    if (bits != 8 && !((bits == 4 || bits == 2) && r == 32)) return FASTAR_ERR_UNSUPPORTED;
    const int n_qb = (n_q + BQ - 1) / BQ;
    const int n_kb_cap = (C + BK - 1) / BK;
    // long caches whose summaries fit four column blocks take the streaming kernel: 768 workgroups that sweep each head's key
    // blocks together
    const int n_cb = (n_qb * n_rep + 31) / 32;
    const bool stream_kernel = streams(r, bits, n_cb, (size_t)n_kb_cap * H);
    const int per_pass = (n_cb + (n_cb + 7) / 8 - 1) / ((n_cb + 7) / 8);   // column blocks per pass, equal ones
    const size_t tile_bytes = (size_t)n_qb * KB_PER_WG * sizeof(int32_t);
    if (!stream_kernel && tile_bytes > 64 * 1024) return FASTAR_ERR_UNSUPPORTED;
    const SelfWs w = self_ws(H, n_q, C, r, BQ, BK, n_rep);
    if (ws_bytes < w.total) return FASTAR_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    // Short caches, query blocks that fill the chip at most once, codes that the XCDs fetch soon enough: one launch instead of three.
    if (bits == 8 && n_rep <= 8 && C <= short_keys(r) && BQ <= 256 && (int64_t)n_qb * H <= SHORT_WGS &&
        (int64_t)std::min(n_qb, 8) * H * C * r <= SHORT_BYTES) {
        const size_t lds = ((size_t)n_kb_cap * 4 + 15) / 16 * 16 + (size_t)BQ * r;
        const dim3 qgrid(n_qb, H);
        if (r == 32)
            hipLaunchKernelGGL(select_short_kernel<32>, qgrid, dim3(SHORT_THREADS), lds, s, qcode, n_q, kcode, len, C, BQ, n_rep,
                               BK, n_qb, n_kb_cap, n_sel, sel, nsel, n_sink, n_local);
        else
            hipLaunchKernelGGL(select_short_kernel<64>, qgrid, dim3(SHORT_THREADS), lds, s, qcode, n_q, kcode, len, C, BQ, n_rep,
                               BK, n_qb, n_kb_cap, n_sel, sel, nsel, n_sink, n_local);
        FASTAR_LAUNCH_CHECK();
        return FASTAR_OK;
    }
    int8_t *rep = (int8_t *)ws + w.rep_off;
    int32_t *score = (int32_t *)((char *)ws + w.score_off);
    const dim3 grid((n_kb_cap + KB_PER_WG - 1) / KB_PER_WG, H);
    constexpr int stream_wgs = 768;   // three resident workgroups per CU (the kernel is built for 168 registers)
    const dim3 grid_stream((unsigned)std::max(1, std::min(std::max(1, stream_wgs / H), (n_kb_cap + 3) / 4)), H);
    auto score_launch = [&](auto r_c, auto bits_c) {
        constexpr int RR = decltype(r_c)::value, BB = decltype(bits_c)::value;
        if constexpr (RR == 32) {
            if (stream_kernel) {
                hipLaunchKernelGGL((score_self_stream_kernel<RR, 4, BB>), grid_stream, dim3(256), 0, s, kcode, len, rep, C, n_q, BQ,
                                   n_rep, BK, n_qb, n_kb_cap, score);
                return;
            }
        }
        auto kernel = per_pass <= 2   ? score_self_kernel<RR, BB, 2>
                      : per_pass <= 4 ? score_self_kernel<RR, BB, 4>
                      : per_pass == 5 ? score_self_kernel<RR, BB, 5>
                                      : score_self_kernel<RR, BB, 8>;
        if constexpr (BB == 8) {
            if (per_pass == 3) kernel = score_self_kernel<RR, BB, 3>;
            if (per_pass == 6) kernel = score_self_kernel<RR, BB, 6>;
            if (per_pass == 7) kernel = score_self_kernel<RR, BB, 7>;
        }
        hipLaunchKernelGGL(kernel, grid, dim3(256), tile_bytes, s, kcode, len, rep, C, n_q, BQ, n_rep, BK, n_qb, n_kb_cap, score);
    };
#define FASTAR_SELF(RR, BB)                                                                                            \
    do {                                                                                                               \
        hipLaunchKernelGGL(rep_kernel<BB>, dim3(n_qb, H), dim3(128), 0, s, qcode, n_q, r, BQ, n_rep, n_qb, rep);       \
        FASTAR_LAUNCH_CHECK();                                                                                         \
        score_launch(std::integral_constant<int, RR>{}, std::integral_constant<int, BB>{});                            \
    } while (0)
    if (bits == 4) FASTAR_SELF(32, 4);
    else if (bits == 2) FASTAR_SELF(32, 2);
    else if (r == 32) FASTAR_SELF(32, 8);
    else FASTAR_SELF(64, 8);
#undef FASTAR_SELF
    FASTAR_LAUNCH_CHECK();
    launch_topk(score, n_kb_cap, len, C, BK, n_qb, H, n_sel, sel, nsel, n_sink, n_local, INT_MIN, s);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

extern "C" int ann_select_self(const int8_t *qcode, int n_q, const int8_t *kcode, const int32_t *len, int H, int C,
                               int r, int BQ, int n_rep, int BK, int n_sel, int32_t *sel, int32_t *nsel, void *ws,
                               size_t ws_bytes, void *stream) {
    return select_self_impl(qcode, n_q, kcode, len, H, C, r, BQ, n_rep, BK, n_sel, sel, nsel, ws, ws_bytes, stream);
}

extern "C" int ann_select_self_forced(const int8_t *qcode, int n_q, const int8_t *kcode, const int32_t *len, int H,
                                      int C, int r, int BQ, int n_rep, int BK, int n_sel, int n_sink, int n_local,
                                      int32_t *sel, int32_t *nsel, void *ws, size_t ws_bytes, void *stream) {
    return select_self_impl(qcode, n_q, kcode, len, H, C, r, BQ, n_rep, BK, n_sel, sel, nsel, ws, ws_bytes, stream, n_sink,
                            n_local);
}

extern "C" int ann_select_self_packed(const int8_t *qcode, int n_q, const int8_t *kcode, const int32_t *len, int H,
                                      int C, int r, int bits, int BQ, int n_rep, int BK, int n_sel, int n_sink,
                                      int n_local, int32_t *sel, int32_t *nsel, void *ws, size_t ws_bytes, void *stream) {
    if (bits != 2 && bits != 4 && bits != 8) return FASTAR_ERR_INVALID_ARG;
    return select_self_impl(qcode, n_q, kcode, len, H, C, r, BQ, n_rep, BK, n_sel, sel, nsel, ws, ws_bytes, stream, n_sink,
                            n_local, bits);
}

// ---- the same selection on the library's own static scratch, for callers that cannot allocate ----------------------
// `scratch` is device memory that every GPU the library runs on holds until the process ends.  In host code the name
// is only a stand-in for the symbol: the device address is looked up once per device (with that device current) and
// kept; kernels, and anything else on the host that needs the memory, use that pointer.
static __device__ __align__(256) unsigned char scratch[FASTAR_STATIC_SCRATCH_BYTES];
static void *scratch_ptr[DeviceOnce::MAX_DEVICES];

namespace fastar {
int static_scratch_setup() {
    static DeviceOnce once;
    return once.run([](int dev) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return FASTAR_ERR_HIP;
        scratch_ptr[dev] = p;
        return FASTAR_OK;
    });
}
}  // namespace fastar

extern "C" int ann_select_self_static(const int8_t *qcode, int n_q, const int8_t *kcode, const int32_t *len, int H,
                                      int C, int r, int BQ, int n_rep, int BK, int n_sel, int32_t *sel, int32_t *nsel,
                                      void *stream) {
    if (H <= 0 || n_q <= 0 || C <= 0 || r <= 0 || BQ <= 0 || n_rep <= 0 || BK <= 0) return FASTAR_ERR_INVALID_ARG;
    if (self_ws(H, n_q, C, r, BQ, BK, n_rep).total > (size_t)FASTAR_STATIC_SCRATCH_BYTES) return FASTAR_ERR_STATIC_SCRATCH;
    if (const int rc = static_scratch_setup(); rc != FASTAR_OK) return rc;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return FASTAR_ERR_HIP;
    // nothing in the scratch has to start from zero: the summaries and every score row that the top-k reads are
    // written by this call's own launches before they are read
    return select_self_impl(qcode, n_q, kcode, len, H, C, r, BQ, n_rep, BK, n_sel, sel, nsel, scratch_ptr[dev],
                            (size_t)FASTAR_STATIC_SCRATCH_BYTES, stream);
}

extern "C" int ann_select_cross(const int8_t *qcode, int n_q, const int8_t *pcode, int n_p, int H, int r, int BQ,
                                int n_sel, int32_t *sel, int32_t *nsel, void *ws, size_t ws_bytes, void *stream) {
    if (!qcode || !pcode || !sel || !nsel || !ws) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || n_p <= 0 || BQ <= 0 || n_sel <= 0) return FASTAR_ERR_INVALID_ARG;
    if (((uintptr_t)qcode & 15) || ((uintptr_t)pcode & 15) || ((uintptr_t)ws & 255)) return FASTAR_ERR_INVALID_ARG;
    if ((r != 32 && r != 64) || n_p > 12288) return FASTAR_ERR_UNSUPPORTED;
    const int n_qb = (n_q + BQ - 1) / BQ;
    if (ws_bytes < select_cross_ws_bytes(H, n_q, n_p, BQ)) return FASTAR_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const size_t lds = (size_t)n_p * sizeof(int32_t);
    auto kernel = r == 32 ? score_cross_kernel<32> : score_cross_kernel<64>;
    hipLaunchKernelGGL(kernel, dim3(n_qb, H), dim3(256), lds, s, qcode, pcode, n_q, n_p, BQ, n_qb, n_sel, sel, nsel);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

extern "C" int ann_cross_attn_fwd(const void *Q, const int8_t *qcode, int n_q, const void *Kp, const void *Vp,
                                  const int8_t *pcode, int n_p, int H, int d, int dtype, int r, int BQ, int n_sel,
                                  float scale, int32_t *sel, int32_t *nsel, void *O, void *stream) {
    if (!Q || !qcode || !Kp || !Vp || !pcode || !sel || !nsel || !O) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || n_p <= 0 || n_sel <= 0) return FASTAR_ERR_INVALID_ARG;
    if (!(scale > 0.0f) || !(scale < INFINITY)) return FASTAR_ERR_INVALID_ARG;
    if (((uintptr_t)Q & 15) || ((uintptr_t)Kp & 15) || ((uintptr_t)Vp & 15) || ((uintptr_t)O & 15) ||
        ((uintptr_t)qcode & 15) || ((uintptr_t)pcode & 15))
        return FASTAR_ERR_INVALID_ARG;
    if (dtype != FASTAR_BF16 || d != 128 || BQ != 128 || n_sel > fused::TK || (r != 32 && r != 64) || n_p > 12288)
        return FASTAR_ERR_UNSUPPORTED;
    const int n_qb = (n_q + 127) / 128;
    const size_t lds = fused::lds_bytes(n_p);
    hipStream_t s = (hipStream_t)stream;
    const float scale_log2 = scale * 1.4426950408889634f;
    if (const int rc = select_setup(); rc != FASTAR_OK) return rc;
    if (r == 32)
        hipLaunchKernelGGL(cross_fused_kernel<32>, dim3(n_qb, H), dim3(256), lds, s, (const unsigned short *)Q, qcode,
                           (const unsigned short *)Kp, (const unsigned short *)Vp, pcode, n_q, n_p, n_qb, n_sel,
                           scale_log2, sel, nsel, (unsigned short *)O);
    else
        hipLaunchKernelGGL(cross_fused_kernel<64>, dim3(n_qb, H), dim3(256), lds, s, (const unsigned short *)Q, qcode,
                           (const unsigned short *)Kp, (const unsigned short *)Vp, pcode, n_q, n_p, n_qb, n_sel,
                           scale_log2, sel, nsel, (unsigned short *)O);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

static int select_lsh_impl(const uint32_t *qbits, int n_q, const uint32_t *kbits, const int32_t *len, int H, int C,
                           int n_bits, int band, int radius, int BQ, int n_rep, int BK, int n_sel, int n_sink, int n_local,
                           int32_t *sel, int32_t *nsel, void *ws, size_t ws_bytes, void *stream) {
    if (!qbits || !kbits || !len || !sel || !nsel || !ws) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || C <= 0 || BQ <= 0 || n_rep <= 0 || BK <= 0 || n_sel <= 0) return FASTAR_ERR_INVALID_ARG;
    if (BQ % n_rep != 0 || ((uintptr_t)ws & 255)) return FASTAR_ERR_INVALID_ARG;
    if (radius < 0 || n_sink < 0 || n_local < 0 || n_sink + n_local > n_sel) return FASTAR_ERR_INVALID_ARG;
    if (n_bits != 64 && n_bits != 128 && n_bits != 256) return FASTAR_ERR_UNSUPPORTED;
    if (band != 0 && band != 4 && band != 8 && band != 16 && band != 32) return FASTAR_ERR_UNSUPPORTED;
    if (!((BK <= 64 && (BK & (BK - 1)) == 0) || BK % 64 == 0)) return FASTAR_ERR_UNSUPPORTED;
    if (band && radius > band) radius = band;   // every bucket of a table is probed from there on
    const int W = n_bits / 32;
    const int n_qb = (n_q + BQ - 1) / BQ;
    const int n_kb_cap = (C + BK - 1) / BK;
    const LshWs w = lsh_ws(H, n_q, C, n_bits, BQ, BK, n_rep);
    if (ws_bytes < w.total) return FASTAR_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    uint32_t *rep = (uint32_t *)((char *)ws + w.rep_off);
    int32_t *score = (int32_t *)((char *)ws + w.score_off);
    if ((size_t)BQ * W * 4 > 48 * 1024) return FASTAR_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(lsh_summary_kernel, dim3(n_qb, H), dim3(256), (size_t)BQ * W * 4, s, qbits, n_q, W, BQ, n_rep, n_qb,
                       rep);
    FASTAR_LAUNCH_CHECK();
    // equal bits of whole 64-key rounds, runs that tile the 32 columns: the matrix cores (15.5 against 51.2 us at
    // 12 x 37440 keys); tables, shorter key blocks and other runs have no such form, and more summaries than 65535
    // workgroups take (8.4 million of 256 bits per head) would exceed what the device allows a grid's z (65536)
    const int64_t n_z = (((int64_t)n_qb * n_rep + 31) / 32 + LSH_MM_KB / W - 1) / (LSH_MM_KB / W);
    if (band == 0 && BK % 64 == 0 && n_rep <= 32 && (n_rep & (n_rep - 1)) == 0 && n_z <= 65535) {
        // four workgroups per compute unit: their summaries are spread once for all of their key blocks
        const int64_t share = (1024 + H * n_z - 1) / (H * n_z);
        dim3 grid((unsigned)std::min<int64_t>((n_kb_cap + 3) / 4, share), H, (unsigned)n_z);
#define FASTAR_LSH_MM(WW) \
    hipLaunchKernelGGL(lsh_score_mm_kernel<WW>, grid, dim3(256), 0, s, kbits, len, rep, C, n_q, BQ, n_rep, BK, n_qb, n_kb_cap, score)
        if (W == 2) FASTAR_LSH_MM(2);
        else if (W == 4) FASTAR_LSH_MM(4);
        else FASTAR_LSH_MM(8);
#undef FASTAR_LSH_MM
    } else {
        const int kb_per_round = BK >= 64 ? 1 : 64 / BK;
        const int n_units = (n_kb_cap + kb_per_round - 1) / kb_per_round;
        dim3 grid((n_units + 3) / 4, H);
        int lds_words = n_qb * n_rep * W;
        if ((size_t)lds_words * 4 > 48 * 1024) lds_words = 0;  // too many summaries (per-query form): read them from memory
        const size_t lds_bytes = (size_t)lds_words * 4;
        const unsigned rc = lsh_radius_addend(band, radius);
#define FASTAR_LSH(WW, BB)                                                                                             \
        hipLaunchKernelGGL((lsh_score_kernel<WW, BB>), grid, dim3(256), lds_bytes, s, kbits, len, rep, C, n_q, BQ, n_rep, BK, \
                           n_qb, n_kb_cap, lds_words, rc, radius, score)
#define FASTAR_LSH_W(BB)                        \
        do {                                        \
            if (W == 2) FASTAR_LSH(2, BB);          \
            else if (W == 4) FASTAR_LSH(4, BB);     \
            else FASTAR_LSH(8, BB);                 \
        } while (0)
        if (band == 0) FASTAR_LSH_W(0);
        else if (band == 4) FASTAR_LSH_W(4);
        else if (band == 8) FASTAR_LSH_W(8);
        else if (band == 16) FASTAR_LSH_W(16);
        else FASTAR_LSH_W(32);
#undef FASTAR_LSH_W
#undef FASTAR_LSH
    }
    FASTAR_LAUNCH_CHECK();
    // with tables only key blocks with a collision are candidates
    launch_topk(score, n_kb_cap, len, C, BK, n_qb, H, n_sel, sel, nsel, n_sink, n_local, band ? 1 : INT_MIN, s);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

extern "C" int ann_select_lsh(const uint32_t *qbits, int n_q, const uint32_t *kbits, const int32_t *len, int H, int C,
                              int n_bits, int BQ, int n_rep, int BK, int n_sel, int32_t *sel, int32_t *nsel, void *ws,
                              size_t ws_bytes, void *stream) {
    return select_lsh_impl(qbits, n_q, kbits, len, H, C, n_bits, 0, 0, BQ, n_rep, BK, n_sel, 0, 0, sel, nsel, ws, ws_bytes,
                           stream);
}

extern "C" int ann_select_lsh_buckets(const uint32_t *qbits, int n_q, const uint32_t *kbits, const int32_t *len, int H,
                                      int C, int n_bits, int band_bits, int radius, int BQ, int n_rep, int BK, int n_sel,
                                      int n_sink, int n_local, int32_t *sel, int32_t *nsel, void *ws, size_t ws_bytes,
                                      void *stream) {
    if (band_bits <= 0) return FASTAR_ERR_INVALID_ARG;
    return select_lsh_impl(qbits, n_q, kbits, len, H, C, n_bits, band_bits, radius, BQ, n_rep, BK, n_sel, n_sink, n_local,
                           sel, nsel, ws, ws_bytes, stream);
}
