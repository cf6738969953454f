// TempCache (Sec. 5.2 of the paper, Lemma 1): merge one frame of new keys/values into the bounded
// per-head cache.  The steps, each a kernel on the caller's stream:
//   tc_match_window  (candidate list that fits LDS, probe = new key: the usual call) codes of the new keys AND the
//                 top-1 candidate slot of every token on exact integer code scores (int8 matrix cores), final in
//                 one launch; clears the group records of the matched slots
//   otherwise     encode (encode.hip) -> tc_match_all (the whole cache, a range of slots per workgroup) or tc_match (a
//                 longer list, in chunks), 64-bit atomicMax -> tc_prep (unpack the match, clear the group records it will touch)
//   tc_verify     cosine test on the 8-bit quantised full-width keys as an int64 inequality; joiners
//                 register in their slot's group record (count, best joiner); age histogram of the live slots
//   tc_plan       per head: ranks of the unmerged tokens (ballot + prefix sum), evictions needed,
//                 victims = oldest untouched slots (histogram select over several workgroups, ordered compaction)
//   tc_apply      representative key, mean value, multiplicity, code, stamp of merged slots; appended
//                 tokens into victims / fresh slots; merge map
// All decisions are integer and order-independent (max / count), so the merge map is reproducible.
#include <limits.h>

#include <algorithm>

#include "encode_dev.hpp"

namespace fastar {

int encode_launch(const void *x, int dtype, int64_t n_vec, int d, const fastar_codec *codec, int r, int8_t *code,
                  unsigned long long *zero_fill, int64_t zero_n, hipStream_t s,
                  ClearRecords clear = {});

constexpr int SCORE_BIAS = 1 << 23;      // makes every score positive inside the packed arg-max key
constexpr int PLAN_SCRATCH_WORDS = 64 + 3 * 1024;  // per-head scratch of tc_plan_kernel (PS_STRIDE)
constexpr int AGE_BINS = 1024;           // bins of an age histogram (frame_id - stamp), the last one collecting everything older
constexpr int AGE_WORDS = AGE_BINS + 16; // a slice's histogram (bins of age_bin) and, behind it, its largest stamp as a key
constexpr int HS_STRIDE = 8;             // per-head scalars: oldL, n_unmerged, e, n_victims, n_dropped, newL, 3 if the workspace is not clean, clean mark
constexpr int WS_CLEAN = 0x5A17C1EA;     // hs word 7 after a call: group records and plan scratch are all zero again
constexpr int WS_FAILED = 0x0BADC0DE;    // hs word 7 after a call whose plan gave up for the head: records and scratch are left as they are

typedef unsigned long long u64;

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Caches of up to SETTLE_SLOTS slots on a persistent workspace: the launches behind the match are one, tc_settle_kernel.
constexpr int SETTLE_SLICE = 8192;        // slots per slice of the age histogram
constexpr int SETTLE_SLOTS = 65536;       // eight slices
constexpr int SETTLE_THREADS = 512;
constexpr int SETTLE_TOKENS = 8192;       // tokens per frame (their list is held in LDS)
__host__ __device__ static inline int settle_slices(int C) { return (C + SETTLE_SLICE - 1) / SETTLE_SLICE; }

// Without a window, workgroups of the encode launch clear the group records of all live slots while these are few, which saves the
// launch that would clear the matched slots' ones (call with that launch -> without, us): 4 heads x 780 tokens x 9360 slots 28.4 ->
// 26.1, 12 x 1560 x 32760 75.2 -> 72.5, 24 x 1560 x 37440 176.8 -> 174.7; 40 x 1560 x 37440 196.0 -> 197.3, 40 x 100 x 150000 115 -> 130.
constexpr int64_t CLEAR_SLOTS_MAX = 1 << 20;

// What a call leaves clean for the next one (group records, per-head scalars, plan scratch) lies in front and has sizes that
// depend on the cache alone, so frames of any length share a persistent workspace.  Behind it is what every call writes before
// it reads it; its offsets move with the frame's length.
struct CompressWs {
    size_t hs, win, grp, ps, best, ck, cp, jstar, sbest, rank, victims, tstamp, ages, slot_age, slot_stamp, total;
};
static CompressWs compress_ws(int H, int C, int n_new, int r) {
    CompressWs w;
    size_t o = 0;
    const size_t T = (size_t)H * (n_new > 0 ? n_new : 1);
    w.hs = o; o += align256((size_t)H * HS_STRIDE * 4);
    w.win = o; o += align256((size_t)H * C * 8);
    w.grp = o; o += align256((size_t)H * C * 4);
    w.ps = o; o += align256((size_t)H * PLAN_SCRATCH_WORDS * 4);   // directly before best: one zero fill covers both
    w.best = o; o += align256(T * 8);
    w.ck = o; o += align256(T * r);
    w.cp = o; o += align256(T * r);
    w.jstar = o; o += align256(T * 4);
    w.sbest = o; o += align256(T * 4);
    w.rank = o; o += align256(T * 4);
    w.victims = o; o += align256(T * 4);
    w.tstamp = o; o += align256(T * 4);
    const size_t slices = C <= SETTLE_SLOTS ? (size_t)H * settle_slices(C) : 0;
    w.ages = o; o += align256(slices * AGE_WORDS * 4);
    w.slot_age = o; o += align256(slices * SETTLE_SLICE * 2);
    w.slot_stamp = o; o += align256(slices * SETTLE_SLICE * 4);
    w.total = o;
    return w;
}
size_t compress_ws_bytes(int H, int C, int n_new, int r) {
    if (H <= 0 || C <= 0 || n_new < 0 || r <= 0) return 0;
    return compress_ws(H, C, n_new, r).total;
}

constexpr int MATCH_NONE = -(1 << 26);       // score word of a missing candidate (minus its "penalty")
constexpr int MATCH_VALID = -(1 << 25);      // every real score is above, every missing one below
// ---- match against a candidate list too long for the LDS window -------------------------------------------------
// D = A x B: A rows = 32 candidate slots (codes gathered by slot id), B columns = 32 tokens (probe codes).
// A lane therefore sees 16 candidates of one token per matrix instruction and keeps the best
// (score, lowest slot) as one 64-bit key: (score + bias) << 32 | ~slot.
// CAND_CHUNK = candidate positions scanned by one workgroup: 64 for a shorter list (more, lighter workgroups hide the
// two dependent loads better), 256 for a longer one (fewer atomics per token).
// Ties go to the smallest slot; the list comes in any order and may repeat ids, so every score is compared as the full
// (score, smallest slot) key.
template <int R, int CAND_CHUNK>
__global__ __launch_bounds__(256) void tc_match_kernel(const int8_t *__restrict__ code, const int32_t *__restrict__ len,
                                                       int C, const int8_t *__restrict__ cp, int n_new,
                                                       const int32_t *__restrict__ cand, int n_cand, int metric,
                                                       u64 *__restrict__ best) {
    constexpr int KS = R / 32;
    constexpr int NIT = CAND_CHUNK / 32;  // groups of 32 candidates per workgroup
    __shared__ __attribute__((aligned(16))) int cpen[4][CAND_CHUNK];   // minus the score penalty: -|code|^2 (metric 0), 0 (metric 1); MATCH_NONE: no candidate
    __shared__ __attribute__((aligned(16))) int cslotw[4][CAND_CHUNK];   // slot of every row
    const int h = blockIdx.z;
    const int L = min(len[h], C);
    const int pos0 = blockIdx.y * CAND_CHUNK;
    const int pos1 = min(pos0 + CAND_CHUNK, n_cand);
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int col = lane & 31, g2 = lane >> 5;
    const int tok = blockIdx.x * 128 + wave * 32 + col;
    const int8_t *cph = cp + (size_t)h * n_new * R;
    const int8_t *ch = code + (size_t)h * C * R;
    i32x4 bfrag[KS];
    {
        const int trow = min(tok, n_new - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bfrag[ks] = *(const i32x4 *)(cph + (size_t)trow * R + ks * 32 + 16 * g2);
    }
    // Two rounds of independent loads for the whole chunk (slot ids, then the codes they name) instead of
    // one dependent pair per group: the chunk costs two memory round trips, not 2 * NIT.
    int slot[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int pos = pos0 + it * 32 + col;
        int sl = -1;
        if (pos < pos1) {
            sl = cand[(size_t)h * n_cand + pos];
            if (sl < 0 || sl >= L) sl = -1;
        }
        slot[it] = sl;
    }
    i32x4 afrag[NIT][KS];
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            i32x4 a = {0, 0, 0, 0};
            if (slot[it] >= 0) a = *(const i32x4 *)(ch + (size_t)slot[it] * R + ks * 32 + 16 * g2);
            afrag[it][ks] = a;
        }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        int nn = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int m = 0; m < 4; ++m) nn = dot4_i8((unsigned)afrag[it][ks][m], (unsigned)afrag[it][ks][m], nn);
        nn += shfl_xor(nn, 32);
        if (g2 == 0) {
            cpen[wave][it * 32 + col] = slot[it] >= 0 ? (metric == 0 ? -nn : 0) : MATCH_NONE;
            cslotw[wave][it * 32 + col] = slot[it];
        }
    }
    __syncthreads();  // every wavefront reads back only its own rows; the barrier orders write and read
    u64 mybest = 0;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        if (pos0 + it * 32 >= pos1) break;  // uniform
        // the accumulator starts from minus the penalty of its rows and takes the product twice for 2 * dot:
        // the matrix unit does the arithmetic of the score
        i32x16 acc;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const i32x4 np = *(const i32x4 *)(&cpen[wave][it * 32 + 8 * q4 + 4 * g2]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * q4 + e] = np[e];
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(afrag[it][ks], bfrag[ks], acc);
        if (metric == 0) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(afrag[it][ks], bfrag[ks], acc);
        }
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const i32x4 sl4 = *(const i32x4 *)(&cslotw[wave][it * 32 + 8 * q4 + 4 * g2]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const u64 key = ((u64)(unsigned)(acc[4 * q4 + e] + SCORE_BIAS) << 32) | (u64)(0xFFFFFFFFu - (unsigned)sl4[e]);
                if (sl4[e] >= 0 && key > mybest) mybest = key;
            }
        }
    }
    {
        const unsigned lo = shfl_xor((unsigned)mybest, 32), hi = shfl_xor((unsigned)(mybest >> 32), 32);
        const u64 other = ((u64)hi << 32) | lo;
        if (other > mybest) mybest = other;
    }
    if (g2 == 0 && tok < n_new && mybest != 0) atomicMax(&best[(size_t)h * n_new + tok], mybest);
}

// ---- scan of a window of candidates held in LDS ------------------------------------------------------------
// Shared by the kernel that stages a candidate list and the one that stages a range of the cache; eight wavefronts, TOKS
// tokens at a time.  ccode: codes chunk-major ([16-byte chunk][candidate], conflict-free operand reads); cslot: slot ids;
// cpen: minus half the penalty.
// A score 2 dot - |code|^2 is twice T = dot - ceil(|code|^2 / 2), plus one where |code|^2 is odd, so the scan needs one
// matrix product instead of two, for T.  Who wins among the candidates of the largest T (odd |code|^2 first, then the
// smallest slot):
//   ORDERED (a range of the cache, or a list ranked into slot order): those with odd |code|^2 come first, slots ascending in
//   each half, so the earliest position is the winner;
//   otherwise (a candidate list in any order, without repeats): positions mean nothing, cslot carries the parity in its top
//   bit (set for even), and the scan notes whether a second group of 32 reaches the largest T, for the caller to settle.
constexpr int WIN_THREADS = 512;
constexpr unsigned SLOT_EVEN = 0x80000000u;
template <int R, int TOKS, bool ORDERED>
struct WindowScan {
    static_assert(TOKS == 64 || TOKS == 256, "one set of token groups, or two");
    static constexpr int KS = R / 32, NCH = R / 16;
    static constexpr int NG = TOKS >= 256 ? 4 : 2;             // groups of 32 tokens a wavefront scans the window for
    static constexpr int TQ = TOKS / (32 * NG);                // such sets of groups
    static constexpr int SPLIT = (WIN_THREADS / 64) / TQ;      // wavefronts sharing one set, each on its share of the window
    static constexpr int TPT = WIN_THREADS / TOKS;             // threads per token of the look-up
    // parity of |code|^2 (the parity of the number of odd entries)
    __device__ static __forceinline__ bool odd_penalty(const i32x4 (&rw)[NCH]) {
        unsigned x = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) x ^= (unsigned)(rw[c][0] ^ rw[c][1] ^ rw[c][2] ^ rw[c][3]);
        return __popc(x & 0x01010101u) & 1;
    }
    __device__ static __forceinline__ void stage(i32x4 *ccode, int *cslot, int *cpen, int n_pad, int metric, int p, int slot,
                                                 const i32x4 (&rw)[NCH]) {
        int nn = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            ccode[c * n_pad + p] = rw[c];
#pragma unroll
            for (int m = 0; m < 4; ++m) nn = dot4_i8((unsigned)rw[c][m], (unsigned)rw[c][m], nn);
        }
        cslot[p] = ORDERED || slot < 0 ? slot : (int)((unsigned)slot | (metric == 0 && (nn & 1) ? 0u : SLOT_EVEN));
        cpen[p] = slot < 0 ? MATCH_NONE : metric == 0 ? -((nn + 1) >> 1) : 0;   // minus half the penalty, rounded up
    }
    // Of two (score, twice the group + tie) words the one with the better score; equal scores of two groups are a tie.
    __device__ static __forceinline__ u64 better(u64 a, u64 b) {
        const unsigned sa = (unsigned)(a >> 32), sb = (unsigned)(b >> 32);
        const u64 tied = a | (u64)(((unsigned)a >> 1) != ((unsigned)b >> 1) ? 1u : (unsigned)b & 1u);
        return sa > sb ? a : sb > sa ? b : tied;
    }
    // Running arg-max of a lane over the 16 scores per group its accumulators hold: only the best score and the group it
    // came from are kept in the loop (a maximum tree and one select per group; a later group replaces the best only on a
    // strictly higher score, so the earliest group wins among equals); which of the group's rows it was is looked up once,
    // after the loop, by recomputing that group's scores for the token.
    // Leaves (best score, earliest group) of this wavefront's share in partbest as one word per token, 0: none seen; not
    // ORDERED: (best score, twice the group, plus one if another group reaches that score).
    __device__ static __forceinline__ void scan(const i32x4 *ccode, const int *cpen, int n_pad, int n_groups, int tq, int ch,
                                                const i32x4 (&bfrag)[NG][KS], u64 (*partbest)[TOKS]) {
        const int lane = lane_id(), col = lane & 31, g2 = lane >> 5;
        int bs[NG], bg[NG];
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            bs[u] = INT_MIN;
            bg[u] = 0;
        }
        // One group of 32 candidates per step.  A wavefront issues in order, so the matrix instructions of one half of the
        // token groups are issued before the maxima of the half before them, and the operands, in two rotating sets, are
        // read most of a step before they are used.  Steps past the end repeat the last group: ORDERED, that changes nothing (only
        // a strictly higher score replaces the best); otherwise they are left out of the maxima, as they would look like ties.
        constexpr int HALF = NG / 2;
        struct Operands {
            i32x4 a[KS];
            i32x16 pen;
        };
        const int n_it = n_groups > ch ? (n_groups - ch + SPLIT - 1) / SPLIT : 0;
        auto group_of = [&](int it) { return min(ch + it * SPLIT, n_groups - 1); };
        // marks the penalties as still in use: the compiler would let the last product of a step overwrite them and copy the
        // next ones into place, 25 moves per step
        auto keep = [](const Operands &s) { asm volatile("" ::"v"(s.pen)); };
        auto rd = [&](Operands &s, int it) {
            const int gi = group_of(it);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) s.a[ks] = ccode[(2 * ks + g2) * n_pad + gi * 32 + col];
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {   // minus the penalty of the accumulators' rows
                const i32x4 np = *(const i32x4 *)(&cpen[gi * 32 + 8 * q4 + 4 * g2]);
#pragma unroll
                for (int e = 0; e < 4; ++e) s.pen[4 * q4 + e] = np[e];
            }
        };
        auto mm = [&](i32x16 (&acc)[HALF], const Operands &s, int u0) {   // the matrix unit subtracts the penalty
#pragma unroll
            for (int u = 0; u < HALF; ++u) acc[u] = mfma_i8_32x32x32(s.a[0], bfrag[u0 + u][0], s.pen);
#pragma unroll
            for (int ks = 1; ks < KS; ++ks)
#pragma unroll
                for (int u = 0; u < HALF; ++u) acc[u] = mfma_i8_32x32x32(s.a[ks], bfrag[u0 + u][ks], acc[u]);
        };
        auto red = [&](const i32x16 (&acc)[HALF], int it, int u0) {
            const int gi = group_of(it);
            if (!ORDERED && it >= n_it) return;   // uniform: the last group again would look like a second one
#pragma unroll
            for (int u = 0; u < HALF; ++u) {
                if constexpr (ORDERED) {
                    int mx = max(acc[u][0], bs[u0 + u]);
#pragma unroll
                    for (int v = 1; v < 16; ++v) mx = max(mx, acc[u][v]);
                    bg[u0 + u] = mx > bs[u0 + u] ? gi : bg[u0 + u];
                    bs[u0 + u] = mx;
                } else {
                    int mx = acc[u][0];
#pragma unroll
                    for (int v = 1; v < 16; ++v) mx = max(mx, acc[u][v]);
                    const int tied = mx == bs[u0 + u] ? bg[u0 + u] | 1 : bg[u0 + u];
                    bg[u0 + u] = mx > bs[u0 + u] ? 2 * gi : tied;
                    bs[u0 + u] = max(mx, bs[u0 + u]);
                }
            }
        };
        if (n_it > 0) {
            Operands o0, o1;
            i32x16 acc0[HALF], acc1[HALF];
            rd(o0, 0);
            rd(o1, 1);
            mm(acc0, o0, 0);
            for (int it = 0; it < n_it; it += 2) {
                mm(acc1, o0, HALF);
                keep(o0);
                rd(o0, it + 2);
                red(acc0, it, 0);
                mm(acc0, o1, 0);
                red(acc1, it, HALF);
                mm(acc1, o1, HALF);
                keep(o1);
                rd(o1, it + 3);
                red(acc0, it + 1, 0);
                mm(acc0, o0, 0);
                red(acc1, it + 1, HALF);
            }
        }
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            u64 key = bs[u] > MATCH_VALID ? ((u64)(unsigned)(bs[u] + SCORE_BIAS) << 32) | (u64)(ORDERED ? 0xFFFFFFFFu - (unsigned)bg[u] : (unsigned)bg[u]) : 0ull;
            const unsigned lo = shfl_xor((unsigned)key, 32), hi = shfl_xor((unsigned)(key >> 32), 32);
            const u64 other = ((u64)hi << 32) | lo;
            if (ORDERED) { if (other > key) key = other; }
            else key = better(key, other);
            if (g2 == 0) partbest[ch][(tq * NG + u) * 32 + col] = key;
        }
    }
    // Best score T of token t and the earliest position `at` that reaches it (false: no real candidate), after a barrier
    // behind scan(); TPT neighbouring threads per token (sub = 0 .. TPT-1), all of them get the answer.  The threads start
    // at different rows: the groups' rows lie at multiples of 512 bytes, all on the same banks.
    __device__ static __forceinline__ bool look_up(const i32x4 *ccode, const int *cpen, int n_pad, const i32x4 (&pc)[NCH],
                                                   bool ok, int t, int sub, const u64 (*partbest)[TOKS], int &T, int &at) {
        constexpr int ROWS = 32 / TPT;
        static_assert(ORDERED, "position order decides");
        u64 best = partbest[0][t];
#pragma unroll
        for (int c = 1; c < SPLIT; ++c) {
            const u64 other = partbest[c][t];
            if (other > best) best = other;
        }
        const bool seen = best != 0 && ok;
        T = (int)(unsigned)(best >> 32) - SCORE_BIAS;
        at = INT_MAX;
        if (seen) {
            const int row0 = (int)(0xFFFFFFFFu - (unsigned)best) * 32 + sub * ROWS;
#pragma unroll
            for (int v = 0; v < ROWS; ++v) {
                const int rw = row0 + ((v + t) & (ROWS - 1));
                int dot = 0;
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    const i32x4 cc = ccode[c * n_pad + rw];
#pragma unroll
                    for (int m = 0; m < 4; ++m) dot = dot4_i8((unsigned)cc[m], (unsigned)pc[c][m], dot);
                }
                if (dot + cpen[rw] == T) at = min(at, rw);
            }
        }
#pragma unroll
        for (int off = 1; off < TPT; off <<= 1) at = min(at, shfl_xor(at, off));
        return seen;
    }
    // The same for candidates in any order: best score T of token t and the winner's cslot word among its group (0xFFFFFFFF:
    // no candidate); tie: another group reaches T too.
    __device__ static __forceinline__ unsigned find(const i32x4 *ccode, const int *cslot, const int *cpen, int n_pad,
                                                    const i32x4 (&pc)[NCH], bool ok, int t, int sub,
                                                    const u64 (*partbest)[TOKS], int &T, bool &tie) {
        static_assert(!ORDERED, "position order decides");
        static_assert(TPT == 8 && SPLIT == 8, "a partial result per thread");
        constexpr int ROWS = 32 / TPT;
        // A tie may leave the threads with different groups; each sees the tie.
        u64 best = partbest[sub][t];
        const auto with = [&](unsigned lo, unsigned hi) { best = better(best, ((u64)hi << 32) | lo); };
        with(lane_of_eight<0>((unsigned)best), lane_of_eight<0>((unsigned)(best >> 32)));
        with(lane_of_eight<1>((unsigned)best), lane_of_eight<1>((unsigned)(best >> 32)));
        with(lane_of_eight<2>((unsigned)best), lane_of_eight<2>((unsigned)(best >> 32)));
        T = (int)(unsigned)(best >> 32) - SCORE_BIAS;
        const bool seen = best != 0 && ok;
        tie = seen && ((unsigned)best & 1u);
        unsigned winner = 0xFFFFFFFFu;
        if (seen) {
            const int row0 = (int)((unsigned)best >> 1) * 32 + sub * ROWS;
#pragma unroll
            for (int v = 0; v < ROWS; ++v) {
                const int rw = row0 + ((v + t) & (ROWS - 1));
                if (score(ccode, cpen, n_pad, pc, rw) == T) winner = min(winner, (unsigned)cslot[rw]);
            }
        }
        winner = min(winner, lane_of_eight<0>(winner));
        winner = min(winner, lane_of_eight<1>(winner));
        winner = min(winner, lane_of_eight<2>(winner));
        return winner;
    }
    // A second scan for candidates in any order, of which the best score is known (best_of: (winner so far, score) per token):
    // the smallest cslot word among those that reach it.
    __device__ static __forceinline__ void settle(const i32x4 *ccode, const int *cslot, const int *cpen, int n_pad, int n_groups,
                                                  int tq, int ch, const i32x4 (&bfrag)[NG][KS], unsigned *best_of) {
        const int lane = lane_id(), col = lane & 31, g2 = lane >> 5;
        int best[NG];
        unsigned w[NG];
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            best[u] = (int)best_of[2 * ((tq * NG + u) * 32 + col) + 1];
            w[u] = 0xFFFFFFFFu;
        }
        for (int gi = ch; gi < n_groups; gi += SPLIT) {
            i32x4 a[KS], sl[4];
            i32x16 pen;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[ks] = ccode[(2 * ks + g2) * n_pad + gi * 32 + col];
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const i32x4 np = *(const i32x4 *)(&cpen[gi * 32 + 8 * q4 + 4 * g2]);
                sl[q4] = *(const i32x4 *)(&cslot[gi * 32 + 8 * q4 + 4 * g2]);
#pragma unroll
                for (int e = 0; e < 4; ++e) pen[4 * q4 + e] = np[e];
            }
#pragma unroll
            for (int u = 0; u < NG; ++u) {
                i32x16 acc = pen;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(a[ks], bfrag[u][ks], acc);
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    w[u] = min(w[u], acc[v] == best[u] ? (unsigned)sl[v >> 2][v & 3] : 0xFFFFFFFFu);
            }
        }
#pragma unroll
        for (int u = 0; u < NG; ++u)
            if (w[u] != 0xFFFFFFFFu) atomicMin(&best_of[2 * ((tq * NG + u) * 32 + col)], w[u]);
    }
    __device__ static __forceinline__ int score(const i32x4 *ccode, const int *cpen, int n_pad, const i32x4 (&pc)[NCH], int rw) {
        int dot = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const i32x4 cc = ccode[c * n_pad + rw];
#pragma unroll
            for (int m = 0; m < 4; ++m) dot = dot4_i8((unsigned)cc[m], (unsigned)pc[c][m], dot);
        }
        return dot + cpen[rw];
    }
};
// Stable partition of up to 4096 ranked candidates, those marked in the bitmap s_odd (one 64-bit word per lane) first.
// Built and used by whole wavefronts.
struct OddFirst {
    u64 mine;
    int excl, n_odd;
    __device__ __forceinline__ explicit OddFirst(const u64 *s_odd) {
        const int lane = lane_id();
        mine = s_odd[lane];
        const int c = __popcll(mine);
        int incl = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, WAVE);
            if (lane >= off) incl += o;
        }
        n_odd = __shfl(incl, 63, WAVE);
        excl = incl - c;
    }
    __device__ __forceinline__ int place(int p) const {
        const unsigned lo = __shfl((int)(unsigned)mine, p >> 6, WAVE), hi = __shfl((int)(unsigned)(mine >> 32), p >> 6, WAVE);
        const u64 w = ((u64)hi << 32) | lo;
        const int below = __shfl(excl, p >> 6, WAVE) + __popcll(w & ((1ull << (p & 63)) - 1ull));
        return (w >> (p & 63)) & 1ull ? below : n_odd + p - below;
    }
};

// ---- match of the whole cache --------------------------------------------------------------------------------
// One workgroup = one range of slots (staged in LDS once) x one share of the frame's tokens, taken in blocks of up to TOKS;
// the best of a range goes to the token's packed (score, smallest slot) word.  What bounds it is not shown: at 12 heads x 1560
// tokens x 32760 slots the maxima (40 cycles per 32 x 32 scores) and the matrix products (32) are 11 to 20 us of the launch's 47;
// a workgroup's last block of tokens (780 in blocks of 224) leaves half of its wavefronts without work.  (A chunk of 256 slots
// per workgroup in registers with doubled products, position words and eight times the atomic operations took 71 us there; two
// workgroups per unit with 128 tokens each 50.)
template <int R, int TOKS>
__global__ __launch_bounds__(WIN_THREADS, 2) void tc_match_all_kernel(const int8_t *__restrict__ code,
                                                                      const int32_t *__restrict__ len, int C,
                                                                      const int8_t *__restrict__ cp, int n_new, int metric,
                                                                      int range, int share, int block,
                                                                      u64 *__restrict__ best) {
    typedef WindowScan<R, TOKS, true> WS;
    constexpr int KS = WS::KS, NCH = WS::NCH, NG = WS::NG, TPT = WS::TPT;
    extern __shared__ __attribute__((aligned(16))) unsigned char wlds[];
    i32x4 *ccode = (i32x4 *)wlds;                             // [NCH][range]
    int *cslot = (int *)(wlds + (size_t)NCH * range * 16);    // [range]
    int *cpen = cslot + range;                                // [range]
    __shared__ u64 partbest[WS::SPLIT][TOKS];
    __shared__ u64 s_odd[WAVE];
    const int h = blockIdx.z;
    const int L = min(len[h], C);
    const int j0 = blockIdx.x * range;
    if (j0 >= L) return;                                      // uniform
    const int n = min(range, L - j0), n_stage = (n + 31) & ~31;   // range is a multiple of 32
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int col = lane & 31, g2 = lane >> 5;
    const int swave = __builtin_amdgcn_readfirstlane(wave);   // uniform: the scan's bookkeeping stays in scalar registers
    const int tq = swave % WS::TQ, ch = swave / WS::TQ;
    const int t = tid / TPT, sub = tid % TPT;
    const int t0 = min((int)blockIdx.y * share, n_new), t1 = min(t0 + share, n_new);
    const int8_t *cph = cp + (size_t)h * n_new * R;
    i32x4 bfrag[NG][KS], pc[NCH];
    auto load_tokens = [&](int base) {   // second operands of the scan, and the look-up's probe code
#pragma unroll
        for (int u = 0; u < NG; ++u)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                bfrag[u][ks] = *(const i32x4 *)(cph + (size_t)min(base + (tq * NG + u) * 32 + col, n_new - 1) * R + ks * 32 + 16 * g2);
#pragma unroll
        for (int c = 0; c < NCH; ++c) pc[c] = *(const i32x4 *)(cph + (size_t)min(base + t, n_new - 1) * R + 16 * c);
    };
    // the range's rows, a batch of four per thread at a time; the parities first when they matter
    constexpr int PER = 4;
    const int8_t *ch_code = code + ((size_t)h * C + j0) * R;
    i32x4 row[PER][NCH];
    auto load_rows = [&](int p0) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
#pragma unroll
            for (int c = 0; c < NCH; ++c)
                row[k][c] = *(const i32x4 *)(ch_code + (size_t)min(p0 + k * WIN_THREADS + tid, n - 1) * R + 16 * c);
    };
    load_rows(0);
    load_tokens(t0);
    if (tid < WAVE) s_odd[tid] = 0ull;
    __syncthreads();
    for (int p0 = 0; p0 < n_stage; p0 += PER * WIN_THREADS) {   // uniform
        if (p0 > 0) load_rows(p0);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int p = p0 + k * WIN_THREADS + tid;           // a wavefront's 64 positions are one word
            const u64 odd = __ballot(metric == 0 && p < n && WS::odd_penalty(row[k]));
            if (lane == 0 && p < n) s_odd[p >> 6] = odd;
        }
    }
    __syncthreads();
    const OddFirst odd_first(s_odd);
    const bool single = n_stage <= PER * WIN_THREADS;           // uniform: the rows are still in registers
    for (int p0 = 0; p0 < n_stage; p0 += PER * WIN_THREADS) {
        if (!single) load_rows(p0);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int p = p0 + k * WIN_THREADS + tid;
            const int at = odd_first.place(min(p, n - 1));
            if (p < n_stage) WS::stage(ccode, cslot, cpen, range, metric, p < n ? at : p, p < n ? j0 + p : -1, row[k]);
        }
    }
    __syncthreads();
    for (int base = t0; base < t1; base += block) {
        const int lim = min(base + block, t1);
        WS::scan(ccode, cpen, range, base + tq * NG * 32 < lim ? n_stage / 32 : 0, tq, ch, bfrag, partbest);
        i32x4 pcur[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) pcur[c] = pc[c];
        if (base + block < t1) load_tokens(base + block);       // in flight during the look-up
        __syncthreads();
        int T, at;
        const bool seen = WS::look_up(ccode, cpen, range, pcur, base + t < lim, t, sub, partbest, T, at);
        if (sub == 0 && seen) {
            const int S = metric == 0 ? 2 * T + (at < odd_first.n_odd ? 1 : 0) : T;
            atomicMax(&best[(size_t)h * n_new + base + t],
                      ((u64)(unsigned)(S + SCORE_BIAS) << 32) | (u64)(0xFFFFFFFFu - (unsigned)cslot[at]));
        }
        __syncthreads();                                        // the next block's scan writes the partial results
    }
}
// slots of a range at most: what fits a compute unit's LDS beside the static arrays (and 4096, OddFirst's words)
static constexpr int match_all_range_max(int r) { return r == 32 ? 3584 : 2048; }
template <int R, int TOKS>
static int allow_match_all_lds() {
    return hipFuncSetAttribute((const void *)tc_match_all_kernel<R, TOKS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               match_all_range_max(R) * (R + 8)) == hipSuccess
               ? FASTAR_OK
               : FASTAR_ERR_HIP;
}
template <int R, int TOKS>
static int launch_match_all(const int8_t *code, const int32_t *len, int C, const int8_t *cp, int n_new, int H, int metric,
                            u64 *best, hipStream_t s) {
    // One workgroup per compute unit (LDS): as few ranges as its LDS allows, the tokens shared out while workgroups are
    // left over, then the ranges made shorter until the chip is covered.  Ranges of at least 512 slots: shorter ones are
    // all staging and look-up.
    constexpr int CUS = 256;
    int ranges = (C + match_all_range_max(R) - 1) / match_all_range_max(R);
    const int blocks = (n_new + TOKS - 1) / TOKS;
    const int splits = std::max(1, std::min(blocks, CUS / std::max(1, ranges * H)));
    ranges = std::max(ranges, std::min((C + 511) / 512, CUS / std::max(1, splits * H)));
    const int range = (((C + ranges - 1) / ranges) + 31) & ~31;
    const int share = (((n_new + splits - 1) / splits) + 31) & ~31;
    const int n_blk = (share + TOKS - 1) / TOKS;
    const int block = (((share + n_blk - 1) / n_blk) + 31) & ~31;
    const dim3 grid((C + range - 1) / range, (n_new + share - 1) / share, H);
    hipLaunchKernelGGL((tc_match_all_kernel<R, TOKS>), grid, dim3(WIN_THREADS), (size_t)range * (R + 8), s, code, len, C, cp,
                       n_new, metric, range, share, block, best);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

// ---- match against a candidate window held in LDS --------------------------------------------------------
// For a candidate list short enough to stage in LDS (the previous frame's slots: n_cand * (R + 8) bytes), one
// workgroup owns 64 tokens and sees every candidate, so the arg-max is final when it ends: no atomics, no packed
// keys to unpack, and the group records of the matched slots are cleared right here.
// With ENC the kernel also is the call's encode step for its 64 tokens (probe = new key): it quantises and projects
// their rows while the window's loads are in flight, leaves the codes in ck for the apply step, and clears the
// eviction plan's scratch words (ps_all) for the launches behind it.
// dynamic LDS of the window kernel; with the static arrays of its largest instantiation with 64 tokens per workgroup
// (r = 64, fused verify: 8.9 KB) it stays within the 160 KB of a compute unit
constexpr size_t WINDOW_LDS_MAX = 148 * 1024;
// What the fused tail of the window kernel needs from the verify step (defined further down).
template <bool BF16, int D>
struct VerifyRows;
// What the launch that settles a call wants of the match and verify launches besides their results (nullptr: the plan and
// apply launches follow instead): the length, the stamps of the matched slots and the slices' age histograms.
struct SettleOut {
    int32_t *hs;
    int32_t *tstamp;
    unsigned *ages;
    unsigned short *slot_age;
    int32_t *slot_stamp;
};
__device__ __forceinline__ void age_slice(const int32_t *__restrict__ len, const int32_t *__restrict__ stamp, int C, int n_new,
                                          int frame_id, const SettleOut &so, unsigned *lhist, int h, int slice);
template <int UN>
__device__ __forceinline__ void age_histogram_slice(const int32_t *__restrict__ len, const int32_t *__restrict__ stamp,
                                                    int C, int n_new, int frame_id, unsigned *__restrict__ ps,
                                                    int hist_word, int fut_word, unsigned *lhist, int part, int n_parts);
struct VerifyArgs {   // the verify step's arguments, for the launch that runs it as its tail
    const void *K;
    int tau2_q16;
    uint8_t *merged;
    const int32_t *stamp;
    int frame_id, hist_word, fut_word;
    int H;
    SettleOut so;
};

// With VERIFY (workspaces that every call leaves clean, see tempcache_compress) the kernel is the verify step too: once
// the arg-max of its 64 tokens is final it runs the cosine test for them and registers the joiners; nothing is cleared
// here (records and plan scratch are clean on entry).  The age histogram the plan wants is counted beside the match: by
// workgroups of its own at the end of the grid's x range (n_hist of them; behind the match it cost every workgroup 2 us),
// with 256 tokens per workgroup, where the grid fills the chip, by every workgroup as its tail (n_hist = 0).  The slices of
// tc_settle_kernel are counted, with 256 tokens per workgroup, in rows of the grid behind the heads': they run where tokens leave
// a unit idle, or after them.  Call at 40 heads x 3600 tokens x 64800 slots 256 us with the slices among each head's workgroups
// (each takes a whole unit's LDS, and the last heads' tokens waited), 208 as their tail, 206 behind; 24 x 2048 x 63488 85, 69, 64.
// TOKS: tokens per workgroup.  64 (eight wavefronts share the window scan) when the call is latency-bound; 256 (four
// wavefronts share the scan for their 128 tokens) when there are many more workgroups than the chip holds at once:
// staging the window is then paid a quarter as often.  The wide form's prefetched rows and operands take 252 registers (r = 32);
// at r = 64 with rows of 128 it spills 144 bytes per lane, around the scan, not in its loop.
//
// What bounds it: the chain of dependent phases of one workgroup.  Mean per phase at 12 heads x 1560 tokens and candidates
// (timestamps inside the kernel, us): list 3.5, repeats 0.7, encode 1.7 and staging 1.0 (the code rows are in flight
// meanwhile), scan 2.0, look-up 1.7, threshold test 2.3.  With 64 tokens, staged in slot order, so that position decides ties,
// list to staging took 8.1 and the encode another 2.1; in list order the scan pays 0.2 for noting ties and the look-up 0.6 for
// settling them.  Launch 21 -> 18, chunk of three calls 293 -> 285.  The look-up is 1.4 since a token's threads read a partial result
// each and meet by lane moves, and one barrier hands over the results and tells of ties (2 heads x 256 tokens: 1.6 -> 1.15).
// The scan was bound by the matrix units (two products per score) and the LDS (a group's codes and penalties, 5 KB, read
// for 32 tokens): one product, and 64 or 128 tokens per read; 256 tokens x 3600 candidates 18 -> 9 us, launch at
// 40 heads x 3600 tokens 113 -> 92.
template <int R, bool ENC, bool BF16, int D, bool VERIFY, int TOKS>
__global__ __launch_bounds__(WIN_THREADS, TOKS == 64 && R == 32 ? 4 : 2) void tc_match_window_kernel(
    const int8_t *__restrict__ code, const int32_t *__restrict__ len, int C, const int8_t *__restrict__ cp, int n_new,
    const int32_t *__restrict__ cand, int n_cand, int metric, int32_t *__restrict__ jstar, int32_t *__restrict__ sbest,
    u64 *__restrict__ win, int32_t *__restrict__ grp, const void *__restrict__ K_new, const int8_t *__restrict__ Rm,
    float qscale, int shift, int8_t *__restrict__ ck, unsigned *__restrict__ ps_all, int ps_words, int n_hist, VerifyArgs va) {
    static_assert(!VERIFY || ENC, "the fused verify step reads the probe codes this kernel encoded");
    static_assert(TOKS == 64 || TOKS == 256, "one pair of token groups, or four");
    constexpr int KS = R / 32;
    constexpr int NCH = R / 16;  // 16-byte chunks per code
    extern __shared__ __attribute__((aligned(16))) unsigned char wlds[];
    const int n_pad = (n_cand + 31) & ~31;
    i32x4 *ccode = (i32x4 *)wlds;                       // [NCH][n_pad]
    int *cslot = (int *)(wlds + (size_t)NCH * n_pad * 16);  // [n_pad]
    int *cpen = cslot + n_pad;                          // [n_pad]
    constexpr bool ORDERED = TOKS >= 256;               // how the window is staged
    typedef WindowScan<R, TOKS, ORDERED> WS;
    constexpr int NG = WS::NG, TQ = WS::TQ, SPLIT = WS::SPLIT;
    // partial arg-maxima of the scan; R before it, the verify hand-over and the age histogram after it
    __shared__ __attribute__((aligned(16))) u64 partbest[SPLIT][TOKS];
    static_assert(sizeof(partbest) >= AGE_BINS * sizeof(unsigned), "the histogram fits");
    const int n_tok_wgs = (int)gridDim.x - n_hist;
    if (VERIFY && TOKS >= 256 && (int)blockIdx.y >= va.H) {   // uniform: age slices behind everyone's tokens
        const int at = ((int)blockIdx.y - va.H) * (int)gridDim.x + (int)blockIdx.x, n_slices = settle_slices(C);
        if (at < va.H * n_slices)
            age_slice(len, va.stamp, C, n_new, va.frame_id, va.so, (unsigned *)partbest, at / n_slices, at % n_slices);
        return;
    }
    if (VERIFY && (int)blockIdx.x >= n_tok_wgs) {       // uniform
        if (va.so.hs)
            age_slice(len, va.stamp, C, n_new, va.frame_id, va.so, (unsigned *)partbest, blockIdx.y, (int)blockIdx.x - n_tok_wgs);
        else
            age_histogram_slice<4>(len, va.stamp, C, n_new, va.frame_id, ps_all + (size_t)blockIdx.y * ps_words, va.hist_word,
                                   va.fut_word, (unsigned *)partbest, (int)blockIdx.x - n_tok_wgs, n_hist);
        return;
    }
    const int h = blockIdx.y;
    const int L = min(len[h], C);
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    if (VERIFY && va.so.hs && blockIdx.x == 0 && tid == 0) va.so.hs[(size_t)h * HS_STRIDE] = L;
    const int col = lane & 31, g2 = lane >> 5;
    const int swave = __builtin_amdgcn_readfirstlane(wave);   // uniform: the scan's bookkeeping stays in scalar registers
    const int tq = swave % TQ, ch = swave / TQ;
    const int8_t *ch_code = code + (size_t)h * C * R;
    // The candidate list is a SET of slots: ids outside [0, L) do not count and a repeat only once, and ties go to the smallest
    // slot.  A bitmap over the slots, held where the codes will go (in several passes when the cache is longer than that area),
    // tells repeats.
    //   64 tokens: the window is staged in the order of the list and the look-up decides ties.
    //   256 tokens (ORDERED): a workgroup stages once for several blocks, so there it pays to rank the ids (set bits, prefix
    //   counts per word) and stage the rows in slot order, odd penalties first (WindowScan): position order then is all that the
    //   arg-max needs, the scan notes no ties, and repeats are not scanned.  Call at 40 heads x 3600 tokens x 230400 slots 162 us
    //   in list order, 152 ranked; 5 x 3600 (64 tokens) 54, 61.
    // The candidates' code rows are in flight meanwhile, and the first block of tokens is encoded.
    constexpr int CPT = ((int)(WINDOW_LDS_MAX / (R + 8)) + WIN_THREADS - 1) / WIN_THREADS;   // list entries per thread
    // of them, rows in flight while the ids are ranked (registers); the rows beyond are loaded when their ranks are known
    constexpr int PF = R == 32 ? (TOKS >= 256 ? CPT : BF16 ? 4 : 2) : 2;
    // R by way of LDS, where it fits and one 8-byte word per thread covers it (all but d = 128, r = 64): a coalesced load
    // per thread now, the operand's pieces from LDS later
    constexpr bool RM_LDS = ENC && (size_t)D * R <= sizeof(partbest) && D * R / 8 <= WIN_THREADS;
    const bool rm_lds = RM_LDS && ((uintptr_t)Rm & 7) == 0;   // uniform
    __shared__ int n_tied;
    __shared__ unsigned char s_tied[TOKS < 256 ? TOKS : 1];
    if (tid == 0) n_tied = 0;
    u64 rm_part = 0;
    if (rm_lds && tid < D * R / 8) rm_part = ((const u64 *)Rm)[tid];
    int ce[CPT];
    {
        const int32_t *ch_cand = cand + (size_t)h * n_cand;
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int p = k * WIN_THREADS + tid;
            ce[k] = p < n_cand ? ch_cand[p] : -1;
        }
    }
    // Tokens of this workgroup: [t0, t1).  64 tokens: its block.  256: an equal share of the frame (whole groups of 32
    // tokens), taken in blocks of 256 once the window is staged; the launcher sizes the grid so that no share is empty.
    const int per = TOKS < 256 ? TOKS : ((((n_new + n_tok_wgs - 1) / n_tok_wgs) + 31) & ~31);
    const int t0 = min((int)blockIdx.x * per, n_new), t1 = min(t0 + per, n_new);
    __shared__ __attribute__((aligned(16))) int8_t pcode[ENC ? TOKS * R : 16];
    CodeMatrix<BF16, D, R> cm;
    // encoding: 16 tokens per wavefront and round; 64 tokens: wavefronts 0..3 once, 256 tokens: all eight twice
    constexpr int EROUNDS = TOKS >= 128 ? TOKS / 128 : 1;
    const bool enc_wave = ENC && (TOKS >= 128 || wave < 4);
    RawVector<BF16, D> xr[EROUNDS];
    if (ENC && !VERIFY)
        for (int k = blockIdx.x * WIN_THREADS + tid; k < ps_words; k += gridDim.x * WIN_THREADS) ps_all[(size_t)h * ps_words + k] = 0u;
    // the rows of a block of tokens to encode
    auto load_block = [&](int base) {   // base: first token of the block
#pragma unroll
        for (int er = 0; er < EROUNDS; ++er) {
            const int etok = base + 16 * (wave + 8 * er) + (lane & 15);  // token this lane helps to encode
            xr[er].load((const char *)K_new + ((size_t)h * n_new + min(etok, n_new - 1)) * (size_t)D * (BF16 ? 2 : 4), lane >> 4);
        }
    };
    constexpr bool EARLY = BF16 || TOKS == 64;   // the first block's rows in flight while the window is staged (registers)
    if (EARLY && enc_wave) load_block(t0);
    unsigned *bm = (unsigned *)wlds;             // bitmap of the slots, [words]
    const int words = R * n_pad / (ORDERED ? 8 : 4);   // the code area; ordered, prefix counts of the words take half of it
    unsigned *wpre = bm + words;
    for (int w = tid; w < min((C + 31) >> 5, words); w += WIN_THREADS) bm[w] = 0u;
    __shared__ int s_wtot[WIN_THREADS / 64];
    __shared__ u64 s_odd[WAVE];                  // by rank in slot order: the candidates with an odd penalty
    static_assert(WINDOW_LDS_MAX / (R + 8) <= 64 * WAVE, "one word of s_odd per lane");
    if (ORDERED && tid < WAVE) s_odd[tid] = 0ull;
    if (rm_lds && tid < D * R / 8) ((u64 *)partbest)[tid] = rm_part;
#pragma unroll
    for (int k = 0; k < CPT; ++k)
        if (ce[k] < 0 || ce[k] >= L) ce[k] = -1;
    i32x4 row[PF][NCH];
#pragma unroll
    for (int k = 0; k < PF; ++k)
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            i32x4 v = {0, 0, 0, 0};
            if (ce[k] >= 0) v = *(const i32x4 *)(ch_code + (size_t)ce[k] * R + c * 16);
            row[k][c] = v;
        }
    // encodes the tokens [base, lim) of a block from the rows that load_block asked for
    auto encode_block = [&](int base, int lim) {
#pragma unroll
        for (int er = 0; er < EROUNDS; ++er) {
            const int etok = base + 16 * (wave + 8 * er) + (lane & 15);
            i32x4 xq[D / 64];
            xr[er].quantise(qscale, xq);
            const auto w = cm.code_words(xq, shift);
            cm.store(pcode + (16 * (wave + 8 * er) + (lane & 15)) * R, w, lane);
            if (etok < lim) cm.store(ck + ((size_t)h * n_new + etok) * R, w, lane);
        }
    };
    int pos[CPT];
    int n_u = 0;   // ordered: staged candidates, positions 0 .. n_u-1 (uniform over the workgroup)
#pragma unroll
    for (int k = 0; k < CPT; ++k) pos[k] = ORDERED ? -1 : k * WIN_THREADS + tid;
    for (int lo = 0; lo < L; lo += 32 * words) {   // uniform; one pass unless the cache is long for the list
        const int nw = min((L - lo + 31) >> 5, words);
        if (lo > 0) {
            __syncthreads();   // everyone is done with the pass before
            for (int w = tid; w < nw; w += WIN_THREADS) bm[w] = 0u;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            if (n_cand <= k * WIN_THREADS) break;   // uniform, here and below
            const int o = ce[k] - lo;
            if (ce[k] >= lo && o < 32 * nw) {
                const unsigned old = atomicOr(&bm[o >> 5], 1u << (o & 31));
                if (!ORDERED && ((old >> (o & 31)) & 1u)) ce[k] = -1;   // below every later lo
            }
        }
        if constexpr (ORDERED) {
            __syncthreads();
            // a thread owns a run of consecutive words, an odd number of them (their addresses spread over the banks); the
            // counts are those of the bits below within the wavefront's words
            const int wpt = ((nw + WIN_THREADS - 1) / WIN_THREADS) | 1;
            const int w0 = tid * wpt, w1 = min(w0 + wpt, nw);
            int c = 0;
            for (int w = w0; w < w1; ++w) c += __popc(bm[w]);
            const int incl = (int)wave_incl_scan((unsigned)c);
            if (lane == 63) s_wtot[wave] = incl;
            int run = incl - c;
            for (int w = w0; w < w1; ++w) {
                wpre[w] = (unsigned)run;
                run += __popc(bm[w]);
            }
            __syncthreads();
            int wtot[WIN_THREADS / 64];
#pragma unroll
            for (int q = 0; q < WIN_THREADS / 64; ++q) wtot[q] = s_wtot[q];
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                if (n_cand <= k * WIN_THREADS) break;
                const int o = ce[k] - lo, w = o >> 5;
                if (ce[k] >= lo && o < 32 * nw) {
                    int below = n_u + (int)wpre[w] + __popc(bm[w] & ((1u << (o & 31)) - 1u));
#pragma unroll
                    for (int q = 0; q + 1 < WIN_THREADS / 64; ++q) below += w >= 64 * wpt * (q + 1) ? wtot[q] : 0;
                    pos[k] = below;
                }
            }
#pragma unroll
            for (int q = 0; q < WIN_THREADS / 64; ++q) n_u += wtot[q];
        }
    }
    if (L <= 0) __syncthreads();   // R has been stored
    if (enc_wave) {
        if (rm_lds) cm.load((const int8_t *)partbest, lane);
        else cm.load(Rm, lane);
        if (!EARLY) load_block(t0);
        encode_block(t0, min(t0 + TOKS, t1));
    }
    // the code row of list entry k, where it was not asked for in advance
    auto row_of = [&](int k, i32x4 (&rw)[NCH]) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            rw[c] = i32x4{0, 0, 0, 0};
            if (k < PF) rw[c] = row[k < PF ? k : 0][c];
            else if (ce[k] >= 0) rw[c] = *(const i32x4 *)(ch_code + (size_t)ce[k] * R + c * 16);
        }
    };
    if (ORDERED && metric == 0) {   // uniform: stable partition by the parity of the penalty
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            if (n_cand <= k * WIN_THREADS) break;
            if (pos[k] < 0) continue;
            i32x4 rw[NCH];
            row_of(k, rw);
            if (WS::odd_penalty(rw)) atomicOr(&s_odd[pos[k] >> 6], 1ull << (pos[k] & 63));
        }
    }
    __syncthreads();   // the bitmap is dead: its memory takes the codes
    int n_odd = 0;
    if constexpr (ORDERED) {
        const OddFirst odd_first(s_odd);
        n_odd = odd_first.n_odd;
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            if (n_cand <= k * WIN_THREADS) break;
            const int p = odd_first.place(max(pos[k], 0));   // whole wavefronts
            if (pos[k] >= 0) pos[k] = p;
        }
    }
    const int n_stage = ORDERED ? (n_u + 31) & ~31 : n_pad;   // <= n_pad
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        if (n_cand <= k * WIN_THREADS) break;
        if (pos[k] < 0 || pos[k] >= n_pad) continue;
        i32x4 rw[NCH];
        row_of(k, rw);
        WS::stage(ccode, cslot, cpen, n_pad, metric, pos[k], ce[k], rw);
    }
    if (ORDERED && tid < n_stage - n_u) {   // the ragged end of the last group of 32
        const i32x4 none[NCH] = {};
        WS::stage(ccode, cslot, cpen, n_pad, metric, n_u + tid, -1, none);
    }
    for (int base = t0; base < t1; base += TOKS) {
    const int lim = min(base + TOKS, t1);   // this block's tokens: [base, lim)
    if (base != t0) {
        __syncthreads();   // the previous block's probe codes and arg-maxima have been read
        if (enc_wave) {
            load_block(base);
            encode_block(base, lim);
        }
    }
    __syncthreads();
    // Scan: the second operands of this wavefront's groups of 32 tokens.
    i32x4 bfrag[NG][KS];
#pragma unroll
    for (int u = 0; u < NG; ++u)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int t = (tq * NG + u) * 32 + col;
            bfrag[u][ks] = ENC ? *(const i32x4 *)(pcode + t * R + ks * 32 + 16 * g2)
                               : *(const i32x4 *)(cp + ((size_t)h * n_new + min(base + t, n_new - 1)) * R + ks * 32 + 16 * g2);
        }
    // a wavefront whose tokens all lie beyond the block's end scans nothing (uniform over the wavefront)
    WS::scan(ccode, cpen, n_pad, base + tq * NG * 32 < lim ? n_stage / 32 : 0, tq, ch, bfrag, partbest);
    __syncthreads();
    {
        constexpr int TPT = WS::TPT;
        const int t = tid / TPT, sub = tid % TPT, tok = base + t;
        i32x4 pc[NCH];
        const int8_t *prow = ENC ? pcode + t * R : cp + ((size_t)h * n_new + min(tok, n_new - 1)) * R;
#pragma unroll
        for (int c = 0; c < NCH; ++c) pc[c] = *(const i32x4 *)(prow + 16 * c);
        int T;   // best score
        // takes down slot j (-1: none) and score S (with the parity) of this thread's token
        auto result = [&](int j, int S) {
            if (sub != 0) return;
            if (tok < lim) {
                if (!VERIFY && j >= 0) {
                    win[(size_t)h * C + j] = 0;
                    grp[(size_t)h * C + j] = 0;
                }
                jstar[(size_t)h * n_new + tok] = j;
                sbest[(size_t)h * n_new + tok] = S;
            }
            // for the threshold test below; only this token's own threads (of this wavefront) have read the word
            if (VERIFY) partbest[0][t] = ((u64)(unsigned)S << 32) | (u64)(unsigned)j;
        };
        if constexpr (ORDERED) {
            int at;
            const bool seen = WS::look_up(ccode, cpen, n_pad, pc, tok < lim, t, sub, partbest, T, at);
            result(seen ? cslot[at] : -1, !seen ? 0 : metric == 0 ? 2 * T + (at < n_odd ? 1 : 0) : T);
            if (VERIFY) __syncthreads();
        } else {
            bool tie;
            unsigned winner = WS::find(ccode, cslot, cpen, n_pad, pc, tok < lim, t, sub, partbest, T, tie);
            auto settled = [&]() {
                const bool seen = winner != 0xFFFFFFFFu;
                result(seen ? (int)(winner & ~SLOT_EVEN) : -1, !seen ? 0 : metric == 0 ? 2 * T + (winner & SLOT_EVEN ? 0 : 1) : T);
            };
            // Ties between groups are settled by the workgroup: one token in a thousand has one on drawn data, most of them on a
            // picture with flat areas.  (winner so far, T) per token, and a list of the tied ones.  Up to MANY of them share
            // the wavefronts, which go through all candidates; more, and all go through the matrix products once more.  Launch at 12 heads x
            // 1560 tokens, share of tokens and candidates that take one of two values 0 / 2 / 10 / 50 / 100 %, us: 19 / 22 / 32 / 132 /
            // 344 with the workgroup on one token after the other; 18 / 21 / 24 / 24 / 23 this way.
            constexpr int MANY = WIN_THREADS / 64;
            unsigned *best_of = (unsigned *)partbest[1];   // the words of this token's own threads
            if (sub == 0) {
                best_of[2 * t] = winner;
                best_of[2 * t + 1] = (unsigned)(tie ? T : INT_MAX);   // INT_MAX: no candidate scores that
                if (tie) s_tied[atomicAdd(&n_tied, 1)] = (unsigned char)t;
            }
            if (!tie) settled();
            __syncthreads();
            const int n = n_tied;
            if (n > 0) {   // uniform
                if (n > MANY) {
                    WS::settle(ccode, cslot, cpen, n_pad, n_pad / 32, tq, ch, bfrag, best_of);
                } else {
                    const int share = n > 4 ? 1 : n > 2 ? 2 : n > 1 ? 4 : 8;   // wavefronts per token
                    const int q = min(swave / share, n - 1);                    // the last token's repeat their work
                    const int tt = (int)s_tied[q], best = (int)best_of[2 * tt + 1];
                    const int8_t *trow = ENC ? pcode + tt * R : cp + ((size_t)h * n_new + min(base + tt, n_new - 1)) * R;
                    i32x4 tc[NCH];
#pragma unroll
                    for (int c = 0; c < NCH; ++c) tc[c] = *(const i32x4 *)(trow + 16 * c);
                    unsigned w = 0xFFFFFFFFu;
#pragma unroll 4
                    for (int rw = 64 * (swave & (share - 1)) + lane; rw < n_pad; rw += 64 * share)
                        if (WS::score(ccode, cpen, n_pad, tc, rw) == best) w = min(w, (unsigned)cslot[rw]);
                    w = ~wave_max_last(~w);
                    if (lane == 63) atomicMin(&best_of[2 * tt], w);
                }
                __syncthreads();
                if (tie) {
                    winner = best_of[2 * t];
                    settled();
                }
                __syncthreads();
            }
        }
    }
    if constexpr (VERIFY) {
        constexpr int NPASS = TOKS * 16 / WIN_THREADS;   // tokens per 16-lane group
        constexpr int PB = TOKS >= 256 ? (BF16 ? 8 : 4) : 2;   // passes whose rows are loaded together (registers)
#pragma unroll
        for (int p0 = 0; p0 < NPASS; p0 += PB) {
            VerifyRows<BF16, D> vr[PB];
#pragma unroll
            for (int pass = 0; pass < PB; ++pass) {   // every row this group will need, in one round of loads
                const int t = (p0 + pass) * (WIN_THREADS / 16) + (tid >> 4);
                const int i = min(base + t, n_new - 1);
                vr[pass].load(va.K, K_new, pcode + t * R, R, C, n_new, metric, h, i, tid & 15, (int)(unsigned)partbest[0][t],
                              va.so.tstamp ? va.stamp : nullptr);
            }
#pragma unroll
            for (int pass = 0; pass < PB; ++pass) {
                const int t = (p0 + pass) * (WIN_THREADS / 16) + (tid >> 4);
                const int i = base + t;
                if (i < lim)   // whole 16-lane groups
                    vr[pass].decide(C, n_new, qscale, metric, va.tau2_q16, win, grp, va.merged, h, i, tid & 15,
                                    (int)(unsigned)partbest[0][t], (int)(unsigned)(partbest[0][t] >> 32), va.so.tstamp);
            }
        }
    }
    if constexpr (TOKS < 256) break;   // one block per workgroup: the grid covers the tokens (and the compiler sees no loop)
    }   // blocks of tokens
    if constexpr (VERIFY) {
        if (n_hist == 0 && !va.so.hs) {   // uniform over the launch
            __syncthreads();
            age_histogram_slice<(TOKS >= 256 ? 20 : 4)>(len, va.stamp, C, n_new, va.frame_id, ps_all + (size_t)h * ps_words,
                                                        va.hist_word, va.fut_word, (unsigned *)partbest, (int)blockIdx.x, n_tok_wgs);
        }
    }
}
static size_t match_window_lds(int n_cand, int r) { return (size_t)((n_cand + 31) & ~31) * (size_t)(r + 8); }
// static LDS of the wide (256 tokens per workgroup) instantiations: probe codes, partial results, under 1 KB of small
// arrays; what is left of a compute unit's 160 KB is their window
static constexpr size_t wide_window_lds_max(int r) { return (size_t)160 * 1024 - ((size_t)256 * r + 4 * 256 * 8 + 1024); }
template <int R, bool ENC, bool BF16, int D, bool VERIFY, int TOKS>
static int allow_window_lds() {
    const size_t lim = TOKS == 64 ? WINDOW_LDS_MAX : wide_window_lds_max(R);
    return hipFuncSetAttribute((const void *)tc_match_window_kernel<R, ENC, BF16, D, VERIFY, TOKS>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lim) == hipSuccess
               ? FASTAR_OK
               : FASTAR_ERR_HIP;
}
struct PlanResidency;
static int plan_residency(PlanResidency *out);
static int plan_residency_setup();
// every instantiation of the window and whole-cache kernels may use more than the default 64 KB of dynamic LDS: requested once per device
int tempcache_setup() {
    if (const int rc = plan_residency_setup(); rc != FASTAR_OK) return rc;
    static DeviceOnce once;
    return once.run([](int) {
        int rc = FASTAR_OK;
#define FASTAR_ALLOW(RR, BF, DD)                                                       \
    do {                                                                               \
        if (rc == FASTAR_OK) rc = allow_window_lds<RR, true, BF, DD, true, 64>();      \
        if (rc == FASTAR_OK) rc = allow_window_lds<RR, true, BF, DD, false, 64>();     \
        if (rc == FASTAR_OK) rc = allow_window_lds<RR, true, BF, DD, true, 256>();     \
        if (rc == FASTAR_OK) rc = allow_window_lds<RR, true, BF, DD, false, 256>();    \
    } while (0)
        FASTAR_ALLOW(32, true, 128); FASTAR_ALLOW(32, false, 128); FASTAR_ALLOW(32, true, 64); FASTAR_ALLOW(32, false, 64);
        FASTAR_ALLOW(64, true, 128); FASTAR_ALLOW(64, false, 128); FASTAR_ALLOW(64, true, 64); FASTAR_ALLOW(64, false, 64);
#undef FASTAR_ALLOW
        if (rc == FASTAR_OK) rc = allow_window_lds<32, false, true, 128, false, 64>();
        if (rc == FASTAR_OK) rc = allow_window_lds<64, false, true, 128, false, 64>();
        if (rc == FASTAR_OK) rc = allow_match_all_lds<32, 64>();
        if (rc == FASTAR_OK) rc = allow_match_all_lds<32, 256>();
        if (rc == FASTAR_OK) rc = allow_match_all_lds<64, 64>();
        if (rc == FASTAR_OK) rc = allow_match_all_lds<64, 256>();
        return rc;
    });
}
template <int R, bool ENC, bool BF16, int D, bool VERIFY, int TOKS, typename... Args>
static int launch_match_window(dim3 grid, size_t lds, hipStream_t s, Args... args) {
    hipLaunchKernelGGL((tc_match_window_kernel<R, ENC, BF16, D, VERIFY, TOKS>), grid, dim3(WIN_THREADS), lds, s, args...);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

// ---- prep (only behind the chunked match, which leaves packed arg-max keys) ---------------------------------
// A packed (score, smallest slot) word: the low word counts down with the slot.  0: no candidate.
__device__ __forceinline__ void unpack_match(u64 key, int &j, int &S) {
    j = key != 0 ? (int)(0xFFFFFFFFu - (unsigned)key) : -1;
    S = key != 0 ? (int)(unsigned)(key >> 32) - SCORE_BIAS : 0;
}
// Unpacks the match and clears the per-slot group records it will touch.  Not needed where the encode launch cleared them all
// (CLEAR_SLOTS_MAX); the verify launch then unpacks the match.
__global__ __launch_bounds__(256) void tc_prep_kernel(const u64 *__restrict__ best, int n_new, int C,
                                                      const int32_t *__restrict__ cand, int n_cand,
                                                      int32_t *__restrict__ jstar, int32_t *__restrict__ sbest,
                                                      u64 *__restrict__ win, int32_t *__restrict__ grp) {
    const int h = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_new) return;
    int j, S;
    unpack_match(best[(size_t)h * n_new + i], j, S);
    if (j >= 0) {
        win[(size_t)h * C + j] = 0;
        grp[(size_t)h * C + j] = 0;
    }
    jstar[(size_t)h * n_new + i] = j;
    sbest[(size_t)h * n_new + i] = S;
}

// Per head, a histogram of the live slots' ages (frame_id - stamp, 1024 bins, the last one collecting everything
// older) for the eviction plan: the verify launch, a whole grid, reads the stamps, where the plan has few
// workgroups per head.  The calling workgroup adds slice `part` of `n_parts` of the slots.  Called by whole workgroups.
// UN: 16-byte loads per lane in flight before the first is used (a slice read in one round trip when it fits).
template <int UN>
__device__ __forceinline__ void age_histogram_slice(const int32_t *__restrict__ len, const int32_t *__restrict__ stamp,
                                                    int C, int n_new, int frame_id, unsigned *__restrict__ ps,
                                                    int hist_word, int fut_word, unsigned *lhist, int part, int n_parts) {
    const int h = blockIdx.y;
    const int L = min(len[h], C);
    if (hist_word < 0) return;   // uniform over the launch: the plan counts the ages itself
    if (L + n_new <= C) return;  // uniform over the head: no eviction can be needed
    for (int k = threadIdx.x; k < AGE_BINS; k += blockDim.x) lhist[k] = 0;
    __syncthreads();
    // every workgroup takes a run of slots that starts on a multiple of four, four consecutive stamps per lane and load
    // (16 bytes when the head's row is aligned), four such loads in flight before the first is used
    const int chunk = ((L + n_parts - 1) / n_parts + 3) & ~3;
    const int j0 = min(part * chunk, L), j1 = min(j0 + chunk, L);
    const int32_t *st = stamp + (size_t)h * C;
    const bool vec = (((uintptr_t)st) & 15) == 0;
    bool future = false;
    // Neighbouring slots were mostly written by the same frame: when all of a wavefront's slots fall into one bin, one
    // lane adds their number (hundreds of additions to one LDS word would be served one after the other).
    for (int jb = j0; jb < j1; jb += (int)blockDim.x * 4 * UN) {   // uniform trip count
        int sv[UN][4];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int j = jb + (u * (int)blockDim.x + (int)threadIdx.x) * 4;
            if (vec && j + 3 < j1) {
                const i32x4 v = *(const i32x4 *)(st + j);
                sv[u][0] = v[0]; sv[u][1] = v[1]; sv[u][2] = v[2]; sv[u][3] = v[3];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) sv[u][e] = j + e < j1 ? st[j + e] : 0;
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int j = jb + (u * (int)blockDim.x + (int)threadIdx.x) * 4;
            unsigned bin[4];
            int n_act = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool act = j + e < j1;
                if (act && sv[u][e] > frame_id) future = true;
                bin[e] = min((unsigned)frame_id - (unsigned)sv[u][e], (unsigned)(AGE_BINS - 1));
                n_act += act ? 1 : 0;
            }
            const u64 m = __ballot(n_act > 0);
            if (m) {   // uniform
                const int first = __ffsll((unsigned long long)m) - 1;
                const unsigned fbin = (unsigned)__shfl((int)bin[0], first);   // an active lane's first slot is active
                bool same = true;
#pragma unroll
                for (int e = 0; e < 4; ++e) same = same && (j + e >= j1 || bin[e] == fbin);
                if (__all(same)) {
                    int tot = n_act;
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) tot += shfl_xor(tot, off);
                    if (lane_id() == first) atomicAdd(&lhist[fbin], (unsigned)tot);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (j + e < j1) atomicAdd(&lhist[bin[e]], 1u);
                }
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < AGE_BINS; k += blockDim.x)
        if (lhist[k]) atomicAdd(&ps[hist_word + k], lhist[k]);
    if (__any(future) && lane_id() == 0) atomicOr(&ps[fut_word], 1u);
}

// The same for tc_settle_kernel: the histogram of one slice of SETTLE_SLICE slots, by one workgroup, stored whole (nothing
// has to be cleared before or after), and every slot's bin: the launch that settles the call replaces stamps while other
// workgroups of it still look for victims.  Ages below AGE_EXACT have a bin each; older ones eight bins per octave.  A stamp in
// the future counts as age 0.  Bins that may hold more than one stamp, those and the first, have their slots' stamps kept too.
constexpr int AGE_EXACT = 832;                    // 13 * 2^6
static_assert(AGE_EXACT + (31 - 9) * 8 + 7 - 5 < AGE_BINS, "the last octave's bins");
__device__ __forceinline__ unsigned stamp_key(int32_t stamp) { return (unsigned)stamp ^ 0x80000000u; }   // ascending
__device__ __forceinline__ unsigned age_bin(int frame_id, int32_t stamp) {
    if (stamp > frame_id) return 0u;
    const unsigned age = (unsigned)frame_id - (unsigned)stamp;
    if (age < (unsigned)AGE_EXACT) return age;
    const int e = 31 - __clz(age);                // 9 .. 31; the three bits below the leading one
    return (unsigned)(AGE_EXACT - 5 + 8 * (e - 9)) + ((age >> (e - 3)) & 7u);
}
// smallest and largest age of a bin from AGE_EXACT on
__device__ __forceinline__ void age_bin_range(int bin, unsigned &lo, unsigned &hi) {
    const int i = bin - (AGE_EXACT - 5), e = 9 + (i >> 3);
    lo = (unsigned)(8 + (i & 7)) << (e - 3);
    hi = lo + ((1u << (e - 3)) - 1u);
}
__device__ __forceinline__ void age_slice(const int32_t *__restrict__ len, const int32_t *__restrict__ stamp, int C, int n_new,
                                          int frame_id, const SettleOut &so, unsigned *lhist, int h, int slice) {
    __shared__ unsigned s_max;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int L = min(len[h], C);
    if (L + n_new <= C) return;   // uniform over the head: no eviction can be needed
    for (int k = tid; k < AGE_BINS; k += nt) lhist[k] = 0;
    if (tid == 0) s_max = 0u;
    __syncthreads();
    const int32_t *st = stamp + (size_t)h * C;
    const int j0 = slice * SETTLE_SLICE, j1 = min(j0 + SETTLE_SLICE, L);
    unsigned short *age = so.slot_age + (size_t)h * settle_slices(C) * SETTLE_SLICE;
    int32_t *kept = so.slot_stamp + (size_t)h * settle_slices(C) * SETTLE_SLICE;
    unsigned kmax = 0u;
    constexpr int UN = 16;   // loads in flight (32 in the verify launch: 107 registers there, and no faster)
    for (int jb = j0; jb < j1; jb += nt * UN) {   // uniform trip count
        int sv[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int j = jb + u * nt + tid;
            sv[u] = j < j1 ? st[j] : 0;
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const bool act = jb + u * nt + tid < j1;
            const unsigned bin = age_bin(frame_id, sv[u]);
            if (act) {
                kmax = max(kmax, stamp_key(sv[u]));
                age[jb + u * nt + tid] = (unsigned short)bin;
                if (bin == 0u || bin >= (unsigned)AGE_EXACT) kept[jb + u * nt + tid] = sv[u];
            }
            // neighbouring slots were mostly written by the same frame: lanes of the first lane's age count together
            const unsigned fbin = (unsigned)__builtin_amdgcn_readfirstlane((int)bin);   // the first lane is in range if any is
            const u64 same = __ballot(act && bin == fbin);
            if (act && lane_id() == 0) atomicAdd(&lhist[fbin], (unsigned)__popcll(same));
            if (act && bin != fbin) atomicAdd(&lhist[bin], 1u);
        }
    }
    kmax = wave_max_last(kmax);
    if (lane_id() == 63) atomicMax(&s_max, kmax);
    __syncthreads();
    unsigned *out = so.ages + ((size_t)h * settle_slices(C) + slice) * AGE_WORDS;
    for (int k = tid; k < AGE_BINS; k += nt) out[k] = lhist[k];
    if (tid == 0) out[AGE_BINS] = s_max;
}

// ---- row pieces: 16 lanes share one row of D elements ----------------------------------------------------
template <bool BF16, int D>
struct RowPiece {
    static constexpr int EPL = D / 16;  // elements per lane
    __device__ static __forceinline__ void load(const void *base, size_t row, int l16, float *out) {
        if (BF16) {
            const unsigned short *p = (const unsigned short *)base + row * D + l16 * EPL;
            if (EPL == 8) {
                u32x4 w = *(const u32x4 *)p;
#pragma unroll
                for (int e = 0; e < 4; ++e) { out[2 * e] = bf16_lo(w[e]); out[2 * e + 1] = bf16_hi(w[e]); }
            } else {
                u32x2 w = *(const u32x2 *)p;
#pragma unroll
                for (int e = 0; e < 2; ++e) { out[2 * e] = bf16_lo(w[e]); out[2 * e + 1] = bf16_hi(w[e]); }
            }
        } else {
            const float *p = (const float *)base + row * D + l16 * EPL;
#pragma unroll
            for (int e = 0; e < EPL; e += 4) {
                f32x4 w = *(const f32x4 *)(p + e);
                out[e] = w[0]; out[e + 1] = w[1]; out[e + 2] = w[2]; out[e + 3] = w[3];
            }
        }
    }
    __device__ static __forceinline__ void store(void *base, size_t row, int l16, const float *v) {
        if (BF16) {
            unsigned short *p = (unsigned short *)base + row * D + l16 * EPL;
            if (EPL == 8) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
                *(u32x4 *)p = w;
            } else {
                u32x2 w;
#pragma unroll
                for (int e = 0; e < 2; ++e) w[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
                *(u32x2 *)p = w;
            }
        } else {
            float *p = (float *)base + row * D + l16 * EPL;
#pragma unroll
            for (int e = 0; e < EPL; e += 4) {
                f32x4 w = {v[e], v[e + 1], v[e + 2], v[e + 3]};
                *(f32x4 *)(p + e) = w;
            }
        }
    }
    // this lane's piece of a row as raw bits (held in registers between an early load and a late store)
    struct Raw {
        u32x4 w[(EPL * (BF16 ? 2 : 4) + 15) / 16];
    };
    __device__ static __forceinline__ Raw load_raw(const void *base, size_t row, int l16) {
        constexpr int BYTES = EPL * (BF16 ? 2 : 4);
        const char *s = (const char *)base + (row * D + (size_t)l16 * EPL) * (BF16 ? 2 : 4);
        Raw r;
        if (BYTES == 8) {
            const u32x2 v = *(const u32x2 *)s;
            r.w[0][0] = v[0]; r.w[0][1] = v[1]; r.w[0][2] = 0; r.w[0][3] = 0;
        } else {
#pragma unroll
            for (int b = 0; b < BYTES; b += 16) r.w[b / 16] = *(const u32x4 *)(s + b);
        }
        return r;
    }
    __device__ static __forceinline__ void store_raw(void *base, size_t row, int l16, const Raw &r) {
        constexpr int BYTES = EPL * (BF16 ? 2 : 4);
        char *d = (char *)base + (row * D + (size_t)l16 * EPL) * (BF16 ? 2 : 4);
        if (BYTES == 8) {
            u32x2 v = {r.w[0][0], r.w[0][1]};
            *(u32x2 *)d = v;
        } else {
#pragma unroll
            for (int b = 0; b < BYTES; b += 16) *(u32x4 *)(d + b) = r.w[b / 16];
        }
    }
    // raw bits -> float values of the piece
    __device__ static __forceinline__ void unpack(const Raw &r, float *out) {
        if (BF16) {
#pragma unroll
            for (int e = 0; e < EPL / 2; ++e) {
                const unsigned w = r.w[e / 4][e % 4];
                out[2 * e] = bf16_lo(w);
                out[2 * e + 1] = bf16_hi(w);
            }
        } else {
#pragma unroll
            for (int e = 0; e < EPL; ++e) out[e] = __uint_as_float(r.w[e / 4][e % 4]);
        }
    }
    // bit copy of this lane's piece of a row
    __device__ static __forceinline__ void copy(void *dst, size_t drow, const void *src, size_t srow, int l16) {
        constexpr int BYTES = EPL * (BF16 ? 2 : 4);
        const char *s = (const char *)src + (srow * D + (size_t)l16 * EPL) * (BF16 ? 2 : 4);
        char *d = (char *)dst + (drow * D + (size_t)l16 * EPL) * (BF16 ? 2 : 4);
        if (BYTES == 8) {
            *(u32x2 *)d = *(const u32x2 *)s;
        } else {
#pragma unroll
            for (int b = 0; b < BYTES; b += 16) *(u32x4 *)(d + b) = *(const u32x4 *)(s + b);
        }
    }
};

// Sum over the 16 lanes of a group (a row of the lane crossbar), in every lane; all 16 take part.
__device__ __forceinline__ int group16_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // row_half_mirror: the other four of eight
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);   // row_mirror: the other eight of sixteen
    return v;
}

// ---- verify --------------------------------------------------------------------------------------------
template <bool BF16, int D>
__device__ __forceinline__ void verify_token(const void *__restrict__ K, const void *__restrict__ K_new,
                                             const int8_t *__restrict__ cp, int r, int C, int n_new, float qscale,
                                             int metric, int tau2_q16, int32_t *__restrict__ jstar,
                                             const int32_t *__restrict__ sbest, const u64 *__restrict__ best,
                                             u64 *__restrict__ win,
                                             int32_t *__restrict__ grp, uint8_t *__restrict__ merged, int h, int i,
                                             int l16, const int32_t *__restrict__ stamp, int32_t *__restrict__ tstamp);

template <bool BF16, int D, bool SETTLE>
__global__ __launch_bounds__(SETTLE ? SETTLE_THREADS : 256) void tc_verify_kernel(const void *__restrict__ K, const void *__restrict__ K_new,
                                                        const int8_t *__restrict__ cp, int r, int C, int n_new,
                                                        float qscale, int metric, int tau2_q16,
                                                        int32_t *__restrict__ jstar,
                                                        const int32_t *__restrict__ sbest, const u64 *__restrict__ best,
                                                        u64 *__restrict__ win,
                                                        int32_t *__restrict__ grp, uint8_t *__restrict__ merged,
                                                        const int32_t *__restrict__ len,
                                                        const int32_t *__restrict__ stamp, int frame_id,
                                                        unsigned *__restrict__ plan_scratch, int hist_word,
                                                        int fut_word, int scratch_words, int n_slices, SettleOut so) {
    typedef RowPiece<BF16, D> RP;
    __shared__ unsigned lhist[AGE_BINS];
    const int h = blockIdx.y;
    if constexpr (SETTLE) {
        const int n_tok_wgs = (int)gridDim.x - n_slices;
        if ((int)blockIdx.x >= n_tok_wgs) {   // uniform
            age_slice(len, stamp, C, n_new, frame_id, so, lhist, h, (int)blockIdx.x - n_tok_wgs);
            return;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) so.hs[(size_t)h * HS_STRIDE] = min(len[h], C);
    }
    const int l16 = threadIdx.x & 15;
    const int i = blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4);
    if (i < n_new) verify_token<BF16, D>(K, K_new, cp, r, C, n_new, qscale, metric, tau2_q16, jstar, sbest, best, win, grp,
                                         merged, h, i, l16, SETTLE ? stamp : nullptr, SETTLE ? so.tstamp : nullptr);  // whole 16-lane groups
    if constexpr (SETTLE) return;
    age_histogram_slice<4>(len, stamp, C, n_new, frame_id, plan_scratch + (size_t)h * scratch_words, hist_word, fut_word,
                        lhist, (int)blockIdx.x, (int)gridDim.x);
}

// Token i of head h, matched to slot j with code score W (j < 0: no candidate); cprow = the token's probe code.
// Two halves, so that a caller with several tokens per lane group can issue all their loads first.  Whole 16-lane groups.
template <bool BF16, int D>
struct VerifyRows {
    typename RowPiece<BF16, D>::Raw ra, rb;   // raw bits: half the registers of the float values while the loads are in flight
    unsigned cw;
    int ts;   // stamp of the slot
    __device__ __forceinline__ void load(const void *__restrict__ K, const void *__restrict__ K_new, const int8_t *cprow,
                                         int r, int C, int n_new, int metric, int h, int i, int l16, int j,
                                         const int32_t *__restrict__ stamp) {
        ts = stamp && l16 == 0 && j >= 0 ? stamp[(size_t)h * C + j] : 0;
        typedef RowPiece<BF16, D> RP;
        ra = RP::load_raw(K_new, (size_t)h * n_new + i, l16);
        cw = (metric == 0 && l16 < r / 4) ? ((const unsigned *)cprow)[l16] : 0u;
        if (j >= 0) rb = RP::load_raw(K, (size_t)h * C + j, l16);
    }
    __device__ __forceinline__ void decide(int C, int n_new, float qscale, int metric, int tau2_q16, u64 *__restrict__ win,
                                           int32_t *__restrict__ grp, uint8_t *__restrict__ merged, int h, int i,
                                           int l16, int j, int W, int32_t *__restrict__ tstamp) const {
        typedef RowPiece<BF16, D> RP;
        const int nn = group16_sum(dot4_i8(cw, cw, 0));  // |probe code|^2 (r <= 64: at most 16 words)
        bool is_merged = false;
        if (j >= 0) {
            float a[RP::EPL], b[RP::EPL];
            RP::unpack(ra, a);
            RP::unpack(rb, b);
            int dot = 0, na = 0, nb = 0;
#pragma unroll
            for (int e = 0; e < RP::EPL; e += 4) {
                const unsigned qa = quant8x4(a[e], a[e + 1], a[e + 2], a[e + 3], qscale);
                const unsigned qb = quant8x4(b[e], b[e + 1], b[e + 2], b[e + 3], qscale);
                dot = dot4_i8(qa, qb, dot);
                na = dot4_i8(qa, qa, na);
                nb = dot4_i8(qb, qb, nb);
            }
            dot = group16_sum(dot);
            na = group16_sum(na);
            nb = group16_sum(nb);
            is_merged = dot > 0 && (long long)dot * dot * 65536ll >= (long long)tau2_q16 * na * nb;
            if (is_merged && l16 == 0) {
                if (metric == 0) W -= nn;
                const u64 key = ((u64)(unsigned)(W + SCORE_BIAS) << 32) | (u64)(0xFFFFFFFFu - (unsigned)i);
                atomicMax(&win[(size_t)h * C + j], key);
                atomicAdd(&grp[(size_t)h * C + j], 1);
            }
        }
        if (l16 == 0) merged[(size_t)h * n_new + i] = is_merged ? 1 : 0;
        if (tstamp && l16 == 0) tstamp[(size_t)h * n_new + i] = ts;
    }
};
template <bool BF16, int D>
__device__ __forceinline__ void verify_core(const void *__restrict__ K, const void *__restrict__ K_new,
                                            const int8_t *cprow, int r, int C, int n_new, float qscale, int metric,
                                            int tau2_q16, u64 *__restrict__ win, int32_t *__restrict__ grp,
                                            uint8_t *__restrict__ merged, int h, int i, int l16, int j, int W,
                                            const int32_t *__restrict__ stamp, int32_t *__restrict__ tstamp) {
    VerifyRows<BF16, D> v;
    v.load(K, K_new, cprow, r, C, n_new, metric, h, i, l16, j, stamp);
    v.decide(C, n_new, qscale, metric, tau2_q16, win, grp, merged, h, i, l16, j, W, tstamp);
}

template <bool BF16, int D>
__device__ __forceinline__ void verify_token(const void *__restrict__ K, const void *__restrict__ K_new,
                                             const int8_t *__restrict__ cp, int r, int C, int n_new, float qscale,
                                             int metric, int tau2_q16, int32_t *__restrict__ jstar,
                                             const int32_t *__restrict__ sbest, const u64 *__restrict__ best,
                                             u64 *__restrict__ win,
                                             int32_t *__restrict__ grp, uint8_t *__restrict__ merged, int h, int i,
                                             int l16, const int32_t *__restrict__ stamp, int32_t *__restrict__ tstamp) {
    // everything addressed by the token first (one round trip), then the matched slot's key row
    const size_t ti = (size_t)h * n_new + i;
    int j, S;
    if (best) {   // the match as its launch left it (uniform; see unpack_match)
        unpack_match(best[ti], j, S);
        if (l16 == 0) jstar[ti] = j;
    } else {
        j = jstar[ti];
        S = sbest[ti];
    }
    verify_core<BF16, D>(K, K_new, cp + ti * r, r, C, n_new, qscale, metric, tau2_q16, win, grp, merged, h, i, l16, j, S, stamp,
                         tstamp);
}

// ---- plan ----------------------------------------------------------------------------------------------
// NB + 1 workgroups of PLAN_THREADS threads per head (grid (NB + 1) x H).  The last one ranks the unmerged tokens.
// Each of the others counts the unmerged tokens and so knows e, the number of evictions needed.  When e > 0 they
// split the slots into NB contiguous ranges and find the e oldest untouched slots together:
//   threshold key T and the number of ties to take -> counts per workgroup -> ordered compaction, victims in
//   ascending slot order.
// T is normally read off the age histogram the verify launch left (no communication); otherwise: range of the keys ->
// histogram over that range (1024 bins, a second one inside the threshold bin when the range is wider).
// Between phases the workgroups of a head meet at a counter in global memory (head_barrier).  The grid is
// kept small enough (NB * H <= PLAN_MAX_GRID workgroups of 256 threads) to be resident at once, and every wait
// is bounded: a wait that runs out raises stats[7] and lets the kernel finish.
constexpr int PLAN_THREADS = 256;
constexpr int PLAN_WAVES = PLAN_THREADS / 64;
constexpr int PLAN_NB_MAX = 16;
constexpr int PLAN_MAX_GRID = 1024;
constexpr int PLAN_BINS = 1024;
constexpr int PLAN_SPIN_LIMIT = 1 << 20;
// per-head scratch in global memory (32-bit words), zeroed by the encode launch
constexpr int PS_BAR = 0;                       // 4 arrival counters
constexpr int PS_MAXK = 4, PS_MAXNK = 5;        // max key, max ~key
constexpr int PS_TOT = 6, PS_ERR = 7;           // eligible slots, bounded wait ran out
constexpr int PS_BLK = 8;                       // per workgroup, 64 bits: valid | count key > T | count key == T
constexpr int PS_FUT = 40;                      // some live slot carries a stamp above this call's frame id
constexpr int PS_HIST = 64;                     // histograms of PLAN_BINS: ages (from the verify launch), two select levels
constexpr int PS_STRIDE = PS_HIST + 3 * PLAN_BINS;
static_assert(PS_STRIDE == PLAN_SCRATCH_WORDS, "workspace layout");

__device__ __forceinline__ unsigned ld_agent(const unsigned *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// How long the plan's workgroups wait for each other, and for how many arrivals: normally PLAN_SPIN_LIMIT rounds for the
// head's own workgroups; the test hook fastar_debug_plan_wait shortens the wait and adds arrivals that never come, so
// that the exit of a wait that runs out can be exercised while every workgroup still finishes.
struct PlanWait {
    int spin_limit;
    unsigned extra_arrivals;
};
// All NB workgroups of a head arrive at counter *ctr; returns when all have (or the bounded wait ran out: bit 0 of *err).
// What the workgroups of a head tell each other inside this kernel goes through device-scope atomic operations only
// (additions / maxima on the head's scratch words before the meeting, atomic loads of them after it), which are performed
// at the memory side, past the per-XCD caches.  So no cache maintenance is needed, only order: every thread waits until
// its own memory operations have been acknowledged (vmcnt(0): on this architecture stores and atomics without a return
// value count there too), then the workgroup meets, then one thread announces the arrival; whoever sees all arrivals
// issues its loads after that.  A device-scope fence instead would write back and invalidate the XCD's L2 (dirty lines of
// the launches before included): measured 10 - 15 us per meeting here.
__device__ __forceinline__ void head_barrier(unsigned *ctr, unsigned nb, unsigned *err, PlanWait pw) {
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    __syncthreads();
    if (nb > 1 && threadIdx.x == 0) {
        atomicAdd(ctr, 1u);
        int spins = 0;
        while (ld_agent(ctr) < nb + pw.extra_arrivals) {
            if (++spins > pw.spin_limit) {
                atomicOr(err, 1u);
                break;
            }
            __builtin_amdgcn_s_sleep(4);
        }
    }
    __syncthreads();
}

// Block-wide ordered exclusive prefix over the threads, for a flag or a per-thread count.
struct BlockScan {
    unsigned *wtot;  // [PLAN_WAVES] in LDS
    __device__ __forceinline__ unsigned excl(bool flag, unsigned &total) {
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        const unsigned long long m = __ballot(flag);
        __syncthreads();  // previous use of wtot finished
        if (lane == 0) wtot[wave] = __popcll(m);
        __syncthreads();
        unsigned pos = __popcll(m & ((1ull << lane) - 1ull));
        total = 0;
#pragma unroll
        for (int w = 0; w < PLAN_WAVES; ++w) {
            const unsigned c = wtot[w];
            if (w < wave) pos += c;
            total += c;
        }
        return pos;
    }
    __device__ __forceinline__ unsigned excl_sum(unsigned v, unsigned &total) {
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        unsigned incl = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned o = __shfl_up(incl, off, WAVE);
            if (lane >= off) incl += o;
        }
        __syncthreads();
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        unsigned pos = incl - v;
        total = 0;
#pragma unroll
        for (int w = 0; w < PLAN_WAVES; ++w) {
            const unsigned c = wtot[w];
            if (w < wave) pos += c;
            total += c;
        }
        return pos;
    }
    __device__ __forceinline__ unsigned sum(unsigned v) {
        unsigned tot;
        excl_sum(v, tot);
        return tot;
    }
};

// PLAN_TOK_MAX: tokens per thread kept in registers (8: frames up to 2048 tokens; 16: up to 4096; longer frames are
// re-read from memory in dependent loads).

// PLAN_PER_MAX: slots per thread kept in registers (longer runs are re-read from memory); 16 for caches up to
// 16 * 256 * NB slots per head, 64 beyond (a 64-frame world-model cache: 57 slots per thread).
template <int PLAN_PER_MAX, int PLAN_TOK_MAX>
__global__ __launch_bounds__(PLAN_THREADS) void tc_plan_kernel(const int32_t *__restrict__ len,
                                                               const int32_t *__restrict__ stamp, int C, int n_new,
                                                               int frame_id, const int32_t *__restrict__ jstar,
                                                               const uint8_t *__restrict__ merged,
                                                               const u64 *__restrict__ win, int32_t *__restrict__ rank,
                                                               int32_t *__restrict__ victims, int32_t *__restrict__ hs,
                                                               int32_t *__restrict__ stats, unsigned *__restrict__ ps_all,
                                                               int ws_persistent, int self_hist, PlanWait pw) {
    extern __shared__ unsigned touched[];  // bitmap over this workgroup's slot range
    __shared__ unsigned lhist[PLAN_BINS];
    __shared__ unsigned wtot[PLAN_WAVES];
    __shared__ unsigned red_a[PLAN_WAVES], red_b[PLAN_WAVES];
    __shared__ unsigned sh_bin, sh_above;
    __shared__ unsigned sh_blk[2 * PLAN_NB_MAX];
    static_assert(PLAN_THREADS * 4 == PLAN_BINS, "one thread per four bins");
    const int h = blockIdx.y, b = blockIdx.x, NB = gridDim.x - 1;  // the last workgroup of a head only ranks
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int L = min(len[h], C);
    unsigned *ps = ps_all + (size_t)h * PS_STRIDE;
    BlockScan scan{wtot};
    const size_t tb = (size_t)h * n_new, cb = (size_t)h * C;

    // workgroup NB of every head only ranks the unmerged tokens, ascending token order
    if (b == NB) {
        unsigned done = 0;
        for (int base = 0; base < n_new; base += PLAN_THREADS) {
            const int i = base + tid;
            const bool unm = i < n_new && merged[tb + i] == 0;
            unsigned tot;
            const unsigned pos = scan.excl(unm, tot);
            if (i < n_new) rank[tb + i] = unm ? (int)(done + pos) : -1;
            done += tot;
        }
        return;
    }
    // First round of loads, all independent: the tokens' merge flags and slots (PLAN_TOK_MAX per thread in
    // registers), this thread's run of stamps, four bins of the age histogram.
    const int32_t *st = stamp + cb;
    int tj[PLAN_TOK_MAX];  // slot a token merged into, -1: not merged (or beyond n_new)
    const bool tok_cached = n_new <= PLAN_TOK_MAX * PLAN_THREADS;
    unsigned n_unm;
    {
        unsigned c = 0;
        if (tok_cached) {
            unsigned char mg[PLAN_TOK_MAX];
#pragma unroll
            for (int k = 0; k < PLAN_TOK_MAX; ++k) {
                const int i = tid + k * PLAN_THREADS;
                mg[k] = i < n_new ? merged[tb + i] : 1;
                tj[k] = i < n_new ? jstar[tb + i] : -1;
            }
#pragma unroll
            for (int k = 0; k < PLAN_TOK_MAX; ++k) {
                c += mg[k] == 0 ? 1u : 0u;
                if (!mg[k] || tid + k * PLAN_THREADS >= n_new) tj[k] = -1;
            }
        } else {
            for (int i = tid; i < n_new; i += PLAN_THREADS) c += merged[tb + i] == 0 ? 1u : 0u;
        }
        // the loads below do not depend on the count: issued before the reduction waits for the ones above
        n_unm = c;
    }
    // Long runs (PLAN_PER_MAX 64) start on multiples of four slots so that their stamps can be read 16 bytes at a time.
    // A thread's run is contiguous, so a load in which every lane reads from its own run touches 64 cache lines: the runs
    // of a wavefront (contiguous too) are instead read in four pieces of 16 runs each, consecutive lanes consecutive
    // 16 bytes, and handed to their owners through a piece of LDS that belongs to the wavefront.
    constexpr bool QUADS = PLAN_PER_MAX > 16;
    __shared__ __attribute__((aligned(16))) int stage[QUADS ? PLAN_WAVES * 16 * PLAN_PER_MAX : 4];
    const int span = QUADS ? (((L + NB - 1) / NB + 3) & ~3) : (L + NB - 1) / NB;
    const int s0 = min(b * span, L), s1 = min(s0 + span, L);
    const int per_raw = (span + PLAN_THREADS - 1) / PLAN_THREADS;
    const int per = QUADS ? ((per_raw + 3) & ~3) : per_raw;
    const int j0 = min(s0 + tid * per, s1), j1 = min(j0 + per, s1);
    const bool maybe = L + n_new > C;  // uniform: otherwise no eviction can be needed
    const bool cached = per <= PLAN_PER_MAX;
    int sreg[PLAN_PER_MAX];
    unsigned hreg[4] = {0, 0, 0, 0};
    if (maybe) {
        if (cached && QUADS && (((uintptr_t)st & 15) == 0)) {
            int *wst = stage + wave * (16 * PLAN_PER_MAX);   // this wavefront's piece: 16 runs
            const int piece = 16 * per;                       // slots of 16 runs: at most 1024, i.e. four 16-byte loads per lane
            const int wbase = s0 + wave * 64 * per;           // first slot of the wavefront's runs (may lie beyond s1)
            auto load_piece = [&](int c, i32x4 (&v)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = u * 64 + lane;              // quad of the piece
                    const int slot = wbase + c * piece + 4 * q;
                    v[u] = i32x4{0, 0, 0, 0};
                    if (4 * q < piece) {
                        if (slot + 3 < s1) {
                            v[u] = *(const i32x4 *)(st + slot);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[u][e] = slot + e < s1 ? st[slot + e] : 0;
                        }
                    }
                }
            };
            i32x4 cur[4], nxt[4];
            load_piece(0, cur);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (c + 1 < 4) load_piece(c + 1, nxt);        // in flight while this piece is handed over
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = u * 64 + lane;
                    if (4 * q < piece) *(i32x4 *)(wst + 4 * q) = cur[u];
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                if ((lane >> 4) == c) {                       // the owners of this piece's runs
                    const int *mine = wst + (lane & 15) * per;
#pragma unroll
                    for (int k = 0; k < PLAN_PER_MAX; k += 4) {
                        if (k < per) {
                            const i32x4 w = *(const i32x4 *)(mine + k);
                            sreg[k] = w[0]; sreg[k + 1] = w[1]; sreg[k + 2] = w[2]; sreg[k + 3] = w[3];
                        }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
            }
        } else if (cached) {
#pragma unroll
            for (int k = 0; k < PLAN_PER_MAX; ++k) sreg[k] = j0 + k < j1 ? st[j0 + k] : 0;
        }
        if (!self_hist) {
#pragma unroll
            for (int q = 0; q < 4; ++q) hreg[q] = ps[PS_HIST + 4 * tid + q];   // written by the previous kernel
        }
    }
    n_unm = scan.sum(n_unm);
    int e = L + (int)n_unm - C;
    if (e < 0) e = 0;
    int n_victims = 0;
    if (e > 0) {  // uniform over the head's workgroups: the cache is full, evict the e oldest untouched slots
        // visit_tok(f): f(token, slot) for the merged tokens this thread looks after
        auto visit_tok = [&](auto &&f) {
            if (tok_cached) {
#pragma unroll
                for (int k = 0; k < PLAN_TOK_MAX; ++k)
                    if (tj[k] >= 0) f(tid + k * PLAN_THREADS, tj[k]);
            } else {
                for (int i = tid; i < n_new; i += PLAN_THREADS)
                    if (merged[tb + i]) f(i, jstar[tb + i]);
            }
        };
        // second round of loads: for the merged tokens, the record of their slot's group and the slot's stamp
        u64 wrec[PLAN_TOK_MAX];
        int wst[PLAN_TOK_MAX];
        if (tok_cached && !self_hist) {
#pragma unroll
            for (int k = 0; k < PLAN_TOK_MAX; ++k) {
                wrec[k] = tj[k] >= 0 ? win[cb + tj[k]] : 0ull;
                wst[k] = tj[k] >= 0 ? st[tj[k]] : 0;
            }
        }
        const int n_words = (span + 31) / 32 + 1;
        for (int w = tid; w < n_words; w += PLAN_THREADS) touched[w] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) lhist[4 * tid + q] = hreg[q];
        __syncthreads();
        visit_tok([&](int, int j) {
            if (j >= s0 && j < s1) atomicOr(&touched[(j - s0) >> 5], 1u << ((j - s0) & 31));
        });
        __syncthreads();
        u64 elig = 0;  // bit k: slot j0 + k is live and untouched
        if (cached && j0 < j1) {   // the run's bits of the bitmap: 64 bits from bit j0 - s0 on, out of three words
            const int o = j0 - s0, w0 = o >> 5, sh = o & 31;
            u64 t = (u64)touched[w0] | ((u64)touched[w0 + 1] << 32);
            if (sh) t = (t >> sh) | ((u64)touched[w0 + 2] << (64 - sh));
            const int n = j1 - j0;
            elig = ~t & (n >= 64 ? ~0ull : ((1ull << n) - 1ull));
        }
        // visit(f): f(slot, key) for the eligible slots of this thread's run, ascending; key: larger = older
        auto visit = [&](auto &&f) {
            if (cached) {
#pragma unroll
                for (int k = 0; k < PLAN_PER_MAX; ++k)
                    if ((elig >> k) & 1ull) f(j0 + k, ~((unsigned)sreg[k] ^ 0x80000000u));
            } else {
                for (int j = j0; j < j1; ++j)
                    if (!((touched[(j - s0) >> 5] >> ((j - s0) & 31)) & 1u)) f(j, ~((unsigned)st[j] ^ 0x80000000u));
            }
        };
        // thread t owns the four bins 1023-4t .. 1020-4t of a histogram gh in global memory (descending keys):
        // finds the bin in which the want-th largest entry lies and the number of entries above that bin
        auto search = [&](const unsigned (&c4)[4], unsigned want, unsigned &total, unsigned &bin, unsigned &above) {
            const unsigned mine = c4[0] + c4[1] + c4[2] + c4[3];
            unsigned before = scan.excl_sum(mine, total);
            if (tid == 0) sh_bin = 0xFFFFFFFFu;
            __syncthreads();
            if (before < want && want <= before + mine) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (before < want && want <= before + c4[q]) {
                        sh_bin = PLAN_BINS - 1 - (4 * tid + q);
                        sh_above = before;
                    }
                    before += c4[q];
                }
            }
            __syncthreads();
            bin = sh_bin;
            above = sh_above;
            __syncthreads();
        };
        bool take_all = false;
        unsigned T = 0, need = (unsigned)e, cnt_el = 0;
        // Fast path: the verify launch left the histogram of all live slots' ages; subtract the slots touched in this
        // frame (each counted once, by the token that represents its group) and read the threshold off it.  Every
        // workgroup does this on the same data, so no meeting is needed.  It does not apply when a stamp lies in
        // the future or the threshold falls into the last bin (ages >= 1023 lumped together).
        // With self_hist the launch before left no histogram (a long cache: reading every stamp there as well costs more
        // than one meeting here): every workgroup counts the ages of its eligible slots from the stamps it holds, a run of
        // equal ages with one addition, the head's workgroups add their bins up in global memory and meet once.
        bool fast = self_hist ? true : ps[PS_FUT] == 0u;   // written by the previous kernel
        unsigned c4[4] = {0u, 0u, 0u, 0u};
        if (fast) {
            if (self_hist) {
                bool future = false;
                unsigned run_bin = 0u, run_n = 0u;
                visit([&](int, unsigned u) {
                    const int sv = (int)(~u ^ 0x80000000u);   // the stamp behind the key
                    future = future || sv > frame_id;
                    const unsigned bin = min((unsigned)frame_id - (unsigned)sv, (unsigned)(PLAN_BINS - 1));
                    if (bin != run_bin && run_n) {
                        atomicAdd(&lhist[run_bin], run_n);
                        run_n = 0u;
                    }
                    run_bin = bin;
                    run_n += 1u;
                });
                if (run_n) atomicAdd(&lhist[run_bin], run_n);
                __syncthreads();
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (lhist[4 * tid + q]) atomicAdd(&ps[PS_HIST + 4 * tid + q], lhist[4 * tid + q]);
                if (__any(future) && lane == 0) atomicOr(&ps[PS_FUT], 1u);
                head_barrier(&ps[PS_BAR + 3], NB, &ps[PS_ERR], pw);
#pragma unroll
                for (int q = 0; q < 4; ++q) c4[q] = ld_agent(&ps[PS_HIST + PLAN_BINS - 1 - (4 * tid + q)]);
                fast = ld_agent(&ps[PS_FUT]) == 0u;   // uniform over the head
            } else {
            if (tok_cached) {
#pragma unroll
                for (int k = 0; k < PLAN_TOK_MAX; ++k)
                    if (tj[k] >= 0 && (int)(0xFFFFFFFFu - (unsigned)wrec[k]) == tid + k * PLAN_THREADS) {
                        const unsigned age = (unsigned)frame_id - (unsigned)wst[k];
                        atomicSub(&lhist[min(age, (unsigned)(PLAN_BINS - 1))], 1u);
                    }
            } else {
                visit_tok([&](int i, int j) {
                    if ((int)(0xFFFFFFFFu - (unsigned)win[cb + j]) == i) {
                        const unsigned age = (unsigned)frame_id - (unsigned)st[j];
                        atomicSub(&lhist[min(age, (unsigned)(PLAN_BINS - 1))], 1u);
                    }
                });
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q) c4[q] = lhist[PLAN_BINS - 1 - (4 * tid + q)];
            }
        }
        if (fast) {
            unsigned bin, above;
            search(c4, (unsigned)e, cnt_el, bin, above);
            take_all = cnt_el <= (unsigned)e;
            if (!take_all) {
                if (bin >= (unsigned)(PLAN_BINS - 1)) {
                    fast = false;
                } else {
                    T = ~((unsigned)(frame_id - (int)bin) ^ 0x80000000u);  // key of the stamp frame_id - bin
                    need = (unsigned)e - above;
                }
            }
        }
        if (!fast) {
            // General path: range of the keys and number of eligible slots over the whole head, then a histogram
            // select on that range (a second histogram inside the threshold bin when the range is wider than the
            // bins), the workgroups of the head meeting between the steps.
            {
                unsigned kmin = 0xFFFFFFFFu, kmax = 0u, c = 0u;
                visit([&](int, unsigned u) {
                    kmin = min(kmin, u);
                    kmax = max(kmax, u);
                    c += 1;
                });
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) {
                    kmin = min(kmin, shfl_xor(kmin, off));
                    kmax = max(kmax, shfl_xor(kmax, off));
                }
                if (lane == 0) {
                    red_a[wave] = kmin;
                    red_b[wave] = kmax;
                }
                c = scan.sum(c);  // its barriers also publish red_a / red_b
                if (tid == 0 && c > 0) {
                    kmin = 0xFFFFFFFFu;
                    kmax = 0u;
                    for (int w = 0; w < PLAN_WAVES; ++w) {
                        kmin = min(kmin, red_a[w]);
                        kmax = max(kmax, red_b[w]);
                    }
                    atomicMax(&ps[PS_MAXK], kmax);
                    atomicMax(&ps[PS_MAXNK], ~kmin);
                    atomicAdd(&ps[PS_TOT], c);
                }
            }
            head_barrier(&ps[PS_BAR + 0], NB, &ps[PS_ERR], pw);
            const unsigned umax = ld_agent(&ps[PS_MAXK]), umin = ~ld_agent(&ps[PS_MAXNK]);
            cnt_el = ld_agent(&ps[PS_TOT]);
            take_all = cnt_el <= (unsigned)e;  // fewer eligible slots than evictions needed: take them all
            T = umax;
            need = (unsigned)e;
            if (!take_all) {
                // Among the keys in [lo, lo + width), with `want` of them to take from the top: histogram over the
                // head (bin = (key - lo) >> sh), then the bin in which the want-th largest key lies.
                auto level = [&](unsigned lo, unsigned width, int sh, unsigned want, int which, unsigned &bin, unsigned &above) {
                    for (int k = tid; k < PLAN_BINS; k += PLAN_THREADS) lhist[k] = 0;
                    __syncthreads();
                    visit([&](int, unsigned u) {
                        const unsigned rel = u - lo;
                        if (u >= lo && rel < width && (rel >> sh) < (unsigned)PLAN_BINS) atomicAdd(&lhist[rel >> sh], 1u);
                    });
                    __syncthreads();
                    unsigned *gh = ps + PS_HIST + (1 + which) * PLAN_BINS;
                    for (int k = tid; k < PLAN_BINS; k += PLAN_THREADS)
                        if (lhist[k]) atomicAdd(&gh[k], lhist[k]);
                    head_barrier(&ps[PS_BAR + 1 + which], NB, &ps[PS_ERR], pw);
                    unsigned c4[4], total;
#pragma unroll
                    for (int q = 0; q < 4; ++q) c4[q] = ld_agent(&gh[PLAN_BINS - 1 - (4 * tid + q)]);
                    search(c4, want, total, bin, above);
                };
                const unsigned range = umax - umin;
                int sh = 0;
                while ((range >> sh) >= (unsigned)PLAN_BINS) ++sh;
                unsigned bin, above;
                level(umin, 0xFFFFFFFFu, sh, (unsigned)e, 0, bin, above);
                if (sh == 0) {
                    T = umin + bin;
                    need = (unsigned)e - above;
                } else {  // resolve inside the coarse bin (ranges up to 2^20 frames; wider ones are not resolved exactly)
                    const unsigned lo2 = umin + (bin << sh);
                    const int sh2 = sh > 10 ? sh - 10 : 0;
                    if (sh2 > 0 && tid == 0) atomicOr(&ps[PS_ERR], 2u);
                    unsigned bin2, above2;
                    level(lo2, 1u << sh, sh2, (unsigned)e - above, 1, bin2, above2);
                    T = lo2 + (bin2 << sh2);
                    need = (unsigned)e - above - above2;
                }
            }
        }
        n_victims = take_all ? (int)cnt_el : e;
        // counts per workgroup, the workgroups meet, then ordered compaction: victims in ascending slot order
        unsigned c_gt = 0, c_eq = 0;
        visit([&](int, unsigned u) {
            c_gt += (take_all || u > T) ? 1u : 0u;
            c_eq += (!take_all && u == T) ? 1u : 0u;
        });
        unsigned blk_gt, blk_eq;
        scan.excl_sum(c_gt, blk_gt);
        const unsigned eq_base_thr = scan.excl_sum(c_eq, blk_eq);
        // Publish this workgroup's counts as one 64-bit word with a valid bit, then wait (bounded) for the words of
        // the workgroups below: only those are needed for the positions, and the wait doubles as the read.
        u64 *blk = (u64 *)(ps + PS_BLK);
        if (tid == 0)
            __hip_atomic_store(&blk[b], (1ull << 63) | ((u64)blk_gt << 32) | (u64)blk_eq, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        if (tid < b) {
            u64 v = 0;
            int spins = 0;
            while (!((v = __hip_atomic_load(&blk[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 63)) {
                if (++spins > pw.spin_limit) {
                    atomicOr(&ps[PS_ERR], 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
            sh_blk[2 * tid] = (unsigned)(v >> 32) & 0x7FFFFFFFu;
            sh_blk[2 * tid + 1] = (unsigned)v;
        }
        __syncthreads();
        unsigned pos_base = 0, eq_before = 0;
        for (int bb = 0; bb < b; ++bb) {
            const unsigned g = sh_blk[2 * bb], q = sh_blk[2 * bb + 1];
            const unsigned tk = eq_before >= need ? 0u : min(q, need - eq_before);
            pos_base += g + tk;
            eq_before += q;
        }
        const unsigned eq_blk_take = eq_before >= need ? 0u : min(blk_eq, need - eq_before);  // ties this workgroup takes
        const unsigned eq_take = eq_base_thr >= eq_blk_take ? 0u : min(c_eq, eq_blk_take - eq_base_thr);
        unsigned tot;
        unsigned pos = pos_base + scan.excl_sum(c_gt + eq_take, tot);
        unsigned eq_seen = 0;
        visit([&](int j, unsigned u) {
            bool take = take_all || u > T;
            if (!take_all && u == T) {
                take = eq_seen < eq_take;
                eq_seen += 1;
            }
            if (take) {
                if (pos < (unsigned)n_new) victims[tb + pos] = j;
                pos += 1;
            }
        });
    }
    if (b == 0 && tid == 0) {
        const int n_dropped = e - n_victims;
        const int n_app = (int)n_unm - n_dropped;
        const int newL = L + n_app - n_victims;
        int32_t *o = hs + (size_t)h * HS_STRIDE;
        const int mark = o[7];
        o[0] = L; o[1] = (int)n_unm; o[2] = e; o[3] = n_victims; o[4] = n_dropped; o[5] = newL;
        int32_t *s = stats + (size_t)h * 8;
        s[0] = newL; s[1] = n_new - (int)n_unm; s[2] = n_app; s[3] = n_victims; s[4] = n_dropped;
        // bit 0 of the error word (a wait ran out) may still be raised by a workgroup that finishes later: the apply
        // launch looks again and, if it is set, leaves the head's cache as it was
        const unsigned err = e > 0 ? ld_agent(&ps[PS_ERR]) : 0u;
        int status = (err & 1u) ? 1 : (err & 2u) ? 2 : 0;
        // a workspace declared persistent must be a zero-filled one or one a finished call left behind
        if (ws_persistent && mark != 0 && mark != WS_CLEAN) status = 3;
        o[6] = status == 3 ? 3 : 0;   // for the apply launch: records and scratch of this workspace mean nothing
        s[5] = 0; s[6] = 0; s[7] = status;
    }
}

// workgroups per head of tc_plan_kernel and its dynamic LDS (the touched bitmap of one workgroup's slot range).
// The workgroups of a head wait for each other, so the whole grid has to be resident at once.  What a compute unit
// holds of the kernel's instantiations without dynamic LDS (registers, wavefront slots) and the number of compute units
// are asked of the runtime once per device; with LDS (bitmap + about 5 KB of static arrays) fewer may fit its 160 KB.
// The grid (nb + 1) * H stays within that (and within PLAN_MAX_GRID).
struct PlanResidency {
    int per_cu, n_cu;
};
static int plan_residency(PlanResidency *out) {
    static DeviceOnce once;
    static PlanResidency table[DeviceOnce::MAX_DEVICES];
    const int rc = once.run([](int dev) {
        int least = INT_MAX, n_cu = 0;
        const void *kernels[4] = {(const void *)tc_plan_kernel<64, 16>, (const void *)tc_plan_kernel<64, 8>,
                                  (const void *)tc_plan_kernel<16, 16>, (const void *)tc_plan_kernel<16, 8>};
        for (const void *k : kernels) {
            int n = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, PLAN_THREADS, 0) != hipSuccess) return FASTAR_ERR_HIP;
            least = std::min(least, n);
        }
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return FASTAR_ERR_HIP;
        if (least < 1 || n_cu < 1) return FASTAR_ERR_HIP;
        table[dev] = {least, n_cu};
        return FASTAR_OK;
    });
    if (rc != FASTAR_OK) return rc;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return FASTAR_ERR_HIP;
    *out = table[dev];
    return FASTAR_OK;
}
static int plan_residency_setup() {
    PlanResidency pr;
    return plan_residency(&pr);
}
static size_t plan_lds_bytes(int C, int nb) { return ((size_t)((C + nb - 1) / nb + 3 + 31) / 32 + 2) * 4; }
static int plan_nb(int H, int C, PlanResidency pr) {
    int nb = (C + 2047) / 2048;
    if (nb > PLAN_NB_MAX) nb = PLAN_NB_MAX;
    if (nb < 1) nb = 1;
    for (; nb > 1; --nb) {
        // static arrays: about 5 KB, and 16 KB more in the instantiation for long runs (the hand-over area of the stamps)
        const bool long_runs = ((C + nb - 1) / nb + PLAN_THREADS - 1) / PLAN_THREADS > 16;
        const size_t lds = plan_lds_bytes(C, nb) + (long_runs ? 21 : 5) * 1024;
        size_t per_cu = (size_t)160 * 1024 / lds;
        if (per_cu > (size_t)pr.per_cu) per_cu = (size_t)pr.per_cu;
        size_t resident = per_cu * (size_t)pr.n_cu;
        if (resident > (size_t)PLAN_MAX_GRID) resident = PLAN_MAX_GRID;
        if ((size_t)(nb + 1) * (size_t)H <= resident) break;
    }
    return nb;
}

// ---- apply ---------------------------------------------------------------------------------------------
// Token i of head h, merged into slot j: the group's representative refreshes the slot.  kraw / vraw: the token's own rows,
// cw: its code word of this lane.  Whole 16-lane groups; sub: which of the wavefront's.
template <bool BF16, int D>
__device__ __forceinline__ void apply_merged_token(void *__restrict__ K, void *__restrict__ V, int8_t *__restrict__ code,
                                                   int32_t *__restrict__ cnt, int32_t *__restrict__ stamp, int r,
                                                   const void *__restrict__ K_new, const void *__restrict__ V_new,
                                                   const int8_t *__restrict__ ck, int n_new, int frame_id,
                                                   const int32_t *__restrict__ jstar, const uint8_t *__restrict__ merged,
                                                   u64 *win, int32_t *grp, int rep_mode, size_t tb, size_t cb, int i, int j,
                                                   int l16, int sub, const typename RowPiece<BF16, D>::Raw &kraw,
                                                   const typename RowPiece<BF16, D>::Raw &vraw, unsigned cw) {
    typedef RowPiece<BF16, D> RP;
    // second round of loads, everything addressed by the slot at once: its records and multiplicity, and already
    // its value row (and key row for the mean key), which only the group's representative goes on to use
    const bool mean_key = rep_mode == 1;
    float acc[RP::EPL], vn[RP::EPL], kacc[RP::EPL], kn[RP::EPL];
    const u64 wkey = win[cb + j];
    const int gc = grp[cb + j];
    const int m0 = cnt[cb + j];
    RP::load(V, cb + j, l16, acc);
    if (mean_key) RP::load(K, cb + j, l16, kacc);
    const int widx = (int)(0xFFFFFFFFu - (unsigned)wkey);
    if (widx == i) {  // this token represents the group: it refreshes the slot
        // ... and clears the group's records behind it: the other joiners only look for their own index in the
        // record, which neither the old nor the cleared value shows them
        if (l16 == 0) {
            win[cb + j] = 0;
            grp[cb + j] = 0;
        }
        // mean value; with rep_mode 1 also the mean key, whose stored bits feed later integer decisions: single
        // float32 operations in a fixed order (multiplicity * old row, members in ascending token order, one division)
#pragma unroll
        for (int e = 0; e < RP::EPL; ++e) acc[e] *= (float)m0;
        if (mean_key) {
#pragma unroll
            for (int e = 0; e < RP::EPL; ++e) kacc[e] = __fmul_rn((float)m0, kacc[e]);
        }
        if (gc == 1) {
            RP::unpack(vraw, vn);
#pragma unroll
            for (int e = 0; e < RP::EPL; ++e) acc[e] += vn[e];
            if (mean_key) {
                RP::unpack(kraw, kn);
#pragma unroll
                for (int e = 0; e < RP::EPL; ++e) kacc[e] = __fadd_rn(kacc[e], kn[e]);
            }
        } else {  // several joiners: add their rows in ascending token order
            for (int base = 0; base < n_new; base += 16) {
                const int t = base + l16;
                const bool member = t < n_new && merged[tb + t] && jstar[tb + t] == j;
                unsigned mm = (unsigned)((__ballot(member) >> (16 * sub)) & 0xFFFFull);
                while (mm) {
                    const int bit = __ffs(mm) - 1;
                    mm &= mm - 1;
                    RP::load(V_new, tb + base + bit, l16, vn);
#pragma unroll
                    for (int e = 0; e < RP::EPL; ++e) acc[e] += vn[e];
                    if (mean_key) {
                        RP::load(K_new, tb + base + bit, l16, kn);
#pragma unroll
                        for (int e = 0; e < RP::EPL; ++e) kacc[e] = __fadd_rn(kacc[e], kn[e]);
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < RP::EPL; ++e) acc[e] = __fdiv_rn(acc[e], (float)(m0 + gc));
        RP::store(V, cb + j, l16, acc);
        if (mean_key) {   // the slot's code follows in tc_recode_kernel, from the stored row
#pragma unroll
            for (int e = 0; e < RP::EPL; ++e) kacc[e] = __fdiv_rn(kacc[e], (float)(m0 + gc));
            RP::store(K, cb + j, l16, kacc);
        } else if (rep_mode == 2) {
            // Medoid key: of {stored key (weight m0), joiners (weight 1)} the member x with the smallest
            // cost(x) = sum_y w_y |x - y|^2 in code space = W |x|^2 + S2 - 2 x . S1 (W = sum of the weights,
            // S1 = weighted sum of the codes, S2 = weighted sum of their squared norms): exact integers, one pass to
            // build the sums and one to evaluate the candidates (stored key first, then tokens ascending; a later
            // candidate wins only on a strictly smaller cost).  Lane l16 owns code word l16 (r <= 64: 16 words).
            // A single joiner never wins: cost(stored) = |d|^2 <= m0 |d|^2 = cost(joiner).
            if (gc > 1) {
                const bool has_w = l16 < r / 4;
                const unsigned ow = has_w ? ((const unsigned *)(code + (cb + j) * r))[l16] : 0u;
                long long S1[4], S2 = (long long)m0 * dot4_i8(ow, ow, 0);
#pragma unroll
                for (int k = 0; k < 4; ++k) S1[k] = (long long)m0 * (int)(signed char)(ow >> (8 * k));
                for (int base = 0; base < n_new; base += 16) {
                    const int t = base + l16;
                    const bool member = t < n_new && merged[tb + t] && jstar[tb + t] == j;
                    unsigned mm = (unsigned)((__ballot(member) >> (16 * sub)) & 0xFFFFull);
                    while (mm) {
                        const int bit = __ffs(mm) - 1;
                        mm &= mm - 1;
                        const unsigned w = has_w ? ((const unsigned *)(ck + (tb + base + bit) * r))[l16] : 0u;
                        S2 += dot4_i8(w, w, 0);
#pragma unroll
                        for (int k = 0; k < 4; ++k) S1[k] += (int)(signed char)(w >> (8 * k));
                    }
                }
                const long long W = (long long)m0 + gc;
                auto group16_sum64 = [](long long v) -> long long {
#pragma unroll
                    for (int off = 1; off < 16; off <<= 1) {
                        const unsigned lo = shfl_xor((unsigned)v, off), hi = shfl_xor((unsigned)((unsigned long long)v >> 32), off);
                        v += (long long)(((unsigned long long)hi << 32) | lo);
                    }
                    return v;
                };
                auto cost_of = [&](unsigned w) -> long long {   // this lane's share of W |x|^2 + S2 - 2 x . S1
                    long long c = W * dot4_i8(w, w, 0) + S2;
#pragma unroll
                    for (int k = 0; k < 4; ++k) c -= 2 * S1[k] * (int)(signed char)(w >> (8 * k));
                    return c;
                };
                long long best_cost = group16_sum64(cost_of(ow));
                int best = -1;   // the stored key
                for (int base = 0; base < n_new; base += 16) {
                    const int t = base + l16;
                    const bool member = t < n_new && merged[tb + t] && jstar[tb + t] == j;
                    unsigned mm = (unsigned)((__ballot(member) >> (16 * sub)) & 0xFFFFull);
                    while (mm) {
                        const int bit = __ffs(mm) - 1;
                        mm &= mm - 1;
                        const unsigned w = has_w ? ((const unsigned *)(ck + (tb + base + bit) * r))[l16] : 0u;
                        const long long c = group16_sum64(cost_of(w));
                        if (c < best_cost) {
                            best_cost = c;
                            best = base + bit;
                        }
                    }
                }
                if (best >= 0) {
                    RP::copy(K, cb + j, K_new, tb + best, l16);
                    if (has_w) ((unsigned *)(code + (cb + j) * r))[l16] = ((const unsigned *)(ck + (tb + best) * r))[l16];
                }
            }
        } else {
            RP::store_raw(K, cb + j, l16, kraw);
            if (l16 < r / 4) ((unsigned *)(code + (cb + j) * r))[l16] = cw;
        }
        if (l16 == 0) {
            cnt[cb + j] = m0 + gc;
            stamp[cb + j] = frame_id;
        }
    }
}

template <bool BF16, int D>
__global__ __launch_bounds__(256) void tc_apply_kernel(void *__restrict__ K, void *__restrict__ V, int8_t *__restrict__ code,
                                                       int32_t *__restrict__ cnt, int32_t *__restrict__ stamp, int C,
                                                       int r, const void *__restrict__ K_new,
                                                       const void *__restrict__ V_new, const int8_t *__restrict__ ck,
                                                       int n_new, int frame_id, const int32_t *__restrict__ jstar,
                                                       const uint8_t *__restrict__ merged, u64 *win, int32_t *grp,
                                                       const int32_t *__restrict__ rank,
                                                       const int32_t *__restrict__ victims, int32_t *hs,
                                                       int32_t *__restrict__ merge_map, int32_t *__restrict__ len,
                                                       int rep_mode, unsigned *__restrict__ ps_all, int ps_words,
                                                       int32_t *__restrict__ stats) {
    typedef RowPiece<BF16, D> RP;
    const int h = blockIdx.y;
    // A wait of the plan ran out for this head (bit 0 of its error word; every workgroup of this launch sees it, because
    // none clears the scratch words then): the victims are not to be trusted, so nothing of the head is applied.  Its
    // cache stays as it was before the call, every token counts as dropped, and the workspace is marked as not clean.
    // The same when the workspace was declared persistent but is neither zero-filled nor left by a finished call
    // (status 3, word 6 of the head's scalars): its records mean nothing.
    const bool ws_dirty = hs[(size_t)h * HS_STRIDE + 6] == 3;
    if (ws_dirty || (ps_all[(size_t)h * ps_words + PS_ERR] & 1u)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            int32_t *s = stats + (size_t)h * 8;
            s[0] = hs[(size_t)h * HS_STRIDE + 0]; s[1] = 0; s[2] = 0; s[3] = 0; s[4] = n_new; s[5] = 0; s[6] = 0;
            s[7] = ws_dirty ? 3 : 1;
            if (!ws_dirty) hs[(size_t)h * HS_STRIDE + 7] = WS_FAILED;
        }
        const int i = blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4);
        if (i < n_new && (threadIdx.x & 15) == 0) {
            merge_map[(size_t)h * n_new + i] = -1;
            const_cast<uint8_t *>(merged)[(size_t)h * n_new + i] = 0;
        }
        return;
    }
    // the new length is published here and not by the plan: its workgroups read len[h] at different times
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        len[h] = hs[(size_t)h * HS_STRIDE + 5];
        hs[(size_t)h * HS_STRIDE + 7] = WS_CLEAN;   // with the two clean-ups below: the workspace is left as a zero-filled one
    }
    // the plan is done with its scratch words: cleared for the next call that shares this workspace
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < ps_words; k += gridDim.x * blockDim.x)
        ps_all[(size_t)h * ps_words + k] = 0u;
    const int l16 = threadIdx.x & 15;
    const int sub = (threadIdx.x & 63) >> 4;  // which 16-lane group of the wavefront
    const int i = blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4);
    if (i >= n_new) return;
    const size_t tb = (size_t)h * n_new, ti = tb + i, cb = (size_t)h * C;
    const int32_t *o = hs + (size_t)h * HS_STRIDE;
    const int L = o[0], n_unm = o[1], n_victims = o[3], n_dropped = o[4];
    // First round of loads, all addressed by the token: flags, destination data, and the token's own rows (bit
    // copies).  The second round (records and value row of the slot, or the victim slot) depends on them.
    const bool mg = merged[ti] != 0;
    const int j = jstar[ti];
    const int a = rank[ti];
    typename RP::Raw kraw = RP::load_raw(K_new, ti, l16), vraw = RP::load_raw(V_new, ti, l16);
    unsigned cw = 0;
    if (l16 < r / 4) cw = ((const unsigned *)(ck + ti * r))[l16];
    int dst = -1;
    if (mg) {
        dst = j;
        apply_merged_token<BF16, D>(K, V, code, cnt, stamp, r, K_new, V_new, ck, n_new, frame_id, jstar, merged, win, grp,
                                    rep_mode, tb, cb, i, j, l16, sub, kraw, vraw, cw);
    } else if (a < n_unm - n_dropped) {
        dst = a < n_victims ? victims[tb + a] : L + (a - n_victims);
        // A plan whose bounded wait ran out (stats[7] = 1) may have left victim positions unwritten: whatever they
        // hold, nothing is stored outside the cache; such a token counts as not placed.
        if ((unsigned)dst >= (unsigned)C) dst = -1;
    }
    if (!mg && dst >= 0) {
        RP::store_raw(K, cb + dst, l16, kraw);
        RP::store_raw(V, cb + dst, l16, vraw);
        if (l16 < r / 4) ((unsigned *)(code + (cb + dst) * r))[l16] = cw;
        if (l16 == 0) {
            cnt[cb + dst] = 1;
            stamp[cb + dst] = frame_id;
        }
    }
    if (l16 == 0) merge_map[ti] = dst;
}

// ---- plan and apply in one launch ----------------------------------------------------------------------
// On a persistent workspace and a cache of at most SETTLE_SLOTS slots nothing that the plan decides needs a meeting: the
// threshold age follows from the slices' age histograms less the slots touched in this frame, and so do the numbers of
// victims in the slices below.  Every workgroup works that out for itself (the same data, the same answer) and goes
// straight on to its share of the rows:
//   - workgroups below n_slices * n_reps: (slice, share).  The slice's victims in ascending order, from its slots' ages; the
//     rows of every n_reps-th of them, starting with the share's, are replaced by those of the unmerged tokens of their
//     rank.  Where the threshold's bin may hold several stamps (age_bin), they select among the bin's stamps first, each for
//     itself and from the copies that the match launch left: ages of 2000 and more, call at 12 heads x 1560 tokens x 37440
//     slots 160 us by one workgroup on the stamps themselves (53 with the plan's meetings) -> 51; one stamp in the future 168 -> 33.
//   - the others: 32 tokens each; the merged ones refresh their slots, the unmerged ones that found no victim are
//     appended.
// They write what no other one reads: a slot is touched or a victim or new; tokens' flags and slots, the old length, the
// touched slots' old stamps, every slot's age and the histograms were left by the match and verify launches.
// What bounds it: the chain of a workgroup.  At 12 heads x 1560 tokens and 37440 slots (timestamps inside the kernel, us, of the
// workgroups for victims): first loads 2.6, lists, bitmap and histogram 3.2, threshold 0.7, slice 1.0, rows 0.7 on average
// and 4 at most; the token workgroups are done after 6.  Launch 16.5, where the plan (17 workgroups per head, one
// meeting) took 13.5 and the apply launch behind it 9.3; a chunk of three such calls 325 -> 293.
// All 888 workgroups have to be resident at once: with 99 registers they took two rounds and 23.8 us, so frames of up to
// 2048 tokens have an instantiation of 64 (it spills 4 words).
constexpr int SETTLE_WAVES = SETTLE_THREADS / 64;
constexpr int SETTLE_GROUPS = SETTLE_THREADS / 16;             // 16-lane groups: rows a workgroup moves at a time
constexpr int SETTLE_SPT = SETTLE_SLICE / SETTLE_THREADS;      // slots per thread of a slice
static_assert(SETTLE_SPT == 16 && AGE_BINS == 2 * SETTLE_THREADS, "a thread's slots are half a bitmap word, its bins two");
// dynamic LDS: bitmap of the touched slots, unmerged tokens by rank, victims of the slice (and a word for what is none)
static size_t settle_lds_bytes(int C, int n_new) {
    return (size_t)((C + 63) / 64) * 8 + (size_t)((n_new + 7) & ~7) * 2 + SETTLE_SLICE * 2 + 16;
}

// Workgroups of tc_settle_kernel, per head, and whether it is the better way.  Shares of a slice's victims: as many as would have
// 64 rows each if nothing merged; every one of them reads the frame's lists, so 128 rows in the form for frames of more than
// 2048 tokens once its workgroups are more than reside at once (512).  Beyond that it is a question of how many times over:
// plan and apply launches against the one, us per call, bf16, d = 128 (workgroups):
//   up to 2048 tokens, at any size measured: 40 heads x 1560 x 37440 slots (2960) 72 -> 70, 40 x 2048 x 63488 (4800) 99 -> 99,
//     12 x 1560 x 37440 (888) 39 -> 33, fp32 24 x 2048 x 49152 (2496) 83 -> 69;
//   up to 4096: 5 x 3600 x 64800 (885) 59 -> 54, 14 x 3600 x 57600 (2030) 78 -> 74, 16 x 3600 x 57600 (2320) 85 -> 84,
//     16 x 4096 x 61440 (2560) 146 -> 152, 40 x 2100 x 42000 (3360) 97 -> 104, 40 x 3600 x 21600 (5720) 144 -> 166;
//   longer ones, which the plan reads again and again: 4 x 8000 x 64000 160 -> 119, 20 x 8000 x 64000 (6280) 462 -> 448,
//     30 x 6000 x 30000 (7080) 411 -> 417, 40 x 8000 x 24000 (12520) 838 -> 868.
struct SettleGrid {
    int n_reps, wgs;   // shares per slice; workgroups per head
    bool better;
};
static SettleGrid settle_grid(int H, int C, int n_new) {
    const int n_slices = settle_slices(C), tok_wgs = (n_new + SETTLE_GROUPS - 1) / SETTLE_GROUPS;
    SettleGrid g;
    for (int rows = 64; rows <= 128; rows *= 2) {
        g.n_reps = ((n_new + rows - 1) / rows + n_slices - 1) / n_slices;
        g.wgs = n_slices * g.n_reps + tok_wgs;
        if (n_new <= 2048 || (int64_t)g.wgs * H <= 512) break;
    }
    g.better = n_new <= 2048 || (int64_t)g.wgs * H <= (n_new <= 4096 ? 2400 : 6400);
    return g;
}

struct Pair {
    unsigned a, b;
};
// Exclusive prefix over the workgroup's threads of two counts at once, and their totals.  wtot: two sets, used in turn, so that
// one barrier is enough.
__device__ __forceinline__ Pair settle_scan(Pair v, Pair (*wtot)[SETTLE_WAVES], int &turn, Pair &total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const Pair incl = {wave_incl_scan(v.a), wave_incl_scan(v.b)};
    Pair *wt = wtot[turn];
    turn ^= 1;
    if (lane == 63) wt[wave] = incl;
    __syncthreads();
    Pair pos = {incl.a - v.a, incl.b - v.b};
    total = {0u, 0u};
#pragma unroll
    for (int w = 0; w < SETTLE_WAVES; ++w) {
        const Pair c = wt[w];
        pos.a += w < wave ? c.a : 0u;
        pos.b += w < wave ? c.b : 0u;
        total.a += c.a;
        total.b += c.b;
    }
    return pos;
}

// TPT: tokens of the list per thread (4: frames of up to 2048 tokens; 16).
template <bool BF16, int D, int TPT>
__global__ __launch_bounds__(SETTLE_THREADS, TPT == 4 && BF16 ? 8 : 4) void tc_settle_kernel(
    void *__restrict__ K, void *__restrict__ V, int8_t *__restrict__ code, int32_t *__restrict__ cnt,
    int32_t *__restrict__ stamp, int C, int r, const void *__restrict__ K_new, const void *__restrict__ V_new,
    const int8_t *__restrict__ ck, int n_new, int frame_id, const int32_t *__restrict__ jstar, uint8_t *merged, u64 *win,
    int32_t *grp, int32_t *hs, int32_t *__restrict__ merge_map, int32_t *__restrict__ len, int rep_mode,
    const int32_t *__restrict__ tstamp, const unsigned *__restrict__ ages, const unsigned short *__restrict__ slot_age,
    const int32_t *__restrict__ slot_stamp, int n_reps, int32_t *__restrict__ stats) {
    typedef RowPiece<BF16, D> RP;
    extern __shared__ __attribute__((aligned(16))) unsigned char slds[];
    __shared__ unsigned h_all[AGE_BINS], h_low[AGE_BINS];   // ages of the head's eligible slots, and of those below this slice
    __shared__ Pair wtot[2][SETTLE_WAVES];
    __shared__ int kcnt[TPT * SETTLE_WAVES];
    __shared__ int sh[4];
    int turn = 0;
    const int h = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int l16 = tid & 15, group = tid >> 4, sub = lane >> 4;
    const int n_slices = settle_slices(C), n_evict_wgs = n_slices * n_reps;
    const size_t tb = (size_t)h * n_new, cb = (size_t)h * C;
    const int L = hs[(size_t)h * HS_STRIDE], mark = hs[(size_t)h * HS_STRIDE + 7];
    const bool dirty = mark != 0 && mark != WS_CLEAN;   // neither zero-filled nor left by a finished call: nothing is applied
    const bool maybe = L + n_new > C;                    // otherwise no eviction can be needed
    unsigned *touched = (unsigned *)slds;                // [ceil(C / 64) * 2]
    unsigned short *unm = (unsigned short *)(touched + 2 * ((C + 63) / 64));
    unsigned short *vict = unm + ((n_new + 7) & ~7);
    auto clear_touched = [&]() {
        for (int w = tid; w < 2 * ((C + 63) / 64); w += SETTLE_THREADS) touched[w] = 0u;
    };

    if ((int)blockIdx.x >= n_evict_wgs) {   // ---- tokens
        const int base = ((int)blockIdx.x - n_evict_wgs) * SETTLE_GROUPS;
        const int i = base + group;
        const bool ok = i < n_new;
        const size_t ti = tb + min(i, n_new - 1);
        // first round of loads: the token's flag, slot and rows, and everybody's flags
        const bool mg = merged[ti] != 0;
        const int j = jstar[ti];
        const typename RP::Raw kraw = RP::load_raw(K_new, ti, l16), vraw = RP::load_raw(V_new, ti, l16);
        unsigned cw = 0;
        if (l16 < r / 4) cw = ((const unsigned *)(ck + ti * r))[l16];
        uint8_t flag[TPT];
#pragma unroll
        for (int k = 0; k < TPT; ++k)
            flag[k] = k * SETTLE_THREADS < n_new ? merged[tb + min(k * SETTLE_THREADS + tid, n_new - 1)] : 1;
        if (dirty) {   // uniform over the head
            if (ok && l16 == 0) {
                merge_map[ti] = -1;
                merged[ti] = 0;
            }
            if (base == 0 && tid == 0) {
                int32_t *st = stats + (size_t)h * 8;
                st[0] = L; st[1] = 0; st[2] = 0; st[3] = 0; st[4] = n_new; st[5] = 0; st[6] = 0; st[7] = 3;
            }
            return;
        }
        unsigned n_mine = 0, n_below = 0;   // unmerged tokens among those this thread looks at, and of them below the workgroup's
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
            const int t = k * SETTLE_THREADS + tid;
            const bool u = t < n_new && flag[k] == 0;
            n_mine += u ? 1u : 0u;
            n_below += u && t < base ? 1u : 0u;
        }
        Pair tot;
        settle_scan({n_mine, n_below}, wtot, turn, tot);
        const int n_unm = (int)tot.a, first_rank = (int)tot.b;
        const int e = max(0, L + n_unm - C);
        int n_victims = e;
        if (e > L - (n_new - n_unm)) {   // there may be fewer untouched slots than that: count the touched ones
            clear_touched();
            __syncthreads();
            unsigned distinct = 0;
            for (int t = tid; t < n_new; t += SETTLE_THREADS)
                if (merged[tb + t]) {
                    const int s = jstar[tb + t];
                    distinct += (atomicOr(&touched[s >> 5], 1u << (s & 31)) >> (s & 31)) & 1u ? 0u : 1u;
                }
            settle_scan({distinct, 0u}, wtot, turn, tot);
            n_victims = min(e, L - (int)tot.a);
        }
        const int n_dropped = e - n_victims;
        // rank of an unmerged token: those below the workgroup's, then those before it in it
        if (l16 == 0) kcnt[group] = ok && !mg ? 1 : 0;
        __syncthreads();
        int a = first_rank;
#pragma unroll
        for (int q = 0; q < SETTLE_GROUPS; ++q) a += q < group ? kcnt[q] : 0;
        if (ok && mg) {
            apply_merged_token<BF16, D>(K, V, code, cnt, stamp, r, K_new, V_new, ck, n_new, frame_id, jstar, merged, win, grp,
                                        rep_mode, tb, cb, i, j, l16, sub, kraw, vraw, cw);
            if (l16 == 0) merge_map[ti] = j;
        } else if (ok && a >= n_victims) {   // appended, or dropped
            const int dst = a < n_unm - n_dropped ? L + (a - n_victims) : -1;
            if (dst >= 0) {
                RP::store_raw(K, cb + dst, l16, kraw);
                RP::store_raw(V, cb + dst, l16, vraw);
                if (l16 < r / 4) ((unsigned *)(code + (cb + dst) * r))[l16] = cw;
                if (l16 == 0) {
                    cnt[cb + dst] = 1;
                    stamp[cb + dst] = frame_id;
                }
            }
            if (l16 == 0) merge_map[ti] = dst;
        }
        if (base == 0 && tid == 0) {
            const int n_app = n_unm - n_dropped, newL = L + n_app - n_victims;
            int32_t *st = stats + (size_t)h * 8;
            st[0] = newL; st[1] = n_new - n_unm; st[2] = n_app; st[3] = n_victims; st[4] = n_dropped; st[5] = 0; st[6] = 0;
            st[7] = 0;
            len[h] = newL;   // the other workgroups read the length of before from hs
            hs[(size_t)h * HS_STRIDE + 7] = WS_CLEAN;
        }
        return;
    }

    // ---- victims
    const int slice = (int)blockIdx.x % n_slices, share = (int)blockIdx.x / n_slices;
    const unsigned *ag = ages + (size_t)h * n_slices * AGE_WORDS;
    // first round of loads: the tokens' flags, slots and slots' stamps, this thread's run of ages, two bins of every slice
    int tj[TPT], ts[TPT];
    uint8_t flag[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int t = min(k * SETTLE_THREADS + tid, n_new - 1);
        tj[k] = jstar[tb + t];
        ts[k] = tstamp[tb + t];
        flag[k] = merged[tb + t];
    }
    const int s0 = slice * SETTLE_SLICE;
    u32x4 run[2];   // ages of slots s0 + 16 tid .. +15
#pragma unroll
    for (int q = 0; q < 2; ++q)
        run[q] = *(const u32x4 *)(slot_age + ((size_t)h * n_slices + slice) * SETTLE_SLICE + SETTLE_SPT * tid + 8 * q);
    constexpr int MAX_SLICES = SETTLE_SLOTS / SETTLE_SLICE;
    u32x2 bins[MAX_SLICES];
    unsigned newest[MAX_SLICES];
#pragma unroll
    for (int q = 0; q < MAX_SLICES; ++q) {
        bins[q] = u32x2{0u, 0u};
        newest[q] = 0u;
        if (q < n_slices) {   // uniform
            bins[q] = *(const u32x2 *)(ag + (size_t)q * AGE_WORDS + 2 * tid);
            newest[q] = ag[(size_t)q * AGE_WORDS + AGE_BINS];
        }
    }
    if (!maybe || dirty) return;   // uniform over the head; after the loads, which do not depend on it
    unsigned all0 = 0, all1 = 0, low0 = 0, low1 = 0, kmax = 0;
#pragma unroll
    for (int q = 0; q < MAX_SLICES; ++q) {
        all0 += bins[q][0]; all1 += bins[q][1];
        low0 += q < slice ? bins[q][0] : 0u;
        low1 += q < slice ? bins[q][1] : 0u;
        kmax = max(kmax, newest[q]);
    }
    clear_touched();
    // unmerged tokens by rank (ascending token order): counts per wavefront and round, every wavefront adds them up itself
    unsigned tmask = 0, umask = 0;   // bit k: token k * SETTLE_THREADS + tid is merged / unmerged
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const bool in = k * SETTLE_THREADS + tid < n_new;
        tmask |= in && flag[k] != 0 ? 1u << k : 0u;
        umask |= in && flag[k] == 0 ? 1u << k : 0u;
        const u64 m = __ballot((umask >> k) & 1u);
        if (lane == 0) kcnt[k * SETTLE_WAVES + wave] = __popcll(m);
    }
    h_all[2 * tid] = all0; h_all[2 * tid + 1] = all1;
    h_low[2 * tid] = low0; h_low[2 * tid + 1] = low1;
    __syncthreads();
    constexpr int CPL = (TPT * SETTLE_WAVES + 63) / 64;   // counts per lane
    static_assert(CPL <= 2, "a wavefront holds all counts");
    int kc[CPL], kbase = 0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
        kc[q] = CPL * lane + q < TPT * SETTLE_WAVES ? kcnt[CPL * lane + q] : 0;
        kbase += kc[q];
    }
    const int kincl = (int)wave_incl_scan((unsigned)kbase);
    kbase = kincl - kbase;   // unmerged tokens before the first count of this lane
    const int n_unm = __builtin_amdgcn_readlane(kincl, 63), e = L + n_unm - C;
    if (e <= 0) return;   // uniform over the head
    unsigned fmask = 0;
#pragma unroll
    for (int k = 0; k < TPT; ++k)   // each touched slot counts once
        if ((tmask >> k) & 1u) fmask |= (((atomicOr(&touched[tj[k] >> 5], 1u << (tj[k] & 31)) >> (tj[k] & 31)) & 1u) ^ 1u) << k;
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const u64 m = __ballot((umask >> k) & 1u);
        const int c = k * SETTLE_WAVES + wave;   // uniform
        int base = __builtin_amdgcn_readlane(kbase, __builtin_amdgcn_readfirstlane(c / CPL));
        if (CPL == 2 && (c & 1)) base += __builtin_amdgcn_readlane(kc[0], __builtin_amdgcn_readfirstlane(c / CPL));
        if ((umask >> k) & 1u) unm[base + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)(k * SETTLE_THREADS + tid);
        const bool first = (fmask >> k) & 1u;
        const u64 fm = __ballot(first);
        if (fm) {   // uniform; most of them carry the stamp of the frame before: lanes of one age count together
            const unsigned bin = age_bin(frame_id, ts[k]);
            const int lead = __ffsll((unsigned long long)fm) - 1;
            const bool same = bin == (unsigned)__builtin_amdgcn_readlane((int)bin, lead), low = tj[k] < s0;
            const u64 sm = __ballot(first && same), lm = __ballot(first && same && low);
            if (lane == lead) {
                atomicSub(&h_all[bin], (unsigned)__popcll(sm));
                if (lm) atomicSub(&h_low[bin], (unsigned)__popcll(lm));
            }
            if (first && !same) {
                atomicSub(&h_all[bin], 1u);
                if (low) atomicSub(&h_low[bin], 1u);
            }
        }
    }
    __syncthreads();   // the lists, the bitmap and the histograms
    // Threshold: the bin, from the oldest on, in which the e-th slot lies; `need` of it are taken.  Victims: the slots of older
    // bins, and of this one those with the smallest stamps, ties in slot order.  low_*: how many of them lie below this slice.
    int bin = 0, need = 0, low_older = 0, low_ties = 0;
    bool exact = true;          // one stamp per bin
    unsigned tkey = 0u;         // otherwise the threshold among the bin's stamps
    Pair tot;                   // of the eligible slots, and of those below this slice
    const int b1 = AGE_BINS - 1 - 2 * tid, b0 = b1 - 1;   // this thread's bins, the older one first
    const unsigned a1 = h_all[b1], a0 = h_all[b0], l1 = h_low[b1], l0 = h_low[b0];
    const Pair older_of = settle_scan({a0 + a1, l0 + l1}, wtot, turn, tot);
    const bool take_all = (int)tot.a <= e;
    if (take_all) {
        low_older = (int)tot.b;
    } else {
        const unsigned before = older_of.a, want = (unsigned)e;
        if (before < want && want <= before + a0 + a1) {
            const bool in1 = want <= before + a1;
            sh[0] = in1 ? b1 : b0;
            sh[1] = (int)(want - before - (in1 ? 0u : a1));
            sh[2] = (int)(older_of.b + (in1 ? 0u : l1));
            sh[3] = (int)(in1 ? l1 : l0);
        }
        __syncthreads();
        bin = sh[0];
        need = sh[1];
        low_older = sh[2];
        low_ties = sh[3];
        exact = bin < AGE_EXACT && (bin > 0 || kmax <= stamp_key(frame_id));
    }
    const size_t ab = (size_t)h * n_slices * SETTLE_SLICE + SETTLE_SPT * tid;   // this thread's run in slice 0
    auto ages_of = [&](const u32x4 (&w)[2], unsigned &older, unsigned &ties) {   // of a run, by bins
        older = ties = 0u;
#pragma unroll
        for (int q = 0; q < SETTLE_SPT; ++q) {
            const int age = (int)((w[q / 8][(q % 8) / 2] >> (16 * (q & 1))) & 0xFFFFu);
            older |= (take_all || age > bin) ? 1u << q : 0u;
            ties |= (!take_all && age == bin) ? 1u << q : 0u;
        }
    };
    auto eligible = [&](int j0) -> unsigned {   // live and untouched slots of the run from j0 on
        const unsigned bits = j0 < C ? (~(touched[j0 >> 5] >> (j0 & 31))) & 0xFFFFu : 0u;
        return j0 + SETTLE_SPT <= L ? bits : j0 < L ? bits & ((1u << (L - j0)) - 1u) : 0u;
    };
    if (!exact) {   // uniform over the head: digits of ten bits of the bin's stamps, over their range
        unsigned age_lo = 0u, age_hi = 0u;
        if (bin > 0) age_bin_range(bin, age_lo, age_hi);
        const unsigned now = stamp_key(frame_id), top = bin > 0 ? now - age_lo : kmax;   // the age occurs: no wrap
        tkey = now - min(age_hi, now);
        const unsigned span = top - tkey;
        for (int shift = span ? 32 - __clz(span) : 0; shift > 0;) {   // uniform
            const int width = min(10, shift);
            shift -= width;
            __syncthreads();   // the counts before have been read
            h_all[2 * tid] = h_all[2 * tid + 1] = 0u;
            h_low[2 * tid] = h_low[2 * tid + 1] = 0u;
            __syncthreads();
            for (int q = 0; q < n_slices; ++q) {
                if (ag[(size_t)q * AGE_WORDS + bin] == 0u) continue;   // uniform
                unsigned older, ties;
                const size_t at = ab + (size_t)q * SETTLE_SLICE;
                const u32x4 w[2] = {*(const u32x4 *)(slot_age + at), *(const u32x4 *)(slot_age + at + 8)};
                ages_of(w, older, ties);
                ties &= eligible(q * SETTLE_SLICE + SETTLE_SPT * tid);
                if (!ties) continue;
                u32x4 sv[SETTLE_SPT / 4];
#pragma unroll
                for (int x = 0; x < SETTLE_SPT / 4; ++x) sv[x] = *(const u32x4 *)(slot_stamp + at + 4 * x);
                unsigned run_digit = 0u, run_n = 0u;   // a run of one digit is one addition
                auto flush = [&]() {
                    if (run_n) {
                        atomicAdd(&h_all[run_digit], run_n);
                        if (q < slice) atomicAdd(&h_low[run_digit], run_n);
                    }
                };
#pragma unroll
                for (int x = 0; x < SETTLE_SPT; ++x) {
                    const unsigned digit = (stamp_key((int)sv[x / 4][x % 4]) - tkey) >> shift;
                    if (!((ties >> x) & 1u) || (digit >> width)) continue;   // below or above what is left of the range
                    if (digit != run_digit) {
                        flush();
                        run_n = 0u;
                    }
                    run_digit = digit;
                    run_n += 1u;
                }
                flush();
            }
            __syncthreads();
            const unsigned a0 = h_all[2 * tid], a1 = h_all[2 * tid + 1], l0 = h_low[2 * tid], l1 = h_low[2 * tid + 1];
            const Pair ex = settle_scan({a0 + a1, l0 + l1}, wtot, turn, tot);
            const unsigned before = ex.a, want = (unsigned)need;
            if (before < want && want <= before + a0 + a1) {
                const bool in0 = want <= before + a0;
                sh[0] = 2 * tid + (in0 ? 0 : 1);
                sh[1] = (int)(want - before - (in0 ? 0u : a0));
                sh[2] = (int)(ex.b + (in0 ? 0u : l0));
                sh[3] = (int)(in0 ? l0 : l1);
            }
            __syncthreads();
            tkey += (unsigned)sh[0] << shift;
            need = sh[1];
            low_older += sh[2];
            low_ties = sh[3];
        }
    }
    // The slice's victims in ascending order, and the rows of every n_reps-th of them
    unsigned older, ties;
    ages_of(run, older, ties);
    if (!exact && ties) {
        const size_t at = ab + (size_t)slice * SETTLE_SLICE;
        const unsigned of_bin = ties;
        ties = 0u;
        for (unsigned todo = of_bin; todo; todo &= todo - 1u) {
            const int q = __ffs(todo) - 1;
            const unsigned key = stamp_key(slot_stamp[at + q]);
            older |= key < tkey ? 1u << q : 0u;
            ties |= key == tkey ? 1u << q : 0u;
        }
    }
    {
        const unsigned bits = eligible(s0 + SETTLE_SPT * tid);
        older &= bits;
        ties &= bits;
    }
    const Pair ex = settle_scan({(unsigned)__popc(older), (unsigned)__popc(ties)}, wtot, turn, tot);
    const int take_ties = min(max(need - low_ties, 0), (int)tot.b);
    const int n_here = (int)tot.a + take_ties, rank0 = low_older + min(need, low_ties);
    unsigned take = older;
    {
        int ties_left = take_ties - (int)ex.b;
        unsigned first = ties_left > 0 ? ties : 0u;
        for (; __popc(first) > ties_left && first; ) first &= ~(0x80000000u >> __clz(first));   // one thread of the slice
        take |= first;
    }
    // all slots of the run, without branches: the others' go to a word of no meaning (victims are mostly whole runs; the set bits one
    // after the other took 1.6 us longer)
    if (__ballot(take != 0u)) {   // uniform
        const int idx = (int)ex.a + min((int)ex.b, take_ties);
#pragma unroll
        for (int q = 0; q < SETTLE_SPT; ++q) {
            const int at = (take >> q) & 1u ? idx + __popc(take & ((1u << q) - 1u)) : SETTLE_SLICE;
            vict[at] = (unsigned short)(SETTLE_SPT * tid + q);
        }
    }
    __syncthreads();
    const int n_rows = n_here > share ? (n_here - share + n_reps - 1) / n_reps : 0;
    constexpr int UN = 2;   // rows of a group in flight
    for (int v0 = group; v0 < n_rows; v0 += SETTLE_GROUPS * UN) {
        typename RP::Raw kr[UN], vr[UN];
        unsigned cw[UN];
        int tok[UN], dst[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int v = v0 + u * SETTLE_GROUPS;
            tok[u] = -1;
            if (v < n_rows) {
                const int a = rank0 + v * n_reps + share;
                dst[u] = s0 + vict[v * n_reps + share];
                tok[u] = a < n_unm ? unm[a] : -1;
            }
            if (tok[u] >= 0) {
                kr[u] = RP::load_raw(K_new, tb + tok[u], l16);
                vr[u] = RP::load_raw(V_new, tb + tok[u], l16);
                cw[u] = l16 < r / 4 ? ((const unsigned *)(ck + (tb + tok[u]) * r))[l16] : 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u)
            if (tok[u] >= 0) {
                RP::store_raw(K, cb + dst[u], l16, kr[u]);
                RP::store_raw(V, cb + dst[u], l16, vr[u]);
                if (l16 < r / 4) ((unsigned *)(code + (cb + dst[u]) * r))[l16] = cw[u];
                if (l16 == 0) {
                    cnt[cb + dst[u]] = 1;
                    stamp[cb + dst[u]] = frame_id;
                    merge_map[tb + tok[u]] = dst[u];
                }
            }
    }
}

// ---- codes of the slots whose key was replaced by a mean (rep_mode 1), from the rows tc_apply_kernel stored -----
// One wavefront per 16 tokens, as in encode_kernel; every merged token encodes its slot (the joiners of one slot
// write the same bytes).
template <bool BF16, int D, int R>
__global__ __launch_bounds__(256) void tc_recode_kernel(const void *__restrict__ K, int8_t *__restrict__ code, int C,
                                                        int n_new, const int32_t *__restrict__ jstar,
                                                        const uint8_t *__restrict__ merged,
                                                        const int8_t *__restrict__ Rm, float qscale, int shift) {
    const int h = blockIdx.y;
    const int lane = lane_id();
    const int col = lane & 15, g = lane >> 4;
    const int i = blockIdx.x * 64 + (threadIdx.x >> 6) * 16 + col;
    const bool act = i < n_new && merged[(size_t)h * n_new + i] != 0;
    const int j = act ? jstar[(size_t)h * n_new + i] : 0;
    CodeMatrix<BF16, D, R> cm;
    cm.load(Rm, lane);
    const char *row = (const char *)K + ((size_t)h * C + j) * (size_t)D * (BF16 ? 2 : 4);
    i32x4 xq[D / 64];
    load_quantised<BF16, D>(row, g, qscale, xq);
    const auto w = cm.code_words(xq, shift);
    if (act) cm.store(code + ((size_t)h * C + j) * R, w, lane);
}

}  // namespace fastar

using namespace fastar;

// what tc_plan_kernel's waits are bounded by (test hook below; the default is what every caller gets)
static PlanWait g_plan_wait = {PLAN_SPIN_LIMIT, 0u};

extern "C" int fastar_debug_plan_wait(int spin_limit, int extra_arrivals) {
    if (extra_arrivals < 0) return FASTAR_ERR_INVALID_ARG;
    g_plan_wait.spin_limit = spin_limit < 0 ? PLAN_SPIN_LIMIT : spin_limit;
    g_plan_wait.extra_arrivals = (unsigned)extra_arrivals;
    return FASTAR_OK;
}

extern "C" int tempcache_compress(const fastar_cache *cache, const fastar_codec *codec, const void *K_new,
                                  const void *V_new, const void *P_new, int n_new, const int32_t *cand, int n_cand,
                                  int metric, int32_t tau2_q16, int32_t frame_id, int rep_mode, int32_t *merge_map,
                                  uint8_t *merged, int32_t *stats, void *ws, size_t ws_bytes, int ws_persistent,
                                  void *stream) {
    if (!cache || !codec || !codec->R || !K_new || !V_new || !merge_map || !merged || !stats || !ws)
        return FASTAR_ERR_INVALID_ARG;
    if (!cache->K || !cache->V || !cache->code || !cache->cnt || !cache->stamp || !cache->len)
        return FASTAR_ERR_INVALID_ARG;
    const int H = cache->H, C = cache->C, d = cache->d, r = cache->r, dtype = cache->dtype;
    if (H <= 0 || C <= 0 || n_new <= 0 || (metric != 0 && metric != 1)) return FASTAR_ERR_INVALID_ARG;
    if (rep_mode != FASTAR_REP_LAST && rep_mode != FASTAR_REP_MEAN && rep_mode != FASTAR_REP_MEDOID) return FASTAR_ERR_INVALID_ARG;
    if (ws_persistent != 0 && ws_persistent != 1) return FASTAR_ERR_INVALID_ARG;
    if (tau2_q16 < 0 || tau2_q16 > 131072) return FASTAR_ERR_INVALID_ARG;
    if (cand && n_cand <= 0) return FASTAR_ERR_INVALID_ARG;
    if (codec->shift < 1 || codec->shift > 16) return FASTAR_ERR_INVALID_ARG;
    if (dtype != FASTAR_F32 && dtype != FASTAR_BF16) return FASTAR_ERR_INVALID_ARG;
    if ((d != 64 && d != 128) || (r != 32 && r != 64)) return FASTAR_ERR_UNSUPPORTED;
    PlanResidency pr;
    if (const int rc0 = plan_residency(&pr); rc0 != FASTAR_OK) return rc0;
    const int nb = plan_nb(H, C, pr);
    if (plan_lds_bytes(C, nb) > 48 * 1024) return FASTAR_ERR_UNSUPPORTED;  // eviction bitmap of a slot range lives in LDS
    // Who counts the live slots' ages for the eviction threshold.  Short caches: the verify step, whose whole grid reads
    // the stamps while the plan's few workgroups would meet for it.  Long caches (a plan thread holds more than 16 stamps,
    // and all of its run, in registers): the plan itself, from the stamps it reads anyway: a second sweep over every
    // stamp costs more than one meeting of the head's workgroups.
    const int plan_span = (((C + nb - 1) / nb) + 3) & ~3;
    const int plan_per = (((plan_span + PLAN_THREADS - 1) / PLAN_THREADS) + 3) & ~3;
    const bool long_runs = ((C + nb - 1) / nb + PLAN_THREADS - 1) / PLAN_THREADS > 16;   // the plan's instantiation with 64 stamps per thread
    const bool self_hist = long_runs && plan_per <= 64;
    if (((uintptr_t)cache->K & 15) || ((uintptr_t)cache->V & 15) || ((uintptr_t)cache->code & 15) ||
        ((uintptr_t)K_new & 15) || ((uintptr_t)V_new & 15) || ((uintptr_t)P_new & 15) || ((uintptr_t)ws & 255))
        return FASTAR_ERR_INVALID_ARG;
    const CompressWs w = compress_ws(H, C, n_new, r);
    if (ws_bytes < w.total) return FASTAR_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char *base = (char *)ws;
    int8_t *ck = (int8_t *)(base + w.ck);
    int8_t *cp = P_new ? (int8_t *)(base + w.cp) : ck;
    u64 *best = (u64 *)(base + w.best);
    int32_t *jstar = (int32_t *)(base + w.jstar), *sbest = (int32_t *)(base + w.sbest);
    int32_t *rank = (int32_t *)(base + w.rank), *victims = (int32_t *)(base + w.victims);
    int32_t *hs = (int32_t *)(base + w.hs);
    unsigned *plan_scratch = (unsigned *)(base + w.ps);
    u64 *win = (u64 *)(base + w.win);
    int32_t *grp = (int32_t *)(base + w.grp);
    const int64_t T = (int64_t)H * n_new;

    const size_t win_lds = cand ? match_window_lds(n_cand, r) : 0;
    const bool window = cand && win_lds <= WINDOW_LDS_MAX;
    const bool fused_encode = window && !P_new;  // the match kernel encodes its own probes
    const bool fused_verify = fused_encode && ws_persistent;   // ... and verifies its matches: nothing to clear first
    // Plan and apply in one launch: short caches, whose age histograms are small enough to be read by every workgroup, and
    // calls of a rollout (the others pay for a clearing launch as it is, and keep the plan and its waits).
    const bool fits = C <= SETTLE_SLOTS && n_new <= SETTLE_TOKENS;
    const bool cleared = !window && (int64_t)H * C <= CLEAR_SLOTS_MAX;
    const SettleGrid sg = fits ? settle_grid(H, C, n_new) : SettleGrid{};
    const bool settle = ws_persistent && fits && sg.better;
    const SettleOut so = settle ? SettleOut{hs, (int32_t *)(base + w.tstamp), (unsigned *)(base + w.ages), (unsigned short *)(base + w.slot_age),
                                          (int32_t *)(base + w.slot_stamp)} : SettleOut{};
    if (!fused_encode) {
        const int64_t zero_words = (int64_t)(w.best - w.ps) / 8 + T;   // ps and best
        int rc = encode_launch(K_new, dtype, T, d, codec, r, ck, (u64 *)plan_scratch, zero_words, s,
                               cleared ? ClearRecords{win, grp, cache->len, H, C} : ClearRecords{});
        if (rc != FASTAR_OK) return rc;
        if (P_new) {
            rc = encode_launch(P_new, dtype, T, d, codec, r, cp, nullptr, 0, s);
            if (rc != FASTAR_OK) return rc;
        }
    }
    if (window) {
        // the whole candidate window fits one workgroup's LDS: final arg-max per token in one launch
        if (const int rc0 = tempcache_setup(); rc0 != FASTAR_OK) return rc0;
        // 256 tokens per workgroup when 64 would give more than two rounds of workgroups over the chip (the window is
        // staged once per workgroup) and the window leaves room for the wider static arrays
        const size_t per_cu = (size_t)160 * 1024 / (win_lds + 9 * 1024);
        const bool wide = fused_encode && win_lds <= wide_window_lds_max(r) &&
                          (size_t)((n_new + 63) / 64) * (size_t)H > 2 * 256 * (per_cu > 0 ? per_cu : 1);
        // With 256 tokens per workgroup a workgroup takes several blocks of tokens, one after the other, once it has
        // staged the window: as many workgroups as the chip holds at once (the staging is then paid once per resident
        // workgroup, and no round of workgroups waits for the one before it).
        int gx = wide ? (n_new + 255) / 256 : (n_new + 63) / 64;
        if (wide) {   // equal shares of whole groups of 32 tokens, none of them empty
            gx = std::min(gx, std::max(1, (int)(256 * (per_cu > 0 ? per_cu : 1)) / H));
            const int per = (((n_new + gx - 1) / gx) + 31) & ~31;
            gx = (n_new + per - 1) / per;
        }
        // the age histogram beside the match: a workgroup per 8192 slots (one round of loads, 4 x 16 bytes per thread)
        const int n_hist = !fused_verify || wide ? 0 : settle ? settle_slices(C) : !self_hist ? (C + 8191) / 8192 : 0;
        const int hist_rows = settle && fused_verify && wide ? (settle_slices(C) * H + gx - 1) / gx : 0;   // behind the heads' rows
        const dim3 grid(gx + n_hist, H + hist_rows);
        const bool bf = dtype == FASTAR_BF16;
        const VerifyArgs va = {cache->K, tau2_q16, merged, cache->stamp, frame_id, self_hist ? -1 : PS_HIST, PS_FUT, H, so};
        int rc = FASTAR_OK;
#define FASTAR_WIN(RR, ENC, BF, DD, VER, TT)                                                                              \
    rc = launch_match_window<RR, ENC, BF, DD, VER, TT>(grid, win_lds, s, cache->code, cache->len, C, cp, n_new, cand,      \
                                                       n_cand, metric, jstar, sbest, win, grp, K_new, codec->R,            \
                                                       codec->qscale, codec->shift, ck, plan_scratch, (int)PS_STRIDE, n_hist, va)
#define FASTAR_WIN_ENC(RR, BF, DD)                                                      \
    do {                                                                                \
        if (fused_verify && wide) FASTAR_WIN(RR, true, BF, DD, true, 256);              \
        else if (fused_verify) FASTAR_WIN(RR, true, BF, DD, true, 64);                  \
        else if (wide) FASTAR_WIN(RR, true, BF, DD, false, 256);                        \
        else FASTAR_WIN(RR, true, BF, DD, false, 64);                                   \
    } while (0)
        if (!fused_encode) { if (r == 32) FASTAR_WIN(32, false, true, 128, false, 64); else FASTAR_WIN(64, false, true, 128, false, 64); }
        else if (r == 32 && d == 128) { if (bf) FASTAR_WIN_ENC(32, true, 128); else FASTAR_WIN_ENC(32, false, 128); }
        else if (r == 32) { if (bf) FASTAR_WIN_ENC(32, true, 64); else FASTAR_WIN_ENC(32, false, 64); }
        else if (d == 128) { if (bf) FASTAR_WIN_ENC(64, true, 128); else FASTAR_WIN_ENC(64, false, 128); }
        else { if (bf) FASTAR_WIN_ENC(64, true, 64); else FASTAR_WIN_ENC(64, false, 64); }
#undef FASTAR_WIN_ENC
#undef FASTAR_WIN
        if (rc != FASTAR_OK) return rc;
    } else {
        if (const int rc0 = tempcache_setup(); rc0 != FASTAR_OK) return rc0;
        if (!cand) {
            // frames of at most 128 tokens leave half of the wavefronts of a 256-token block without work
            int rc;
#define FASTAR_MATCH_ALL(RR, TT) rc = launch_match_all<RR, TT>(cache->code, cache->len, C, cp, n_new, H, metric, best, s)
            if (n_new <= 128) { if (r == 32) FASTAR_MATCH_ALL(32, 64); else FASTAR_MATCH_ALL(64, 64); }
            else { if (r == 32) FASTAR_MATCH_ALL(32, 256); else FASTAR_MATCH_ALL(64, 256); }
#undef FASTAR_MATCH_ALL
            if (rc != FASTAR_OK) return rc;
        } else {
            const int chunk = n_cand <= 4096 ? 64 : 256;
            dim3 grid((n_new + 127) / 128, (n_cand + chunk - 1) / chunk, H);
#define FASTAR_MATCH(RR, CH)                                                                                              \
    hipLaunchKernelGGL((tc_match_kernel<RR, CH>), grid, dim3(256), 0, s, cache->code, cache->len, C, cp, n_new, cand, n_cand, \
                       metric, best)
            if (r == 32 && chunk == 64) FASTAR_MATCH(32, 64);
            else if (r == 32) FASTAR_MATCH(32, 256);
            else if (chunk == 64) FASTAR_MATCH(64, 64);
            else FASTAR_MATCH(64, 256);
#undef FASTAR_MATCH
        }
        FASTAR_LAUNCH_CHECK();
        if (!cleared) {
            hipLaunchKernelGGL(tc_prep_kernel, dim3((n_new + 255) / 256, H), dim3(256), 0, s, best, n_new, C, cand, n_cand,
                               jstar, sbest, win, grp);
            FASTAR_LAUNCH_CHECK();
        }
    }
    const dim3 tgrid((n_new + 15) / 16, H);
    const bool bf = dtype == FASTAR_BF16;
#define FASTAR_TC(KERNEL, GRID, THREADS, ...)                                                                          \
    do {                                                                                                               \
        if (bf && d == 128) hipLaunchKernelGGL((KERNEL(true, 128)), GRID, dim3(THREADS), 0, s, __VA_ARGS__);           \
        else if (bf) hipLaunchKernelGGL((KERNEL(true, 64)), GRID, dim3(THREADS), 0, s, __VA_ARGS__);                   \
        else if (d == 128) hipLaunchKernelGGL((KERNEL(false, 128)), GRID, dim3(THREADS), 0, s, __VA_ARGS__);           \
        else hipLaunchKernelGGL((KERNEL(false, 64)), GRID, dim3(THREADS), 0, s, __VA_ARGS__);                          \
    } while (0)
#define FASTAR_VERIFY(BF, DD) tc_verify_kernel<BF, DD, false>
#define FASTAR_VERIFY_SETTLE(BF, DD) tc_verify_kernel<BF, DD, true>
#define FASTAR_APPLY(BF, DD) tc_apply_kernel<BF, DD>
    if (!fused_verify) {
        // twice the threads where the launch also counts the ages: a slice is then one round of loads (11.6 -> 9 us at 12 heads x
        // 1560 tokens x 32760 slots)
        const int threads = settle ? SETTLE_THREADS : 256, n_slices = settle ? settle_slices(C) : 0;
        const dim3 vgrid((n_new + threads / 16 - 1) / (threads / 16) + n_slices, H);
#define FASTAR_VERIFY_ARGS                                                                                              \
    cache->K, K_new, cp, r, C, n_new, codec->qscale, metric, tau2_q16, jstar, sbest, cleared ? best : nullptr, win, grp,  \
        merged, cache->len, cache->stamp, frame_id, plan_scratch, self_hist ? -1 : PS_HIST, PS_FUT, PS_STRIDE, n_slices, so
        if (settle) FASTAR_TC(FASTAR_VERIFY_SETTLE, vgrid, threads, FASTAR_VERIFY_ARGS);
        else FASTAR_TC(FASTAR_VERIFY, vgrid, threads, FASTAR_VERIFY_ARGS);
#undef FASTAR_VERIFY_ARGS
        FASTAR_LAUNCH_CHECK();
    }
    if (settle) {
        const dim3 sgrid(sg.wgs, H);
        const size_t lds = settle_lds_bytes(C, n_new);
#define FASTAR_SETTLE_T(BF, DD, TT)                                                                                      \
    hipLaunchKernelGGL((tc_settle_kernel<BF, DD, TT>), sgrid, dim3(SETTLE_THREADS), lds, s, cache->K, cache->V, cache->code,    \
                       cache->cnt, cache->stamp, C, r, K_new, V_new, ck, n_new, frame_id, jstar, merged, win, grp, hs,     \
                       merge_map, cache->len, rep_mode, so.tstamp, so.ages, so.slot_age, so.slot_stamp, sg.n_reps, stats)
#define FASTAR_SETTLE(BF, DD)                                  \
    do {                                                       \
        if (n_new <= 4 * SETTLE_THREADS) FASTAR_SETTLE_T(BF, DD, 4); \
        else FASTAR_SETTLE_T(BF, DD, 16);                      \
    } while (0)
        if (bf && d == 128) FASTAR_SETTLE(true, 128);
        else if (bf) FASTAR_SETTLE(true, 64);
        else if (d == 128) FASTAR_SETTLE(false, 128);
        else FASTAR_SETTLE(false, 64);
#undef FASTAR_SETTLE
#undef FASTAR_SETTLE_T
        FASTAR_LAUNCH_CHECK();
    } else {
        const bool long_frame = n_new > 8 * PLAN_THREADS;
#define FASTAR_PLAN(PM, TM)                                                                                            \
    hipLaunchKernelGGL((tc_plan_kernel<PM, TM>), dim3(nb + 1, H), dim3(PLAN_THREADS), plan_lds_bytes(C, nb), s, cache->len, \
                       cache->stamp, C, n_new, frame_id, jstar, merged, win, rank, victims, hs, stats, plan_scratch,   \
                       ws_persistent, self_hist ? 1 : 0, g_plan_wait)
        if (long_runs && long_frame) FASTAR_PLAN(64, 16);
        else if (long_runs) FASTAR_PLAN(64, 8);
        else if (long_frame) FASTAR_PLAN(16, 16);
        else FASTAR_PLAN(16, 8);
#undef FASTAR_PLAN
        FASTAR_LAUNCH_CHECK();
        FASTAR_TC(FASTAR_APPLY, tgrid, 256, cache->K, cache->V, cache->code, cache->cnt, cache->stamp, C, r, K_new, V_new, ck, n_new,
                  frame_id, jstar, merged, win, grp, rank, victims, hs, merge_map, cache->len, rep_mode, plan_scratch,
                  (int)PS_STRIDE, stats);
        FASTAR_LAUNCH_CHECK();
    }
#undef FASTAR_TC
#undef FASTAR_VERIFY
#undef FASTAR_VERIFY_SETTLE
#undef FASTAR_APPLY
    if (rep_mode == FASTAR_REP_MEAN) {
        const dim3 rgrid((n_new + 63) / 64, H);
#define FASTAR_RECODE(BF, DD, RR)                                                                                     \
    hipLaunchKernelGGL((tc_recode_kernel<BF, DD, RR>), rgrid, dim3(256), 0, s, cache->K, cache->code, C, n_new, jstar, \
                       merged, codec->R, codec->qscale, codec->shift)
        if (bf && d == 128) { if (r == 32) FASTAR_RECODE(true, 128, 32); else FASTAR_RECODE(true, 128, 64); }
        else if (bf) { if (r == 32) FASTAR_RECODE(true, 64, 32); else FASTAR_RECODE(true, 64, 64); }
        else if (d == 128) { if (r == 32) FASTAR_RECODE(false, 128, 32); else FASTAR_RECODE(false, 128, 64); }
        else { if (r == 32) FASTAR_RECODE(false, 64, 32); else FASTAR_RECODE(false, 64, 64); }
#undef FASTAR_RECODE
        FASTAR_LAUNCH_CHECK();
    }
    return FASTAR_OK;
}
