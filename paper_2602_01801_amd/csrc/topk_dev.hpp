// Exact top-k of a row of integer scores by one workgroup: shared by the selection kernels.
#pragma once

#include <limits.h>

#include <type_traits>

#include "common.hpp"

namespace fastar {

constexpr int TOPK_LDS_CAP = 8192; // row entries cached in LDS by the callers of topk_row
constexpr int TOPK_WAVE_MAX = 1024;   // entries of a row that one wavefront selects from, from registers
constexpr int TOPK_REG_MAX = 4096;    // ... and that four select from
constexpr int TOPK_QUARTER_SEL = 128; // at most so many of them: a quarter of the row per wavefront
constexpr int TOPK_DIGIT = 9;         // otherwise: bits per pass over the keys
constexpr int TOPK_BINS = 1 << TOPK_DIGIT;
constexpr int TOPK_WAVE_BINS = 256;
constexpr int TOPK_SCRATCH = 4 * (TOPK_WAVE_BINS + 2 * TOPK_QUARTER_SEL) + 4;   // words: a histogram and a list for each wavefront, the lists' lengths

// Exact top-k by ONE wavefront: entry 64 e + lane of the row in register e (key + 1, 0: no entry), so positions come out in order
// and no barrier is needed.  One histogram of 256 bins over the row's own range leaves, as a rule, a handful of entries in the
// threshold's bin; the bits below are tried one by one, with a comparison and a scalar bit count per register, until exactly k
// entries lie above.  What bounds it is the issue of one wavefront (about seven cycles an instruction alone on its SIMD), where
// four wavefronts (the form further down) are a chain of barriers: 16 of 64 entries 2.0 -> 1.1 us, 64 of 512 2.9 -> 1.5; top-k launch
// for 444 rows of 585 7.2 -> 5.8.  All bits one by one, ten of them on the average: 64 of 512 2.3 us, of 1024 3.9 (now 2.2).
template <int NR>
__device__ __forceinline__ int topk_count(const unsigned (&my)[NR], unsigned limit) {   // entries >= limit > 0; uniform
    int c = 0;
#pragma unroll
    for (int e = 0; e < NR; ++e) c += __popcll(__ballot(my[e] >= limit));
    return c;
}
// Passes the k largest entries (0 < k <= number of entries; ties: the first ones) to out(position, entry, key + 1), entries
// ascending.  `forced` of the entries rank above all others; lo, hi: range of those (where there are any).  hist:
// TOPK_WAVE_BINS words of LDS, 16-byte aligned, this wavefront's own.
template <int NR, typename Out>
__device__ __forceinline__ void topk_wave(const unsigned (&my)[NR], int k, int forced, unsigned lo, unsigned hi, unsigned *hist,
                                          Out &&out) {
    const int lane = lane_id();
    unsigned T = (1u << 22) + 1u, need = (unsigned)k;   // threshold key + 1, and how many of the entries equal to it are taken
    if (forced < k) {      // uniform
        ((u32x4 *)hist)[lane] = u32x4{0u, 0u, 0u, 0u};
        const unsigned span = hi - lo, want = (unsigned)(k - forced);
        int shift = span ? max(24 - __clz(span), 0) : 0;   // the bins are the eight leading bits of the span
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int e = 0; e < NR; ++e)
            if (my[e] - lo <= span) atomicAdd(&hist[(my[e] - lo) >> shift], 1u);   // neither missing nor forced
        __builtin_amdgcn_wave_barrier();
        // lane l owns the bins 255 - 4 l .. 252 - 4 l: where does the running count from the top reach `want`?
        const u32x4 c4 = ((const u32x4 *)hist)[63 - lane];
        const unsigned sum = (c4[0] + c4[1]) + (c4[2] + c4[3]), incl = wave_incl_scan(sum);
        unsigned before = incl - sum, bin = 0u, left = 0u, count = 0u;
        const bool mine = before < want && want <= incl;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned c = c4[3 - q];
            const bool here = (before < want) & (want <= before + c);
            bin = here ? (unsigned)(255 - 4 * lane - q) : bin;
            left = here ? want - before : left;
            count = here ? c : count;
            before += c;
        }
        const int src = __ffsll((unsigned long long)__ballot(mine)) - 1;   // exactly one lane
        bin = (unsigned)__builtin_amdgcn_readlane((int)bin, src);
        left = (unsigned)__builtin_amdgcn_readlane((int)left, src);
        count = (unsigned)__builtin_amdgcn_readlane((int)count, src);
        T = lo + (bin << shift);
        int above = k - (int)left;          // entries above what T may still become
        bool whole = left == count;
        for (unsigned step = (1u << shift) >> 1; step != 0u && !whole; step >>= 1) {   // uniform
            const int c = topk_count(my, T + step);
            if (c >= k) T += step;
            else above = c;
            whole = c == k;
        }
        need = (unsigned)(k - above);
        if (whole) {   // everything from T on
            T -= 1u;
            need = 0u;
        }
    }
    unsigned at = 0u, eq = 0u;   // entries taken, entries equal to T, of the registers before (uniform)
    auto rank = [&](unsigned long long m, unsigned base) {   // of this lane among those of m, from base on
        return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, base));
    };
    if (need == 0u) {   // uniform
#pragma unroll
        for (int e = 0; e < NR; ++e) {
            const unsigned long long m = __ballot(my[e] > T);
            if (my[e] > T) out((int)rank(m, at), 64 * e + lane, my[e]);
            at += (unsigned)__popcll(m);
        }
    } else {
#pragma unroll
        for (int e = 0; e < NR; ++e) {
            const bool is_eq = my[e] == T;   // T > 0
            const unsigned long long m_eq = __ballot(is_eq);
            const bool take = (my[e] > T) | (is_eq & (rank(m_eq, eq) < need));   // without branches
            const unsigned long long m = __ballot(take);
            if (take) out((int)rank(m, at), 64 * e + lane, my[e]);
            at += (unsigned)__popcll(m);
            eq += (unsigned)__popcll(m_eq);
        }
    }
}
// Selects from row[0 .. n), n <= 64 NR, of keys key_of(entry, score), and returns how many it passed to out(position, entry,
// key + 1): at most n_sel, and no more than there are candidates.
template <int NR, typename KeyOf, typename Out>
__device__ __forceinline__ int topk_wave_of(const int32_t *row, int n, int n_sel, int forced, unsigned cand_key, KeyOf &&key_of,
                                            unsigned *hist, Out &&out) {
    if (n <= 0) return 0;   // uniform
    const int lane = lane_id();
    unsigned my[NR];
#pragma unroll
    for (int e = 0; e < NR; ++e) my[e] = (unsigned)row[min(64 * e + lane, n - 1)];
    __builtin_amdgcn_sched_barrier(0);   // all in flight at once (not each where its key turns out to be needed)
#pragma unroll
    for (int e = 0; e < NR; ++e) asm volatile("" : "+v"(my[e]));
    unsigned hi = 0u, nlo = 0u;   // largest, and complement of the smallest, of the entries that are not forced (the last one counts again)
#pragma unroll
    for (int e = 0; e < NR; ++e) {
        const int t = min(64 * e + lane, n - 1);
        my[e] = key_of(t, (int32_t)my[e]) + 1u;
        const bool in = forced == 0 || my[e] != (1u << 22) + 1u;
        hi = max(hi, in ? my[e] : 0u);
        nlo = max(nlo, in ? ~my[e] : 0u);
        my[e] = 64 * e + lane < n ? my[e] : 0u;
    }
    hi = (unsigned)__builtin_amdgcn_readlane((int)wave_max_last(hi), 63);
    nlo = (unsigned)__builtin_amdgcn_readlane((int)wave_max_last(nlo), 63);
    const int k = min(n_sel, cand_key == 0u ? n : topk_count(my, cand_key + 1u));
    if (k > 0) topk_wave(my, k, forced, ~nlo, hi, hist, out);
    return k;
}

// Rows of more than TOPK_WAVE_MAX and up to TOPK_REG_MAX entries from which more than TOPK_QUARTER_SEL are wanted, by four
// wavefronts.  Every thread holds a run of KPT consecutive entries in registers (key + 1, 0: no entry).
// What bounds it is the chain of barriers, and of same-address additions where the keys' leading bits are alike.  So the
// row's range comes first (one barrier), the digits are those of its span, every wavefront reads the threshold digit off the
// histogram itself (one barrier per pass), and once the threshold's bin holds at most 64 entries, as a rule after the
// first pass, every wavefront ranks those (one barrier); one more for the positions.  Selection of 64 out of 2048 scores
// 9.5 -> 5.9 us (before: three fixed digits with three barriers each and a compaction with three per 256 entries).  Digits of ten
// bits: no faster, and their 16 bins per lane cost registers.  One wavefront on 64 registers of keys instead: select of 400 out of
// 4000 prompt tokens for 12 x 37 query blocks 22.8 -> 26.8 us, of 360 out of 3600 key blocks for 40 x 29 24.4 -> 22.7.
template <int KPT, typename KeyOf>
__device__ __forceinline__ void topk_from_registers(const int32_t *row, int n, int n_sel, int32_t *__restrict__ out,
                                                    int32_t *__restrict__ nsel_out, unsigned *keys, int forced,
                                                    unsigned cand_key, KeyOf &&key_of, unsigned *scratch) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    unsigned *hist = scratch, *wsum = scratch + 2 * TOPK_BINS;   // wsum: [4] max, [4] ~min, [4] candidates, [4] counts, list length
    constexpr unsigned FORCED = (1u << 22) + 1u;                 // key + 1 of a forced entry
    int kpt = (n + 255) / 256;
    if (kpt < KPT) kpt |= 1;   // an odd stride: the threads' runs start on different banks
    unsigned my[KPT];
    if (keys != nullptr) {   // row in global memory: coalesced loads, all in flight at once, staged through LDS
        int32_t v[KPT];
#pragma unroll
        for (int e = 0; e < KPT; ++e) {
            const int t = e * 256 + tid;
            v[e] = t < n ? row[t] : 0;
        }
        for (int t = tid; t < 2 * TOPK_BINS; t += 256) hist[t] = 0u;
#pragma unroll
        for (int e = 0; e < KPT; ++e) {
            const int t = e * 256 + tid;
            if (t < n) keys[t] = key_of(t, v[e]);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < KPT; ++e) {
            const int i = tid * kpt + e;
            my[e] = (e < kpt && i < n) ? keys[i] + 1u : 0u;
        }
    } else {
        for (int t = tid; t < 2 * TOPK_BINS; t += 256) hist[t] = 0u;
#pragma unroll
        for (int e = 0; e < KPT; ++e) {
            const int i = tid * kpt + e;
            my[e] = (e < kpt && i < n) ? key_of(i, row[i]) + 1u : 0u;
        }
    }
    unsigned hi = 0u, nlo = 0u, n_cand = 0u;   // largest key + 1 and the complement of the smallest, forced entries aside; candidates
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
        if (e >= kpt) break;
        const bool in = my[e] != 0u && my[e] != FORCED;
        hi = max(hi, in ? my[e] : 0u);
        nlo = max(nlo, in ? ~my[e] : 0u);
        n_cand += (unsigned)__popcll(__ballot(my[e] > cand_key));
    }
    hi = wave_max_last(hi);
    nlo = wave_max_last(nlo);
    if (lane == 63) {
        wsum[wave] = hi;
        wsum[4 + wave] = nlo;
        wsum[8 + wave] = n_cand;
    }
    if (tid == 0) wsum[16] = 0u;
    __syncthreads();   // also: the histograms are clear
    const int k = min(n_sel, (int)(wsum[8] + wsum[9] + wsum[10] + wsum[11]));
    if (tid == 0) *nsel_out = k;
    for (int t = k + tid; t < n_sel; t += 256) out[t] = -1;
    if (k == 0) return;   // uniform
    unsigned T, need;   // threshold key + 1 and how many of the entries equal to it belong to the selection
    if (forced >= k) {  // uniform
        T = FORCED;
        need = (unsigned)k;
    } else {
        hi = max(max(wsum[0], wsum[1]), max(wsum[2], wsum[3]));
        const unsigned lo = ~max(max(wsum[4], wsum[5]), max(wsum[6], wsum[7]));
        need = (unsigned)(k - forced);
        int shift = hi == lo ? 0 : 32 - __clz(hi - lo);   // bits of the span still undecided
        unsigned prefix = 0;
        bool whole = false;
        for (int pass = 0; shift > 0 && !whole; ++pass) {   // uniform: at most three passes
            const int width = min(TOPK_DIGIT, shift);
            unsigned *h = hist + (pass & 1) * TOPK_BINS;
            if (pass == 2) {   // every wavefront is past the pass before, and so past the first one's counts
                for (int t = tid; t < TOPK_BINS; t += 256) h[t] = 0u;
                __syncthreads();
            }
#pragma unroll
            for (int e = 0; e < KPT; ++e) {
                if (e >= kpt) break;   // uniform, here and below
                const unsigned rel = my[e] - lo;
                if (my[e] != 0u && my[e] != FORCED && (rel >> shift) == prefix)
                    atomicAdd(&h[(rel >> (shift - width)) & ((1u << width) - 1u)], 1u);
            }
            __syncthreads();
            // lane l owns the bins 511 - 8 l .. 504 - 8 l: where does the running count from the top reach `need`?
            constexpr int BPL = TOPK_BINS / 64;
            unsigned c[BPL], sum = 0;   // descending
#pragma unroll
            for (int q = 0; q < BPL / 4; ++q) {
                const u32x4 w = ((const u32x4 *)h)[(BPL / 4) * (63 - lane) + BPL / 4 - 1 - q];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    c[4 * q + e] = w[3 - e];
                    sum += w[3 - e];
                }
            }
            const unsigned incl = wave_incl_scan(sum);
            unsigned before = incl - sum, bin = 0, left = 0, count = 0;
            const bool mine = before < need && need <= incl;
#pragma unroll
            for (int q = 0; q < BPL; ++q) {
                const bool here = mine && before < need && need <= before + c[q];
                bin = here ? (unsigned)(TOPK_BINS - 1 - BPL * lane - q) : bin;
                left = here ? need - before : left;
                count = here ? c[q] : count;
                before += c[q];
            }
            const int src = __ffsll((unsigned long long)__ballot(mine)) - 1;   // exactly one lane
            bin = (unsigned)__builtin_amdgcn_readlane((int)bin, src);
            need = (unsigned)__builtin_amdgcn_readlane((int)left, src);
            count = (unsigned)__builtin_amdgcn_readlane((int)count, src);
            whole = need == count;   // all of the bin: no finer threshold needed
            shift -= width;
            prefix = (prefix << width) | bin;
            if (!whole && shift > 0 && count <= 64u) {   // uniform: rank the bin's entries
                unsigned *list = hist + ((pass & 1) ^ 1) * TOPK_BINS;   // not in use, or no longer
#pragma unroll
                for (int e = 0; e < KPT; ++e) {
                    if (e >= kpt) break;
                    if (my[e] != 0u && my[e] != FORCED && ((my[e] - lo) >> shift) == prefix) list[atomicAdd(&wsum[16], 1u)] = my[e];
                }
                if (tid < 3) list[count + tid] = 0u;   // the last four are read together
                __syncthreads();
                const unsigned mine = lane < (int)count ? list[lane] : 0u;
                unsigned gt = 0;   // entries above this lane's
                for (unsigned j = 0; j < count; j += 4) {
                    const u32x4 other = *(const u32x4 *)(list + j);
#pragma unroll
                    for (int q = 0; q < 4; ++q) gt += other[q] > mine ? 1u : 0u;
                }
                // the smallest entry with fewer than `need` above it is the threshold
                const unsigned most = (unsigned)__builtin_amdgcn_readlane((int)wave_max_last(gt < need ? gt + 1u : 0u), 63) - 1u;
                const int at = __ffsll((unsigned long long)__ballot(gt == most && mine != 0u)) - 1;
                need -= most;
                prefix = (unsigned)__builtin_amdgcn_readlane((int)mine, at) - lo;
                shift = 0;
            }
        }
        T = lo + (prefix << shift);
        if (whole) {   // everything from the bin's lower edge on
            T -= 1u;
            need = 0u;
        }
    }
    unsigned n_gt = 0, n_eq = 0;
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
        if (e >= kpt) break;
        n_gt += my[e] > T ? 1u : 0u;
        n_eq += my[e] == T ? 1u : 0u;
    }
    const unsigned packed = (n_gt << 16) | n_eq;   // both totals stay below 4097
    const unsigned incl = wave_incl_scan(packed);
    if (lane == 63) wsum[12 + wave] = incl;
    __syncthreads();
    unsigned excl = incl - packed;
#pragma unroll
    for (int w = 0; w < 4; ++w)
        if (w < wave) excl += wsum[12 + w];
    unsigned eq_rank = excl & 0xFFFFu;
    unsigned pos = (excl >> 16) + min(eq_rank, need);
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
        if (e >= kpt) break;
        const bool take = my[e] > T || (my[e] != 0u && my[e] == T && eq_rank < need);
        if (my[e] == T) eq_rank += 1;
        if (take) out[pos++] = tid * kpt + e;
    }
}

// Entries of a row that are candidates: score >= cand_min, or forced (first n_sink / last n_local).  All 256 threads.
__device__ __forceinline__ int count_candidates(const int32_t *row, int n, int n_sink, int n_local, int cand_min) {
    __shared__ int cand_w[4];
    int c = 0;
    for (int base = 0; base < n; base += 256) {   // uniform trip count
        const int t = base + threadIdx.x;
        const bool is_cand = t < n && (row[t] >= cand_min || t < n_sink || t >= n - n_local);
        c += __popcll(__ballot(is_cand));
    }
    if (lane_id() == 0) cand_w[threadIdx.x >> 6] = c;
    __syncthreads();
    return cand_w[0] + cand_w[1] + cand_w[2] + cand_w[3];
}

// Scores are sums of at most 64 products of 8-bit codes (or counts of equal hash bits): |score| < 2^21, and anything below
// (the INT_MIN of a block without a live key) is clamped there, so an order-preserving key has 22 bits.
__device__ __forceinline__ unsigned topk_key(int32_t sc) { return (unsigned)(max(sc, -(1 << 21)) + (1 << 21)); }

// topk_row (below) of a row of up to MAX_N entries, by one wavefront.
template <int MAX_N>
__device__ __forceinline__ void topk_row_wave(const int32_t *row, int n, int n_sel, int32_t *__restrict__ out,
                                              int32_t *__restrict__ nsel_out, unsigned *hist, int n_sink = 0, int n_local = 0,
                                              int cand_min = INT_MIN) {
    const int first = min(n, max(n_sink, 0)), forced = first + min(max(n_local, 0), n - first);
    const unsigned cand_key = cand_min > INT_MIN ? topk_key(cand_min) : 0u;
    const auto key_of = [&](int t, int32_t sc) -> unsigned {
        return (t < n_sink || t >= n - n_local) ? (1u << 22) : topk_key(sc);
    };
    const auto put = [&](int pos, int t, unsigned) { out[pos] = t; };
    int k = 0;
    const auto select = [&](auto nr) {   // uniform
        constexpr int NR = decltype(nr)::value;
        if constexpr (64 * NR <= MAX_N) k = topk_wave_of<NR>(row, n, n_sel, forced, cand_key, key_of, hist, put);
    };
    if (n <= 256) select(std::integral_constant<int, 4>{});
    else if (n <= 512) select(std::integral_constant<int, 8>{});
    else if (n <= 768) select(std::integral_constant<int, 12>{});
    else select(std::integral_constant<int, 16>{});
    if (lane_id() == 0) *nsel_out = k;
    for (int t = k + lane_id(); t < n_sel; t += 64) out[t] = -1;
}

// ---- exact top-k per row ----------------------------------------------------------------------------
// A row of n scores (row may point to global memory or to LDS).  The k = min(n_sel, n) largest are selected
// (ties: lowest index) and their indices written ascending to out[0..k), the rest of out[0..n_sel) padded with
// -1; *nsel_out = k.  Called by all 256 threads of a workgroup.
// keys: LDS staging for up to TOPK_LDS_CAP entries of a row in global memory, or nullptr (row read in place).
// cand_min > INT_MIN: only entries that score at least that much (or are forced) may be selected, and k is at most their
// number.
// n_sink / n_local: the first / last entries of the row are forced (sink and local key blocks of AnnSA): they rank
// ahead of every real score, so they are always among the selected ones while n_sink + n_local <= n_sel.
// scratch: TOPK_SCRATCH words of LDS, 16-byte aligned (the caller's own use of them must be over on entry, behind a barrier).
__device__ __forceinline__ void topk_row(const int32_t *row, int n, int n_sel, int32_t *__restrict__ out,
                                         int32_t *__restrict__ nsel_out, unsigned *keys, unsigned *scratch, int n_sink = 0,
                                         int n_local = 0, int cand_min = INT_MIN) {
    // key of entry t with score sc: real scores stay below 2^22, forced entries sit exactly there
    auto key_of = [&](int t, int32_t sc) -> unsigned {
        return (t < n_sink || t >= n - n_local) ? (1u << 22) : topk_key(sc);
    };
    if (n <= TOPK_WAVE_MAX) {   // uniform; the other wavefronts are done
        if (threadIdx.x < 64) topk_row_wave<TOPK_WAVE_MAX>(row, n, n_sel, out, nsel_out, scratch, n_sink, n_local, cand_min);
        return;
    }
    if (n <= TOPK_REG_MAX) {
        // Forced entries rank ahead of all others: the k - forced largest of the others are to be found.
        const int first = min(n, max(n_sink, 0)), forced = first + min(max(n_local, 0), n - first);
        const unsigned cand_key = cand_min > INT_MIN ? topk_key(cand_min) : 0u;   // candidates: key + 1 > cand_key
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        if (n_sel > TOPK_QUARTER_SEL) {   // uniform
            topk_from_registers<TOPK_REG_MAX / 256>(row, n, n_sel, out, nsel_out, keys, forced, cand_key, key_of, scratch);
            return;
        }
        // every wavefront selects from its quarter, then one of them from the four lists; a wavefront's own words: histogram,
        // keys and positions of its list
        constexpr int OWN = TOPK_WAVE_BINS + 2 * TOPK_QUARTER_SEL, KEYS = TOPK_WAVE_BINS, POS = KEYS + TOPK_QUARTER_SEL;
        static_assert(4 * OWN + 4 <= TOPK_SCRATCH, "the lists fit");
        unsigned *own = scratch + wave * OWN, *lcnt = scratch + 4 * OWN;
        const int per = (((n + 3) >> 2) + 63) & ~63, t0 = wave * per, m = min(max(n - t0, 0), per);
        const int forced_here = max(min(first, t0 + m) - t0, 0) + max(t0 + m - max(n - (forced - first), t0), 0);
        const auto key_here = [&](int t, int32_t sc) { return key_of(t0 + t, sc); };
        const auto put = [&](int pos, int t, unsigned key) {
            own[KEYS + pos] = key;
            own[POS + pos] = (unsigned)(t0 + t);
        };
        const int c = per <= 512   ? topk_wave_of<8>(row + t0, m, n_sel, forced_here, cand_key, key_here, own, put)
                      : per <= 768 ? topk_wave_of<12>(row + t0, m, n_sel, forced_here, cand_key, key_here, own, put)
                                   : topk_wave_of<16>(row + t0, m, n_sel, forced_here, cand_key, key_here, own, put);
        if (lane == 0) lcnt[wave] = (unsigned)c;
        __syncthreads();
        if (wave > 0) return;
        const int n_list[4] = {(int)lcnt[0], (int)lcnt[1], (int)lcnt[2], (int)lcnt[3]};
        const int k = min(n_sel, n_list[0] + n_list[1] + n_list[2] + n_list[3]);
        const auto merge = [&](auto per_list) {   // registers per list
            constexpr int PL = decltype(per_list)::value;
            unsigned my[4 * PL], hi = 0u, nlo = 0u;
#pragma unroll
            for (int e = 0; e < 4 * PL; ++e) {
                const int pos = 64 * (e % PL) + lane;
                my[e] = scratch[(e / PL) * OWN + KEYS + pos];
                my[e] = pos < n_list[e / PL] ? my[e] : 0u;
                const bool in = my[e] != 0u && my[e] != (1u << 22) + 1u;
                hi = max(hi, in ? my[e] : 0u);
                nlo = max(nlo, in ? ~my[e] : 0u);
            }
            hi = (unsigned)__builtin_amdgcn_readlane((int)wave_max_last(hi), 63);
            nlo = (unsigned)__builtin_amdgcn_readlane((int)wave_max_last(nlo), 63);
            if (k > 0)
                topk_wave(my, k, forced, ~nlo, hi, own, [&](int pos, int t, unsigned) {
                    out[pos] = (int32_t)scratch[(t / (64 * PL)) * OWN + POS + t % (64 * PL)];
                });
        };
        if (n_sel <= 64) merge(std::integral_constant<int, 1>{});
        else merge(std::integral_constant<int, 2>{});
        if (threadIdx.x == 0) *nsel_out = k;
        for (int t = k + lane; t < n_sel; t += 64) out[t] = -1;
        return;
    }
    const int tid = threadIdx.x;
    const int lane = lane_id(), wave = tid >> 6;
    const int k = min(min(n_sel, n), cand_min > INT_MIN ? count_candidates(row, n, n_sink, n_local, cand_min) : n);
    if (tid == 0) *nsel_out = k;
    for (int t = k + tid; t < n_sel; t += 256) out[t] = -1;
    if (k == 0) return;
    if (k == n) {  // budget covers the row: everything, ascending
        for (int t = tid; t < n; t += 256) out[t] = t;
        return;
    }
    // Longer rows: three digits of eight bits, the row read again for each.
    unsigned *hist = scratch, *wtot_a = scratch + 256, *wtot_b = scratch + 260;
    unsigned &sh_bin = scratch[264], &sh_remaining = scratch[265];
    const bool cached = keys != nullptr && n <= TOPK_LDS_CAP;
    if (cached) {
        for (int t0 = 0; t0 < n; t0 += 4 * 256) {   // four loads in flight per thread
            int32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = t0 + e * 256 + tid;
                v[e] = t < n ? row[t] : 0;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = t0 + e * 256 + tid;
                if (t < n) keys[t] = key_of(t, v[e]);
            }
        }
    }
    auto key_at = [&](int i) -> unsigned { return cached ? keys[i] : key_of(i, row[i]); };

    // radix select, most significant digit first: after the loop `prefix` is the k-th largest key and
    // `remaining` the number of entries equal to it that belong to the selection
    unsigned prefix = 0, mask = 0, remaining = (unsigned)k;
    for (int shift = 16; shift >= 0; shift -= 8) {
        hist[tid] = 0;
        __syncthreads();
        // The leading digits of a row's scores are often all alike: when every candidate of a wavefront falls into one
        // bin, one lane adds their number (64 additions to one LDS word are served one after the other).
        for (int base = 0; base < n; base += 256) {   // uniform trip count
            const int t = base + tid;
            unsigned bin = 0;
            bool act = false;
            if (t < n) {
                const unsigned u = key_at(t);
                act = (u & mask) == prefix;
                bin = (u >> shift) & 255u;
            }
            const unsigned long long m = __ballot(act);
            if (m) {
                const int first = __ffsll(m) - 1;
                const unsigned fbin = (unsigned)__shfl((int)bin, first, WAVE);
                if (__all(!act || bin == fbin)) {
                    if (lane == first) atomicAdd(&hist[fbin], (unsigned)__popcll(m));
                } else if (act) {
                    atomicAdd(&hist[bin], 1u);
                }
            }
        }
        __syncthreads();
        if (wave == 0) {
            // lane l owns bins 255-4l .. 252-4l (descending); find where the running count reaches `remaining`
            unsigned c[4], s = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                c[e] = hist[255 - 4 * lane - e];
                s += c[e];
            }
            unsigned incl = s;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                unsigned o = __shfl_up(incl, off, WAVE);
                if (lane >= off) incl += o;
            }
            unsigned before = incl - s;
            if (before < remaining && incl >= remaining) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (before < remaining && before + c[e] >= remaining) {
                        sh_bin = 255 - 4 * lane - e;
                        sh_remaining = remaining - before;
                        before = 0xFFFFFFFFu;  // stop
                    } else if (before != 0xFFFFFFFFu) {
                        before += c[e];
                    }
                }
            }
        }
        __syncthreads();
        prefix |= sh_bin << shift;
        mask |= 0xFFu << shift;
        remaining = sh_remaining;
    }
    const unsigned T = prefix, need = remaining;

    // ordered compaction
    unsigned eq_before = 0, out_before = 0;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    for (int base = 0; base < n; base += 256) {
        const int i = base + tid;
        const bool valid = i < n;
        const unsigned u = valid ? key_at(i) : 0u;
        const bool is_gt = valid && u > T, is_eq = valid && u == T;
        const unsigned long long m_eq = __ballot(is_eq);
        if (lane == 0) wtot_a[wave] = __popcll(m_eq);
        __syncthreads();
        unsigned eq_rank = eq_before + __popcll(m_eq & lt_mask), eq_total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) eq_rank += wtot_a[w];
            eq_total += wtot_a[w];
        }
        const bool take = is_gt || (is_eq && eq_rank < need);
        const unsigned long long m_take = __ballot(take);
        if (lane == 0) wtot_b[wave] = __popcll(m_take);
        __syncthreads();
        unsigned pos = out_before + __popcll(m_take & lt_mask), take_total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) pos += wtot_b[w];
            take_total += wtot_b[w];
        }
        if (take) out[pos] = i;
        eq_before += eq_total;
        out_before += take_total;
        __syncthreads();  // wtot_a / wtot_b are rewritten by the next chunk
    }
}

}  // namespace fastar
