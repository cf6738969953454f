// Block-sparse attention in fp32 (sparse_attn_fwd with FASTAR_F32): fp32 products, sums, softmax and outputs, on the
// fp32 matrix instructions.
//
// v_mfma_f32_16x16x4_f32 multiplies and adds in fp32 like a chain of fma, at twice the rate of the vector ALU, and needs
// no operand broadcast: a wavefront owns 16 queries and walks tiles of 32 listed keys, with both contractions transposed
// so that everything that belongs to a query stays in its lane (lane l: query l % 16):
//     S^T = K Q^T    A = K rows by way of LDS (lane l: key l % 16, coordinates 16 c + 4 (l / 16) .. + 3),
//                    B = Q in registers; accumulator register v of lane l is key 4 (l / 16) + v
//     O^T = V^T P^T  B = the S^T registers as they are (k slot l / 16 of step v is key 4 (l / 16) + v),
//                    A = V rows straight from global memory: which output column a row of A stands for is free, so block
//                    4 g + e of D / 16 takes columns 64 g + 4 (l % 16) + e: 16 lanes read 256 consecutive bytes of a row
// No tile is shared inside a workgroup, so there is no barrier in the loop: a wavefront's tile of K goes from global memory
// straight into its own piece of LDS, under the second product of the tile before; V is in flight under the first.
//
// Why K goes by way of LDS: operand A wants neighbouring lanes on different rows, and a load whose neighbouring lanes lie on
// different 64-byte pieces takes one piece at a time: 16 rows x 64 bytes per instruction bring 38 bytes per ns and compute
// unit wherever the data comes from, 1 KB in two rows or 256 bytes in four rows 125 to 135 from L2 (probe of such loads).  With K
// read that way every size ran at 9 TB/s through the first level.
// What bounds it now: where the chip is full, the matrix instructions: with the loads, the LDS reads, the softmax and the look-ups
// taken out they alone take 0.87 of the launch (2.2 us per tile of 128 instructions and SIMD: real data lowers their
// rate, and no vector instruction runs beside an fp32 one, probe); one wavefront per SIMD (196 groups) adds the latency of a
// tile's chain.  Measured, d = 128, 64-row blocks, K by rows -> by way of LDS, in us: 196 groups x 15 blocks 34.4 -> 26.4, 256 x 63 113 -> 89,
// 1248 x 59 489 -> 402, 3680 x 13 330 -> 261 (92 TFLOP/s; the instructions alone reach 155 on data that does not change);
// d = 64: 156 groups x 47 blocks 54.7 -> 37.4, 1024 x 32 116 -> 103.  Asking of every tile whether a weight lies below 2^-126 is 2 to 5 % of
// that where the chip is full (389, 256, 98.5 without; in one branch with the maximum's: 403, 264, 107).  Tried: scores of the next tile under the softmax (no gain:
// nothing overlaps), loads spread among the products (no gain), tiles of 16 keys with three wavefronts per SIMD (no gain).
#include "common.hpp"

#include <type_traits>

namespace fastar {

namespace f32a {

constexpr int QW = 16;    // queries per wavefront
constexpr int TKF = 32;   // listed keys per step
constexpr float LN2 = 0.6931471805599453f;

__device__ __forceinline__ f32x4 mfma_f32_16x16x4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Maximum over the four lanes of a query (lane % 16).
__device__ __forceinline__ float max_of_quarters(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// What masked positions (padding, rows past len, the end of the list) fetch: a row of the cache that nothing selects need not
// be finite, and inf + -inf or 0 * inf would reach the output.
__device__ __attribute__((aligned(16))) float zero_row[128];

// KS: wavefronts of a workgroup; they share one query group and split its tiles.
// UNI: key blocks of 32 or 64 rows, so that a tile lies in one of them.
template <int D, int KS, bool UNI>
__global__ __launch_bounds__(KS * 64, 2) void attn_f32_kernel(
    const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V, const int32_t *__restrict__ cnt,
    const int32_t *__restrict__ len, const int32_t *__restrict__ sel, const int32_t *__restrict__ nsel, int n_q, int C,
    int BQ, int BK, int n_sel, int n_qb, int groups_per_block, int n_groups, float scale_log2, float *__restrict__ O,
    float *__restrict__ lse) {
    constexpr int CH = D / 16;   // 16-coordinate chunks of a row, and V columns per lane
    constexpr int RP = D / 4;    // 16-byte pieces of a row
    constexpr int RI = 64 / RP;  // rows one direct load brings: 64 lanes of 16 bytes
    constexpr int PS = 65;       // pitch of a register's 64 lanes among the partial sums (banks)
    __shared__ __attribute__((aligned(16))) long long trows[KS][TKF];
    __shared__ __attribute__((aligned(16))) float tbiases[KS][TKF];
    // the wavefronts' K tiles; after the loop the partial O^T, as it sits in the registers
    __shared__ __attribute__((aligned(1024))) float ktiles[KS][TKF * D];   // rows at multiples of their size: see kaddr
    static_assert(TKF * D >= 4 * CH * PS, "the partial sums fit");
    __shared__ float pm[KS][QW], pl[KS][QW];   // reference maxima and row sums
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qc = lane & 15, quarter = lane >> 4;
    // contiguous ranges of query groups per XCD: the groups of a head share its L2
    const int per = ((int)gridDim.x + 7) / 8;   // the grid is a multiple of 8
    const int gi = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);   // (head, block, group of the block)
    if (gi >= n_groups) return;
    const int b_all = gi / groups_per_block, h = b_all / n_qb, b = b_all % n_qb;
    const int q_in = (gi % groups_per_block) * QW;           // first query of the group inside its block
    const int q0 = b * BQ + q_in;
    const int nq_here = min(min(QW, BQ - q_in), n_q - q0);
    if (nq_here <= 0) return;                                // (uniform over the workgroup)
    const int L = min(len[h], C);
    const int n_listed = L > 0 ? min(nsel[b_all], n_sel) : 0;
    const int32_t *sel_row = sel + (size_t)b_all * n_sel;
    const int n_pos = max(n_listed, 0) * BK;
    const int nt = (n_pos + TKF - 1) / TKF;
    const int32_t *cnt_h = cnt ? cnt + (size_t)h * C : nullptr;
    const float *Kh = K + (size_t)h * C * D;
    const float *Vh = V + (size_t)h * C * D;

    f32x4 q[CH], o[CH];
    {
        const float *qrow = Q + ((size_t)h * n_q + q0 + min(qc, nq_here - 1)) * D;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            q[c] = *(const f32x4 *)(qrow + 16 * c + 4 * quarter);
            o[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    float m_run = -INFINITY, m_safe = 0.0f, l_run = 0.0f;   // of this lane's query; l_run over this lane's keys only

    // Row table of this wavefront's tile (byte offsets from the head's own K or V) for tiles with masked positions or of
    // small key blocks, and the bias of its 32 positions.
    long long *trow = trows[ks];
    float *tbias = tbiases[ks], *ktile = ktiles[ks];
    const long long zk = (const char *)zero_row - (const char *)Kh, zv = (const char *)zero_row - (const char *)Vh;
    // What is known of a tile: its list entry (of position lane % 32; UNI: of the whole tile), asked for a step before it is
    // resolved; `row`, the position's slot (-1: masked), `whole`: UNI and no position masked, `first`: UNI, its first slot;
    // the position's multiplicity, asked for a step before it is used.
    const int eshift = UNI ? __builtin_ctz(BK / TKF) : 0;
    const int pl32 = lane & (TKF - 1);
    auto entry = [&](int t) {
        if (UNI) return sel_row[min(t >> eshift, n_listed - 1)];
        return sel_row[min((t * TKF + pl32) / BK, n_listed - 1)];
    };
    struct Tile {
        int first, row;
        bool whole;
    };
    auto resolve = [&](int t, int kb) {
        Tile x;
        if (UNI) {
            x.first = kb * BK + (t & ((1 << eshift) - 1)) * TKF;
            const int live = kb < 0 ? 0 : L - x.first;
            x.whole = live >= TKF;
            x.row = pl32 < live ? x.first + pl32 : -1;
        } else {
            const int p = t * TKF + pl32;
            const int k = kb * BK + p % BK;
            x.first = 0;
            x.whole = false;
            x.row = p < n_pos && kb >= 0 && k < L ? k : -1;
        }
        return x;
    };
    // branch-free, so that waiting for it does not drain the loads behind it
    const int32_t *np = cnt_h ? cnt_h : len;
    const unsigned nmask = cnt_h ? 0x7FFFFFFFu : 0u;
    auto multiplicity = [&](const Tile &x) { return np[(unsigned)max(x.row, 0) & nmask]; };
    const int lrow = lane / RP, lpiece = lane % RP;
    unsigned koff[16 / RI];   // this lane's piece of its row in the first 16 rows' loads
#pragma unroll
    for (int i = 0; i < 16 / RI; ++i) koff[i] = (unsigned)(lrow * (D * 4) + 16 * (lpiece ^ (i * RI + lrow)));
    // K of a tile straight into LDS, rows [from, to) of it; piece c of row w lies at piece c ^ (w & 15) of it
    auto load_k = [&](const Tile &x, int from, int to) {
        if (UNI && x.whole) {
            const char *base = (const char *)(Kh + (size_t)x.first * D);
#pragma unroll
            for (int i = from / RI; i < to / RI; ++i)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(base + i * RI * D * 4 + koff[i % (16 / RI)]),
                    (__attribute__((address_space(3))) void *)(ktile + i * RI * D), 16, 0, 0);
        } else {
            if (from == 0 && lane < TKF) trow[lane] = x.row >= 0 ? (long long)x.row * (D * 4) : zk;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int i = from / RI; i < to / RI; ++i) {
                const int w = i * RI + lrow;
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)((const char *)Kh + trow[w] + 16 * (lpiece ^ (w & 15))),
                    (__attribute__((address_space(3))) void *)(ktile + i * RI * D), 16, 0, 0);
            }
        }
    };
    // V row of this lane's key 16 hh + 4 quarter + v, i = 4 hh + v
    float vf[2][4][CH];
    auto load_v = [&](auto whole, const Tile &x, int i) {
        const char *vp;
        if constexpr (decltype(whole)::value) {
            vp = (const char *)(Vh + (size_t)x.first * D) + (unsigned)(quarter * (16 * D) + 16 * qc + ((i >> 2) * 16 + (i & 3)) * (D * 4));
        } else {
            vp = (const char *)(Vh + 4 * qc) + trow[(i >> 2) * 16 + 4 * quarter + (i & 3)];
        }
#pragma unroll
        for (int c = 0; c < CH; c += 4) {
            const f32x4 w = *(const f32x4 *)(vp + 64 * c);
#pragma unroll
            for (int e = 0; e < 4; ++e) vf[i >> 2][i & 3][c + e] = w[e];
        }
    };
    // LDS address of piece `quarter` of this lane's key of the first half tile; chunk c is 64 c bytes on, by exclusive or
    const unsigned kaddr = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float *)ktile + (unsigned)(qc * (D * 4) + 16 * (quarter ^ qc));
    auto read_k = [&](int c, f32x4 (&f)[2]) {
        const unsigned at = kaddr ^ (unsigned)(64 * c);
        asm volatile("ds_read_b128 %0, %1" : "=v"(f[0]) : "v"(at));
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f[1]) : "v"(at), "n"(16 * D * 4));
    };
    auto wait_k = [&](f32x4 (&f)[2], int behind) {   // at most `behind` LDS reads of read_k later than f's
        if (behind == 2) asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(f[0]), "+v"(f[1]));
        else if (behind == 1) asm volatile("s_waitcnt lgkmcnt(2)" : "+v"(f[0]), "+v"(f[1]));
        else asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]));
    };
    // S^T of the tile in LDS
    auto scores = [&](f32x4 (&s)[2]) {
        f32x4 kf[4][2];   // operands are asked for two chunks ahead
        read_k(0, kf[0]);
        read_k(1, kf[1]);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) s[hh] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (c + 2 < CH) read_k(c + 2, kf[(c + 2) & 3]);
            wait_k(kf[c & 3], c + 2 < CH ? 2 : c + 1 < CH ? 1 : 0);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) s[hh] = mfma_f32_16x16x4(kf[c & 3][hh][e], q[c][e], s[hh]);
        }
    };
    auto store_bias = [&](const Tile &x, int n) {
        const float bias = x.row < 0 ? -INFINITY : cnt_h ? log2f((float)n) : 0.0f;
        if (lane < TKF) tbias[lane] = bias;
    };

    Tile cur = {0, -1, false};
    int n_cur = 1, kb_next = -1;
    if (ks < nt) {
        cur = resolve(ks, entry(ks));
        n_cur = multiplicity(cur);
        kb_next = entry(ks + KS);
        load_k(cur, 0, TKF);
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) asm volatile("" : "+v"(q[c]));   // waited for here, not in the loop
    asm volatile("" : "+v"(n_cur));
    if (!UNI) asm volatile("" : "+v"(kb_next));
    auto step = [&](auto whole, int t) {
        store_bias(cur, n_cur);
        if constexpr (!decltype(whole)::value) {
            if (lane < TKF) trow[lane] = cur.row >= 0 ? (long long)cur.row * (D * 4) : zv;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        const Tile next = resolve(t + KS, kb_next);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // K of the tile has landed
        int n_next = multiplicity(next);
        kb_next = entry(t + 2 * KS);
#pragma unroll
        for (int i = 0; i < 8; ++i) load_v(whole, cur, i);
        f32x4 s[2];
        scores(s);
        f32x4 bv[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) bv[hh] = *(const f32x4 *)(tbias + 16 * hh + 4 * quarter);
        // V is waited for before the next K is asked for: the compiler's wait would be for both
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int c = 0; c < CH; ++c) asm volatile("" : "+v"(vf[hh][v][c]));
        asm volatile("" : "+v"(n_next)::"memory");
        if (!UNI) asm volatile("" : "+v"(kb_next));
        if (t + KS < nt) load_k(next, 0, TKF);   // the tile in LDS has been read: wait_k saw its last operand
        float mx = -INFINITY, mn = INFINITY;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[hh][v] = fmaf(s[hh][v], scale_log2, bv[hh][v]);
                mx = fmaxf(mx, s[hh][v]);
                mn = fminf(mn, s[hh][v]);
            }
        mx = max_of_quarters(mx);
        if (__any(mx > m_run)) {   // (uniform) a new maximum: what is summed up so far moves to it
            const float m_new = fmaxf(m_run, mx);
            const float alpha = exp2f(m_run - m_new);                    // m_new is finite where it is new
            const float al = m_new == -INFINITY ? 1.0f : alpha;
            m_run = m_new;
            m_safe = m_new == -INFINITY ? 0.0f : m_new;                  // every key so far masked
            l_run *= al;
#pragma unroll
            for (int c = 0; c < CH; ++c) o[c] *= al;
        }
        auto weigh = [&](auto exponential) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[hh][v] = exponential(s[hh][v] - m_safe);
                    l_run += s[hh][v];
                }
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
#pragma unroll
                    for (int c = 0; c < CH; ++c) o[c] = mfma_f32_16x16x4(vf[hh][v][c], s[hh][v], o[c]);
                }
        };
        // The bare instruction makes weights below 2^-126 zero, exp2f does not, at five instructions each; elsewhere they are the
        // same.  The products are in either branch so that the exponentials run between them.
        if (__any(mn - m_safe < -126.0f)) weigh([](float x) { return exp2f(x); });   // uniform
        else weigh([](float x) { return __builtin_amdgcn_exp2f(x); });
        cur = next;
        n_cur = n_next;
    };
    for (int t = ks; t < nt;) {   // loops of their own, so that the sums stay in place
        if constexpr (UNI)
            for (; t < nt && cur.whole; t += KS) step(std::true_type{}, t);
        for (; t < nt && !(UNI && cur.whole); t += KS) step(std::false_type{}, t);
    }
    float l_tot = l_run + shfl_xor(l_run, 16);
    l_tot += shfl_xor(l_tot, 32);

    // The partial sums meet in LDS and leave it in rows.  o[c][v]: column 64 (c / 4) + 4 (4 quarter + v) + c % 4 of query qc.
    float *po = ktile;   // every wavefront is done with its own tiles
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < CH; ++c) po[(v * CH + c) * PS + lane] = o[c][v];
    if (quarter == 0) {
        pm[ks][qc] = m_run;
        pl[ks][qc] = l_tot;
    }
    __syncthreads();
    static_assert(QW * RP % (KS * 64) == 0, "whole rounds");
#pragma unroll
    for (int i = 0; i < QW * RP / (KS * 64); ++i) {
        const int row = (i * KS * 64 + tid) / RP, piece = tid % RP;   // 4 columns of one query
        float m_all = -INFINITY;
#pragma unroll
        for (int k = 0; k < KS; ++k) m_all = fmaxf(m_all, pm[k][row]);
        float wgt[KS], l_all = 0.0f;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            wgt[k] = m_all == -INFINITY ? 0.0f : exp2f(pm[k][row] - m_all);
            l_all += wgt[k] * pl[k][row];
        }
        const float inv = l_all > 0.0f ? 1.0f / l_all : 0.0f;
        const float *pr = &ktiles[0][0] + ((piece & 3) * CH + 4 * (piece >> 4)) * PS + row + 16 * ((piece >> 2) & 3);
        f32x4 r = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < KS; ++k) r[e] += wgt[k] * pr[k * (TKF * D) + e * PS];
        if (row < nq_here) {
            *(f32x4 *)(O + ((size_t)h * n_q + q0 + row) * D + 4 * piece) = r * inv;
            if (lse && piece == 0) lse[(size_t)h * n_q + q0 + row] = l_all > 0.0f ? (m_all + log2f(l_all)) * LN2 : -INFINITY;
        }
    }
}

template <int D>
static auto kernel_of(int ks, bool uni) {
    return ks == 2 ? (uni ? attn_f32_kernel<D, 2, true> : attn_f32_kernel<D, 2, false>)
                   : (uni ? attn_f32_kernel<D, 4, true> : attn_f32_kernel<D, 4, false>);
}

}  // namespace f32a

int launch_attn_f32(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len, int H, int C,
                    int d, const int32_t *sel, const int32_t *nsel, int BQ, int BK, int n_sel, float scale_log2, void *O,
                    float *lse, hipStream_t s) {
    using namespace f32a;
    const int n_qb = (n_q + BQ - 1) / BQ, gpb = (BQ + QW - 1) / QW;
    const long long n_groups = (long long)H * n_qb * gpb;
    if (n_groups >= (1ll << 30)) return FASTAR_ERR_UNSUPPORTED;
    const bool uni = BK == 32 || BK == 64;
    const long long n_tiles = ((long long)n_sel * BK + TKF - 1) / TKF;
    // Two wavefronts per group where four would have a tile or none each: up to two tiles always (us with two / four wavefronts:
    // 224 groups 7.3 / 7.6, 1152 groups 18.5 / 25.3, 3680 groups 41 / 62), up to four where the chip is full (1152 groups
    // 26.3 / 27.2; 32 groups of 8 tiles of 64 coordinates 8.7 / 6.3).
    const int ks = n_tiles <= 2 || (n_tiles <= 4 && n_groups >= 1024) ? 2 : 4;
    const dim3 grid((unsigned)((n_groups + 7) / 8 * 8));
    hipLaunchKernelGGL((d == 128 ? kernel_of<128>(ks, uni) : kernel_of<64>(ks, uni)), grid, dim3(ks * 64), 0, s, (const float *)Q,
                       (const float *)K, (const float *)V, cnt, len, sel, nsel, n_q, C, BQ, BK, n_sel, n_qb, gpb, (int)n_groups,
                       scale_log2, (float *)O, lse);
    if (hipGetLastError() != hipSuccess) return FASTAR_ERR_HIP;
    return FASTAR_OK;
}

}  // namespace fastar
