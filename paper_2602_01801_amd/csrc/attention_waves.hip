// Block-sparse attention in bf16 over few query blocks: a workgroup is one group of 32 queries, its S wavefronts share the
// group's tiles of 32 listed keys (wavefront s takes tiles s, s + S, ..) and put their sums together through LDS at the end.
//
// What bounds a launch of few query blocks is the chain of one tile after another (row look-up, gather, products,
// exponentials, products) on a chip mostly idle.  Kernels whose wavefronts share a tile, 32 queries each, meet at a barrier
// per tile and have a quarter of the workgroups; here a wavefront's tiles are its own: K and V go straight into its own piece
// of LDS (8 KB per tile at d = 64, 16 at d = 128), the next K under the softmax and the second product, the next V under the
// first, and nothing is met before the end.  The price is that the groups of a query block gather its rows once each, from
// L2, which is what bounds it as the blocks become many (at d = 128 18 TB/s), so the launcher keeps the other kernels there.
// Both products are computed transposed, as in the other bf16 kernels: S^T = K Q^T from the keys' bias on, O^T = V^T P^T with
// the S^T registers as the second operand.
// Measured (us, the kernel that took it before -> this one; launches back to back): d = 64: 2 blocks of 128 queries x 60 entries 66.7 ->
// 19.7, 57 x 47 60.5 -> 19.8, 39 blocks of 64 x 11 13.4 -> 8.7; d = 128: 64 x 7 13.1 -> 9.2 (the split two-block kernel), 27 x 18 17.8 ->
// 13.7 (its parts), 49 x 3 8.7 -> 7.1 (the one-block kernel).  Tiles of 64 keys and half of the resident wavefronts at d = 64: the same
// within 5 %; 16 wavefronts per group: slower at every size.
#include "common.hpp"

#include <type_traits>

namespace fastar {

namespace aw {

typedef __attribute__((ext_vector_type(4))) short s16x4;
constexpr int QW = 32;   // queries per workgroup
constexpr int TK = 32;   // keys per tile
constexpr float LN2 = 0.6931471805599453f;

// What masked positions fetch: rows that nothing selects need not be finite, and 0 * inf would reach the output.
__device__ __attribute__((aligned(16))) unsigned short zero_row[128];

__device__ __forceinline__ float max_across_halves(float x) {
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ bf16x8 lds_read_b128(unsigned addr) {
    bf16x8 r;
    asm volatile("ds_read_b128 %0, %1" : "=v"(r) : "v"(addr));
    return r;
}
// lane 4 q + m of a group of 16 receives element m of the 8-byte pieces addressed by lanes q, q + 4, q + 8, q + 12
template <int OFF>
__device__ __forceinline__ s16x4 lds_read_tr16(unsigned addr) {
    s16x4 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
    return r;
}
template <int N, class T>
__device__ __forceinline__ void wait_lds(T &a) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(N));
}
template <int N, class T>
__device__ __forceinline__ void wait_lds(T &a, T &b) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
template <int I, int N, class F>
__device__ __forceinline__ void unrolled(F &&f) {   // f(integral_constant<int, I>) .. f(<N - 1>)
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<I + 1, N>(f);
    }
}

// S: wavefronts of the workgroup; wavefront s takes tiles s, s + S, ..
// UNI: key blocks of 64 rows, so that a tile lies in one of them.
template <int D, int S, bool UNI>
__global__ __launch_bounds__(S * 64, D == 64 ? 4 : 2) void attn_bf16_waves_kernel(
    const unsigned short *__restrict__ Q, const unsigned short *__restrict__ K, const unsigned short *__restrict__ V,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int BQ, int bk_shift, int n_sel, int n_qb, int groups_per_block, int n_groups,
    float scale_log2, float inv_scale_log2, unsigned short *__restrict__ O, float *__restrict__ lse) {
    constexpr int NDB = D / 32, NS = D / 16;
    constexpr int RB = D * 2, RP = RB / 16, RI = 64 / RP;   // bytes and 16-byte pieces of a row, rows per direct load
    constexpr int NI = TK / RI;               // direct loads per tile
    constexpr int PS = 65;                    // pitch of a register's 64 lanes among the partial sums (banks)
    __shared__ __attribute__((aligned(1024))) unsigned char tiles[S][2 * TK * RB];
    __shared__ __attribute__((aligned(16))) float tbiases[S][TK];
    __shared__ unsigned trows[S][TK];
    __shared__ __attribute__((aligned(16))) int tcnts[S][64];   // multiplicities of a tile's positions
    __shared__ float pm[S][QW], pl[S][QW];
    static_assert(2 * TK * RB >= 16 * NDB * PS * 4 / 2, "half of the partial sums fit");
    const int tid = threadIdx.x, lane = tid & 63;
    const int ws = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int per = ((int)gridDim.x + 7) / 8;   // the grid is a multiple of 8; contiguous ranges of groups per XCD
    const int gi = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (gi >= n_groups) return;
    const int b_all = gi / groups_per_block, h = b_all / n_qb, b = b_all % n_qb;
    const int q0 = b * BQ + (gi % groups_per_block) * QW;
    const int nq_here = min(QW, n_q - q0);
    if (nq_here <= 0) return;                   // (uniform over the workgroup)
    const int L = min(len[h], C);
    const int n_listed = L > 0 ? min(nsel[b_all], n_sel) : 0;
    const int32_t *sel_row = sel + (size_t)b_all * n_sel;
    const int n_pos = max(n_listed, 0) << bk_shift;
    const int nt = (n_pos + TK - 1) / TK;
    const int32_t *cnt_h = cnt ? cnt + (size_t)h * C : nullptr;
    const unsigned short *Kh = K + (size_t)h * C * D;
    const unsigned short *Vh = V + (size_t)h * C * D;

    bf16x8 qf[NS];
    {
        const unsigned short *qrow = Q + ((size_t)h * n_q + q0 + min(col, nq_here - 1)) * D;
#pragma unroll
        for (int s = 0; s < NS; ++s) qf[s] = *(const bf16x8 *)(qrow + 16 * s + 8 * g);
    }
    f32x16 o[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.0f;
    float m_run = -INFINITY, m_safe = 0.0f, l_run = 0.0f;   // of this lane's query; l_run over this half's keys only

    unsigned char *ktile = tiles[ws], *vtile = tiles[ws] + TK * RB;
    float *tbias = tbiases[ws];
    unsigned *trow = trows[ws];
    // What is known of a tile: its list entry (of position lane % TK; UNI: of the whole tile), asked for a step before it is
    // resolved; `row`, the position's slot (-1: masked), `whole`: UNI and no position masked, `first`: UNI, its first slot.
    const int plane = lane & (TK - 1);
    auto entry = [&](int t) {
        const int e = UNI ? t >> 1 : (t * TK + plane) >> bk_shift;
        return sel_row[min(e, n_listed - 1)];
    };
    struct Tile {
        int first, row;
        bool whole;
    };
    auto resolve = [&](int t, int kb) {
        Tile x;
        if (UNI) {
            x.first = kb * 64 + (t & 1) * TK;
            const int live = kb < 0 ? 0 : L - x.first;
            x.whole = live >= TK;
            x.row = plane < live ? x.first + plane : -1;
        } else {
            const int p = t * TK + plane;
            const int k = (kb << bk_shift) + (p & ((1 << bk_shift) - 1));
            x.first = 0;
            x.whole = false;
            x.row = p < n_pos && kb >= 0 && k < L ? k : -1;
        }
        return x;
    };
    // A tile of K or V straight into LDS: piece c of row w lies at piece c ^ x(w) of it, x(w) = w / 2 % 8 (d = 64) or w % 16, so
    // that 16 lanes on neighbouring rows, or on a row's pieces, lie on different banks.
    const int lrow = lane / RP;
    const unsigned off0 = (unsigned)(lrow * RB + 16 * ((lane % RP) ^ (lane >> 4)));
    auto load_tile = [&](const Tile &x, const unsigned short *base_h, unsigned char *dst) {
        if (UNI && x.whole) {
            const char *base = (const char *)(base_h + (size_t)x.first * D);
#pragma unroll
            for (int i = 0; i < NI; ++i)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(base + i * RI * RB + (off0 ^ (unsigned)(16 * (D == 64 ? 4 * (i & 1) : (4 * i) & 15)))),
                    (__attribute__((address_space(3))) void *)(dst + i * RI * RB), 16, 0, 0);
        } else {
            if (lane < TK) trow[lane] = x.row >= 0 ? (unsigned)x.row : 0xFFFFFFFFu;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const unsigned w = trow[i * RI + lrow];
                const unsigned piece = (off0 ^ (unsigned)(16 * (D == 64 ? 4 * (i & 1) : (4 * i) & 15))) & (RB - 1);
                const char *row = w == 0xFFFFFFFFu ? (const char *)zero_row : (const char *)(base_h + (size_t)w * D);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + piece),
                                                 (__attribute__((address_space(3))) void *)(dst + i * RI * RB), 16, 0, 0);
            }
        }
    };
    auto lds_addr = [](unsigned char *p) { return (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)p; };
    // operand addresses, by exclusive or: K piece 2 s + g of row col is at kaddr ^ 32 s
    const unsigned kaddr = lds_addr(ktile) + (unsigned)(col * RB + 16 * (g ^ (D == 64 ? (col >> 1) & 7 : col & 15)));
    // V^T: lane (of 16) i addresses columns 4 (i % 4) .. of key i / 4, see lds_read_tr16; column block db at vaddr ^ 64 db,
    // keys + 8 at vaddr ^ VR
    constexpr unsigned VR = D == 64 ? 64 : 128;
    unsigned vaddr;
    {
        const int j = (lane & 15) >> 2, q = lane & 3, hc = (lane >> 4) & 1;
        const int xl = D == 64 ? 2 * g + (j >> 1) : 4 * g + j;
        vaddr = lds_addr(vtile) + (unsigned)((4 * g + j) * RB + 16 * ((2 * hc + (q >> 1)) ^ xl) + 8 * (q & 1));
    }
    // Multiplicities go into LDS like the tiles: a load into a register would have to be waited for by itself, and the compiler's
    // wait for anything but direct loads drains those too.  For the same reason what they bring is read by assembly.
    auto load_cnt = [&](const Tile &x) {
        if (cnt_h)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(cnt_h + max(x.row, 0)),
                                             (__attribute__((address_space(3))) void *)tcnts[ws], 4, 0, 0);
    };
    const unsigned caddr = lds_addr((unsigned char *)tcnts[ws]) + 4 * lane, baddr = lds_addr((unsigned char *)tbias) + 16 * g;
    auto store_bias = [&](const Tile &x) {
        float bias = 0.0f;
        if (cnt_h) {
            int n;
            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(n) : "v"(caddr) : "memory");
            bias = __log2f((float)n) * inv_scale_log2;
        }
        if (lane < TK) tbias[lane] = x.row < 0 ? -INFINITY : bias;
        asm volatile("" ::: "memory");
    };

    Tile cur = {0, -1, false};
    int kb_next = -1;
    if (ws < nt) {
        cur = resolve(ws, entry(ws));
        kb_next = entry(ws + S);
        load_cnt(cur);
        load_tile(cur, Kh, ktile);
        load_tile(cur, Vh, vtile);
        if (!UNI) asm volatile("" : "+v"(kb_next));
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NI) : "memory");
        store_bias(cur);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(qf[s]));   // waited for here, not in the loop
    for (int t = ws; t < nt; t += S) {
        const bool more = t + S < nt;
        const Tile next = resolve(t + S, kb_next);
        // the tile's K has landed when at most its V, asked for behind it, is out
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI) : "memory");
        // scores, from the keys' bias on
        f32x16 s;
        {
            f32x4 bv[4];
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:32\n\tds_read_b128 %2, %4 offset:64\n\t"
                         "ds_read_b128 %3, %4 offset:96\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(bv[0]), "=&v"(bv[1]), "=&v"(bv[2]), "=&v"(bv[3])
                         : "v"(baddr)
                         : "memory");
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = bv[v >> 2][v & 3];
            bf16x8 kf[NS];
#pragma unroll
            for (int c = 0; c < NS; ++c) kf[c] = lds_read_b128(kaddr ^ (unsigned)(32 * c));
            unrolled<0, NS>([&](auto c) {
                wait_lds<NS - 1 - c>(kf[c]);
                s = mfma_bf16_32x32x16(kf[c], qf[c], s);
            });
        }
        asm volatile("" ::: "memory");
        if (more) {
            kb_next = entry(t + 2 * S);
            load_cnt(next);
            load_tile(next, Kh, ktile);   // the tile in LDS has been read: wait_lds saw its last operand
        }
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = max_across_halves(mx) * scale_log2;
        if (__any(mx > m_run)) {   // (uniform) a new maximum: what is summed up so far moves to it
            const float m_new = fmaxf(m_run, mx);
            const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            m_safe = m_new == -INFINITY ? 0.0f : m_new;   // every key so far masked
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
        }
        float ls[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], scale_log2, -m_safe));
            ls[v & 3] += s[v];
        }
        l_run += (ls[0] + ls[1]) + (ls[2] + ls[3]);
        // V (and the next tile's multiplicities) have landed when at most the next tile's K is out
        if (more) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI) : "memory");
            store_bias(next);
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        {
            s16x4 vf[2][NDB][2];   // by steps of 16 keys
            unrolled<0, 2>([&](auto st) {
                unrolled<0, NDB>([&](auto db) {
                    vf[st][db][0] = lds_read_tr16<16 * st * RB>(vaddr ^ (unsigned)(64 * db));
                    vf[st][db][1] = lds_read_tr16<(16 * st + 8) * RB>(vaddr ^ (unsigned)(64 * db) ^ VR);
                });
            });
            unrolled<0, 2>([&](auto st) {
                bf16x8 pf;
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[e] = (__bf16)s[8 * st + e];
                unrolled<0, NDB>([&](auto db) {
                    constexpr int behind = 2 * (2 * NDB - 1 - (st * NDB + db));
                    wait_lds<(behind > 15 ? 15 : behind)>(vf[st][db][0], vf[st][db][1]);
                    struct { s16x4 a, b; } pr = {vf[st][db][0], vf[st][db][1]};
                    bf16x8 a;
                    __builtin_memcpy(&a, &pr, 16);
                    o[db] = mfma_bf16_32x32x16(a, pf, o[db]);
                });
            });
        }
        asm volatile("" ::: "memory");
        if (more) load_tile(next, Vh, vtile);
        cur = next;
    }
    float l_tot = l_run + shfl_xor(l_run, 32);

    // The partial sums meet in LDS, half of the columns at a time, and leave it in rows: o[db][v] is column
    // 32 db + 8 (v / 4) + 4 g + v % 4 of query col.
    if (g == 0) {
        pm[ws][col] = m_run;
        pl[ws][col] = l_tot;
    }
    float *po = (float *)tiles[ws];
    constexpr int PP = RP / 2;   // 8-column pieces of half a row
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __syncthreads();   // everyone is done with the tiles, or with the other half
#pragma unroll
        for (int i = 0; i < 8 * NDB; ++i) po[i * PS + lane] = o[(half * 8 * NDB + i) / 16][(half * 8 * NDB + i) % 16];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < (QW * PP + S * 64 - 1) / (S * 64); ++it) {
            const int at = it * S * 64 + tid;
            const int row = at / PP, piece = at % PP;
            if (QW * PP % (S * 64) != 0 && at >= QW * PP) break;
            float m_all = -INFINITY;
#pragma unroll
            for (int k = 0; k < S; ++k) m_all = fmaxf(m_all, pm[k][row]);
            float wgt[S], l_all = 0.0f;
#pragma unroll
            for (int k = 0; k < S; ++k) {
                wgt[k] = m_all == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(pm[k][row] - m_all);
                l_all += wgt[k] * pl[k][row];
            }
            const float inv = l_all > 0.0f ? 1.0f / l_all : 0.0f;
            float r[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                r[e] = 0.0f;
#pragma unroll
                for (int k = 0; k < S; ++k) r[e] += wgt[k] * ((const float *)tiles[k])[(4 * piece + (e & 3)) * PS + row + 32 * (e >> 2)];
                r[e] *= inv;
            }
            if (row < nq_here) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(r[2 * e], r[2 * e + 1]);
                *(u32x4 *)(O + ((size_t)h * n_q + q0 + row) * D + half * (D / 2) + 8 * piece) = w;
                if (lse && half == 0 && piece == 0)
                    lse[(size_t)h * n_q + q0 + row] = l_all > 0.0f ? (m_all + __log2f(l_all)) * LN2 : -INFINITY;
            }
        }
    }
}

template <int D>
static auto kernel_of(int S, bool uni) {
    return S == 8 ? (uni ? attn_bf16_waves_kernel<D, 8, true> : attn_bf16_waves_kernel<D, 8, false>)
         : S == 4 ? (uni ? attn_bf16_waves_kernel<D, 4, true> : attn_bf16_waves_kernel<D, 4, false>)
                  : (uni ? attn_bf16_waves_kernel<D, 2, true> : attn_bf16_waves_kernel<D, 2, false>);
}

}  // namespace aw

int launch_attn_bf16_waves(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len, int H, int C,
                           int d, const int32_t *sel, const int32_t *nsel, int BQ, int bk_shift, int n_sel, float scale_log2, int S,
                           void *O, float *lse, hipStream_t s) {
    using namespace aw;
    const int n_qb = (n_q + BQ - 1) / BQ, gpb = BQ / QW;
    const long long n_groups = (long long)H * n_qb * gpb;
    if (n_groups >= (1ll << 30)) return FASTAR_ERR_UNSUPPORTED;
    const bool uni = bk_shift == 6;
    const dim3 grid((unsigned)((n_groups + 7) / 8 * 8));
    auto k = d == 64 ? kernel_of<64>(S, uni) : kernel_of<128>(S, uni);
    hipLaunchKernelGGL(k, grid, dim3(S * 64), 0, s, (const unsigned short *)Q, (const unsigned short *)K, (const unsigned short *)V, cnt,
                       len, sel, nsel, n_q, C, BQ, bk_shift, n_sel, n_qb, gpb, (int)n_groups, scale_log2, 1.0f / scale_log2,
                       (unsigned short *)O, lse);
    if (hipGetLastError() != hipSuccess) return FASTAR_ERR_HIP;
    return FASTAR_OK;
}

}  // namespace fastar
