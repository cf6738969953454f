// Block-sparse attention over the selected key blocks (Eq. 1 restricted to the candidate set of
// Sec. 5.1; logits shifted by +ln(cnt) as Lemma 1 prescribes for merged groups).
//
// bf16 path (matrix cores).  One workgroup = one query block of BQ = 32*NW queries, one wavefront
// = 32 queries.  Key tiles of 64 rows are gathered by the selection list into LDS (K row-major,
// V transposed so that a lane can fetch 4 consecutive keys of one value column), the next tile is
// prefetched into registers while the current one is consumed.  Both contractions are computed
// "transposed" so that every per-query quantity lives in one lane:
//     S^T = K Q^T   (A = K tile from LDS, B = Q fragment held in registers)  -> lane = query, regs = keys
//     O^T = V^T P^T (A = V^T tile from LDS, B = P^T = the S^T registers, no data movement) -> lane = query
// Softmax runs in fp32 in the log2 domain with a running maximum; masked keys (padding of the list,
// slots beyond len) get a -inf bias and zeroed K/V rows.
//
// Few query blocks (S > 1): the workgroup has S groups of wavefronts, group i takes every S-th tile from i on in tile space
// of its own, and group 0 adds the others' sums up at the end.  A tile costs a chain of row table, gather, staging and
// products (about 2 us for a lone workgroup), which otherwise follow one another: 39 blocks of
// 64 queries x 11 tiles 21.5 -> 13.5 us with four groups.
//
// fp32: attention_f32.hip.
#include "common.hpp"

namespace fastar {

constexpr int TK = 64;  // keys per tile
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

struct __attribute__((aligned(16))) TileMeta {
    int idx[TK];     // cache row of each tile position, -1 = masked
    float bias[TK];  // log2(cnt) of that row, -inf when masked
};

// Fill the row table of tile `t` (p = the thread's index in its group; threads 0..63).
__device__ __forceinline__ void fill_meta(TileMeta &m, int t, const int32_t *__restrict__ sel_row, int n_listed,
                                          int bk_shift, int L, const int32_t *__restrict__ cnt_h, int p) {
    if (p < TK) {
        const int listpos = t * TK + p;
        const int entry = listpos >> bk_shift;
        int key = -1;
        if (entry < n_listed) {
            const int kb = sel_row[entry];
            if (kb >= 0) {
                key = (kb << bk_shift) + (listpos & ((1 << bk_shift) - 1));
                if (key >= L) key = -1;
            }
        }
        float bias = -INFINITY;
        if (key >= 0) bias = cnt_h ? __log2f((float)cnt_h[key]) : 0.0f;
        m.idx[p] = key;
        m.bias[p] = bias;
    }
}

template <int D, int NW>
struct AttnCfg {
    static constexpr int NT = NW * 64;
    static constexpr int KSTR = D + 8;    // bf16 elements per K row in LDS (16-byte pad: conflict-free b128 reads)
    static constexpr int VSTR = TK + 4;   // bf16 elements per V^T row in LDS
    static constexpr int CPR = D / 8;     // 16-byte chunks per row
    static constexpr int KCH = TK * CPR / NT;                  // K chunks staged per thread
    static constexpr int VBLK_TOTAL = (TK / 4) * CPR;          // 4-key x 8-column blocks per tile
    static constexpr int VBLK = (VBLK_TOTAL + NT - 1) / NT;    // per thread
    static constexpr int K_BYTES = TK * KSTR * 2;
    static constexpr int V_BYTES = D * VSTR * 2;
    static constexpr int O_BYTES = NW * 32 * KSTR * 2;         // epilogue staging, reuses the tile space
    static constexpr int PART_BYTES = (D / 2 + 2) * 64 * 4;    // a wavefront's accumulators, maxima and row sums
    static constexpr int TILE_BYTES = (K_BYTES + V_BYTES) > O_BYTES ? (K_BYTES + V_BYTES) : O_BYTES;
};

template <int D, int NW, int S>
__global__ __launch_bounds__(S * NW * 64, 2) void attn_bf16_kernel(
    const unsigned short *__restrict__ Q, const unsigned short *__restrict__ K, const unsigned short *__restrict__ V,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int bk_shift, int n_sel, int n_qb, int H, float scale_log2,
    unsigned short *__restrict__ O, float *__restrict__ lse) {
    typedef AttnCfg<D, NW> Cfg;
    constexpr int NT = Cfg::NT, KSTR = Cfg::KSTR, VSTR = Cfg::VSTR, CPR = Cfg::CPR;
    static_assert((S - 1) * NW * Cfg::PART_BYTES <= S * Cfg::TILE_BYTES, "the groups' sums reuse the tile space");
    __shared__ __attribute__((aligned(16))) unsigned char tile_mem[S * Cfg::TILE_BYTES];
    __shared__ TileMeta meta_all[S][3];
    const int grp = S == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NT);   // wave-uniform
    TileMeta *meta = meta_all[grp];
    unsigned short *Ks = (unsigned short *)(tile_mem + grp * Cfg::TILE_BYTES);
    unsigned short *Vt = (unsigned short *)(tile_mem + grp * Cfg::TILE_BYTES + Cfg::K_BYTES);

    // workgroup -> (head, query block).  Workgroups are dealt round-robin to the 8 XCDs; give each
    // XCD a contiguous range of (head, block) pairs so that the K/V of a head stay in one L2.
    int h, b;
    {
        const int total = n_qb * H;
        const int wg = blockIdx.x;
        const int per = (total + 7) / 8;      // the grid holds 8 * per workgroups
        const int item = (wg & 7) * per + (wg >> 3);
        if (item >= total) return;            // padding of the last XCD's range (uniform)
        h = item / n_qb;
        b = item % n_qb;
    }
    const int tid = threadIdx.x - grp * NT, lane = tid & 63, wave = tid >> 6;   // of the group
    const int col = lane & 31, g = lane >> 5;
    const int L = min(len[h], C);
    const int n_listed = min(nsel[(size_t)h * n_qb + b], n_sel);
    const int32_t *sel_row = sel + ((size_t)h * n_qb + b) * n_sel;
    const int32_t *cnt_h = cnt ? cnt + (size_t)h * C : nullptr;
    const unsigned short *Kh = K + (size_t)h * C * D;
    const unsigned short *Vh = V + (size_t)h * C * D;
    const int nt = ((n_listed << bk_shift) + TK - 1) / TK;
    const int steps = (nt + S - 1) / S;   // the same for every group: a tile past the list is all masked rows

    // Q fragments of this wavefront's 32 queries (B operand: column = query, k-slots = 8 coordinates)
    const int q_idx = b * (NW * 32) + wave * 32 + col;
    bf16x8 qf[D / 16];
    {
        const unsigned short *qrow = Q + ((size_t)h * n_q + min(q_idx, n_q - 1)) * D;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) qf[s] = *(const bf16x8 *)(qrow + 16 * s + 8 * g);
    }

    f32x16 o_acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o_acc[db][v] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;

    u32x4 kst[Cfg::KCH];
    u32x4 vst[Cfg::VBLK][4];
    auto issue_loads = [&](const TileMeta &m) {
#pragma unroll
        for (int c = 0; c < Cfg::KCH; ++c) {
            const int ch = tid + c * NT;
            const int row = ch / CPR, cc = ch % CPR;
            const int key = m.idx[row];
            u32x4 z = {0, 0, 0, 0};
            kst[c] = key >= 0 ? *(const u32x4 *)(Kh + (size_t)key * D + cc * 8) : z;
        }
#pragma unroll
        for (int vb = 0; vb < Cfg::VBLK; ++vb) {
            const int blk = tid + vb * NT;
            const int a = blk / CPR, cc = blk % CPR;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                u32x4 z = {0, 0, 0, 0};
                int key = -1;
                if (blk < Cfg::VBLK_TOTAL) key = m.idx[4 * a + rr];
                vst[vb][rr] = key >= 0 ? *(const u32x4 *)(Vh + (size_t)key * D + cc * 8) : z;
            }
        }
    };
    auto store_tiles = [&]() {
#pragma unroll
        for (int c = 0; c < Cfg::KCH; ++c) {
            const int ch = tid + c * NT;
            const int row = ch / CPR, cc = ch % CPR;
            *(u32x4 *)(Ks + row * KSTR + cc * 8) = kst[c];
        }
#pragma unroll
        for (int vb = 0; vb < Cfg::VBLK; ++vb) {
            const int blk = tid + vb * NT;
            if (blk < Cfg::VBLK_TOTAL) {
                const int a = blk / CPR, cc = blk % CPR;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned w0 = vst[vb][0][q], w1 = vst[vb][1][q], w2 = vst[vb][2][q], w3 = vst[vb][3][q];
                    u32x2 even = {(w0 & 0xFFFFu) | (w1 << 16), (w2 & 0xFFFFu) | (w3 << 16)};
                    u32x2 odd = {(w0 >> 16) | (w1 & 0xFFFF0000u), (w2 >> 16) | (w3 & 0xFFFF0000u)};
                    *(u32x2 *)(Vt + (cc * 8 + 2 * q) * VSTR + 4 * a) = even;
                    *(u32x2 *)(Vt + (cc * 8 + 2 * q + 1) * VSTR + 4 * a) = odd;
                }
            }
        }
    };

    auto fill = [&](int t) { fill_meta(meta[t % 3], t * S + grp, sel_row, n_listed, bk_shift, L, cnt_h, tid); };
    if (steps > 0) {
        fill(0);
        if (steps > 1) fill(1);
        __syncthreads();
        issue_loads(meta[0]);
    }
    for (int t = 0; t < steps; ++t) {
        __syncthreads();  // tile t-1 fully consumed; row table of tile t+1 visible
        store_tiles();
        __syncthreads();
        if (t + 1 < steps) issue_loads(meta[(t + 1) % 3]);
        if (t + 2 < steps) fill(t + 2);
        if (S > 1 && t * S + grp >= nt) break;   // uniform for the wavefront; only in the last step, no barrier is left in the loop
        const TileMeta &mt = meta[t % 3];

        // S^T = K Q^T : two blocks of 32 keys x 32 queries
        f32x16 s_acc[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s_acc[kb][v] = 0.0f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                const bf16x8 a = *(const bf16x8 *)(Ks + (32 * kb + col) * KSTR + 16 * s + 8 * g);
                s_acc[kb] = mfma_bf16_32x32x16(a, qf[s], s_acc[kb]);
            }
        }
        // logits in the log2 domain, masked keys at -inf
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 bv = *(const f32x4 *)(&mt.bias[32 * kb + 8 * q4 + 4 * g]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float sv = fmaf(s_acc[kb][4 * q4 + e], scale_log2, bv[e]);
                    s_acc[kb][4 * q4 + e] = sv;
                    mx = fmaxf(mx, sv);
                }
            }
        mx = fmaxf(mx, shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        float psum = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = __builtin_amdgcn_exp2f(s_acc[kb][v] - m_safe);
                s_acc[kb][v] = p;
                psum += p;
            }
        l_run = l_run * alpha + psum;
        m_run = m_new;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o_acc[db][v] *= alpha;

        // O^T += V^T P^T : four steps of 16 keys
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                bf16x8 pf;
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[e] = (__bf16)s_acc[kb][8 * half + e];
                const int kbase = 32 * kb + 16 * half;
#pragma unroll
                for (int db = 0; db < D / 32; ++db) {
                    const unsigned short *vp = Vt + (32 * db + col) * VSTR + kbase + 4 * g;
                    const u32x2 lo = *(const u32x2 *)vp;
                    const u32x2 hi = *(const u32x2 *)(vp + 8);
                    u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
                    bf16x8 a;
                    __builtin_memcpy(&a, &w, 16);
                    o_acc[db] = mfma_bf16_32x32x16(a, pf, o_acc[db]);
                }
            }
    }

    __syncthreads();
    if constexpr (S > 1) {
        // the other groups' accumulators, maxima and sums, lane by lane
        if (grp > 0) {
            float *part = (float *)(tile_mem + ((grp - 1) * NW + wave) * Cfg::PART_BYTES) + lane;
#pragma unroll
            for (int i = 0; i < D / 2; ++i) part[i * 64] = o_acc[i / 16][i % 16];
            part[(D / 2) * 64] = m_run;
            part[(D / 2 + 1) * 64] = l_run;
        }
        __syncthreads();
        if (grp == 0) {
#pragma unroll
            for (int o = 1; o < S; ++o) {
                const float *part = (const float *)(tile_mem + ((o - 1) * NW + wave) * Cfg::PART_BYTES) + lane;
                const float m_o = part[(D / 2) * 64];
                const float m_new = fmaxf(m_run, m_o), m_safe = m_new == -INFINITY ? 0.0f : m_new;
                const float a0 = __builtin_amdgcn_exp2f(m_run - m_safe), a1 = __builtin_amdgcn_exp2f(m_o - m_safe);
#pragma unroll
                for (int i = 0; i < D / 2; ++i) o_acc[i / 16][i % 16] = fmaf(o_acc[i / 16][i % 16], a0, part[i * 64] * a1);
                l_run = fmaf(l_run, a0, part[(D / 2 + 1) * 64] * a1);
                m_run = m_new;
            }
        }
        __syncthreads();
        if (grp > 0) return;   // whole wavefronts; the last barrier orders a wavefront's own rows only
    }
    // epilogue: normalise, transpose through LDS (each wavefront its own rows), store rows coalesced
    const float l_tot = l_run + shfl_xor(l_run, 32);
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    unsigned short *Os = (unsigned short *)tile_mem + (size_t)wave * 32 * KSTR;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            u32x2 w = {pack_bf16x2(o_acc[db][4 * q4] * inv, o_acc[db][4 * q4 + 1] * inv),
                       pack_bf16x2(o_acc[db][4 * q4 + 2] * inv, o_acc[db][4 * q4 + 3] * inv)};
            *(u32x2 *)(Os + col * KSTR + 32 * db + 8 * q4 + 4 * g) = w;
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    {
        constexpr int LPR = CPR;          // lanes per row (16-byte chunks)
        constexpr int RPI = 64 / LPR;     // rows per iteration
        const int rr = lane / LPR, cc = lane % LPR;
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int r = it * RPI + rr;
            const int qi = b * (NW * 32) + wave * 32 + r;
            if (qi < n_q) *(u32x4 *)(O + ((size_t)h * n_q + qi) * D + cc * 8) = *(const u32x4 *)(Os + r * KSTR + cc * 8);
        }
    }
    if (lse && g == 0 && q_idx < n_q)
        lse[(size_t)h * n_q + q_idx] = l_tot > 0.0f ? (m_run + __log2f(l_tot)) * LN2 : -INFINITY;
}

int launch_attn_f32(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len, int H, int C,
                    int d, const int32_t *sel, const int32_t *nsel, int BQ, int BK, int n_sel, float scale_log2, void *O,
                    float *lse, hipStream_t s);
int launch_attn_bf16_d128(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len,
                          int H, int C, const int32_t *sel, const int32_t *nsel, int BQ, int bk_shift, int n_sel,
                          float scale_log2, void *O, float *lse, hipStream_t s);
int launch_attn_bf16_d128_pp(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt,
                             const int32_t *len, int H, int C, const int32_t *sel, const int32_t *nsel, int bk_shift,
                             int n_sel, float scale_log2, void *O, float *lse, int n_parts, void *ws, hipStream_t s);

size_t attn_sk_ws_bytes();
int launch_attn_bf16_d128_sk(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len,
                             int H, int C, const int32_t *sel, const int32_t *nsel, int bk_shift, int n_sel,
                             float scale_log2, void *O, float *lse, void *ws, int full_per, hipStream_t s);

}  // namespace fastar

using namespace fastar;

static int sparse_attn_impl(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt,
                            const int32_t *len, int H, int C, int d, int dtype, const int32_t *sel,
                            const int32_t *nsel, int BQ, int BK, int n_sel, float scale, void *O, float *lse,
                            void *ws, size_t ws_bytes, void *stream);

extern "C" int sparse_attn_fwd(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt,
                               const int32_t *len, int H, int C, int d, int dtype, const int32_t *sel,
                               const int32_t *nsel, int BQ, int BK, int n_sel, float scale, void *O, float *lse,
                               void *stream) {
    return sparse_attn_impl(Q, n_q, K, V, cnt, len, H, C, d, dtype, sel, nsel, BQ, BK, n_sel, scale, O, lse, nullptr, 0,
                            stream);
}

extern "C" int sparse_attn_fwd_ws(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt,
                                  const int32_t *len, int H, int C, int d, int dtype, const int32_t *sel,
                                  const int32_t *nsel, int BQ, int BK, int n_sel, float scale, void *O, float *lse,
                                  void *ws, size_t ws_bytes, void *stream) {
    if (!ws || ((uintptr_t)ws & 255)) return FASTAR_ERR_INVALID_ARG;
    if (ws_bytes < attn_sk_ws_bytes()) return FASTAR_ERR_WORKSPACE;
    return sparse_attn_impl(Q, n_q, K, V, cnt, len, H, C, d, dtype, sel, nsel, BQ, BK, n_sel, scale, O, lse, ws, ws_bytes,
                            stream);
}

static int sparse_attn_impl(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt,
                               const int32_t *len, int H, int C, int d, int dtype, const int32_t *sel,
                               const int32_t *nsel, int BQ, int BK, int n_sel, float scale, void *O, float *lse,
                               void *ws, size_t ws_bytes, void *stream) {
    (void)ws_bytes;
    if (!Q || !K || !V || !len || !sel || !nsel || !O) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || C <= 0 || BQ <= 0 || BK <= 0 || n_sel <= 0) return FASTAR_ERR_INVALID_ARG;
    if (dtype != FASTAR_F32 && dtype != FASTAR_BF16) return FASTAR_ERR_INVALID_ARG;
    if (!(scale > 0.0f) || !(scale < INFINITY)) return FASTAR_ERR_INVALID_ARG;
    if (((uintptr_t)Q & 15) || ((uintptr_t)K & 15) || ((uintptr_t)V & 15) || ((uintptr_t)O & 15))
        return FASTAR_ERR_INVALID_ARG;
    if (d != 64 && d != 128) return FASTAR_ERR_UNSUPPORTED;
    const int n_qb = (n_q + BQ - 1) / BQ;
    hipStream_t s = (hipStream_t)stream;
    const float scale_log2 = scale * LOG2E;
    if (dtype == FASTAR_BF16) {
        if ((BQ != 64 && BQ != 128) || BK > 64 || (BK & (BK - 1)) != 0) return FASTAR_ERR_UNSUPPORTED;
        if ((unsigned long long)C * (unsigned long long)d * 2ull >= (1ull << 32)) return FASTAR_ERR_UNSUPPORTED;  // 32-bit row offsets
        int bk_shift = 0;
        while ((1 << bk_shift) < BK) ++bk_shift;
        const dim3 grid((unsigned)(((n_qb * H + 7) / 8) * 8));
#define FASTAR_ATTN(DD, NW, S)                                                                                     \
    hipLaunchKernelGGL((attn_bf16_kernel<DD, NW, S>), grid, dim3(S * NW * 64), 0, s, (const unsigned short *)Q,          \
                       (const unsigned short *)K, (const unsigned short *)V, cnt, len, sel, nsel, n_q, C, bk_shift, \
                       n_sel, n_qb, H, scale_log2, (unsigned short *)O, lse)
        // Two query blocks per workgroup in anti-phase (matrix | vector) on each SIMD; one workgroup fills a CU, so the
        // work comes in rounds of 512 query blocks: when the last round would be less than half full, the kernel with
        // one block per workgroup (two workgroups per CU, started as slots free up) finishes earlier.
        const int n_items = n_qb * H;
        // With a workspace, and more query blocks than the chip holds at once in a number that leaves a short last
        // round (an XCD holds 64 workgroups of the one-block kernel; a round that only a few of them take part in lasts
        // half as long as a full one, with most of the chip idle): the one-block kernel on whole rounds, then the query
        // blocks left over cut into equal shares of their tiles for all resident workgroups (long enough shares to pay for
        // the fragments and their combination).
        const int n_tiles = (int)(((long long)n_sel * BK + 63) / 64);
        const int full_per = attn_split_full_per(n_items, n_tiles);
        if (ws && d == 128 && BQ == 128 && full_per > 0)
            return launch_attn_bf16_d128_sk(Q, n_q, K, V, cnt, len, H, C, sel, nsel, bk_shift, n_sel, scale_log2, O, lse, ws,
                                            full_per, s);
        // At most one query block per compute unit: both groups of the two-block kernel on one block (156 blocks of 48 tiles
        // 85 -> 51 us, one-block workgroups take 67), with a workspace several workgroups per block where that pays
        // (8 blocks of 96 tiles 161 -> 21 us).  Very short lists stay with the one-block kernel (3 tiles: 8.5 us against 9.5,
        // 6 tiles 12.2 against 12.1), also beyond 256 blocks (444 blocks of 64 single keys 9.9 us against 11.2).
        if (d == 128 && BQ == 128 && n_items <= 256 && n_tiles > 5)
            return launch_attn_bf16_d128_pp(Q, n_q, K, V, cnt, len, H, C, sel, nsel, bk_shift, n_sel, scale_log2, O, lse,
                                            ws ? attn_parts(n_items, n_tiles, 2, 1.65f, 0.0f) : 1, ws, s);
        if (d == 128 && BQ == 128 && n_items <= 512 && n_tiles <= 5 && (n_items <= 256 || n_tiles <= 2))
            return launch_attn_bf16_d128(Q, n_q, K, V, cnt, len, H, C, sel, nsel, BQ, bk_shift, n_sel, scale_log2, O, lse, s);
        if (d == 128 && BQ == 128 && (n_items <= 512 || n_items % 512 == 0 || n_items % 512 >= 256))
            return launch_attn_bf16_d128_pp(Q, n_q, K, V, cnt, len, H, C, sel, nsel, bk_shift, n_sel, scale_log2, O, lse, 0,
                                            nullptr, s);
        if (d == 128)  // tuned path: direct-to-LDS tiles, LDS transpose loads
            return launch_attn_bf16_d128(Q, n_q, K, V, cnt, len, H, C, sel, nsel, BQ, bk_shift, n_sel, scale_log2, O, lse, s);
        // d = 64.  At most one query block per compute unit: its tiles over several groups of wavefronts (256 blocks of 64
        // queries x 11 tiles 22.1 -> 14.7 us, 40 tiles 70 -> 36; of 128 queries 21.9 -> 18.6 and 66 -> 49; lists of 2 tiles
        // the same).  With 480 blocks it is already slower (2 tiles 9.7 -> 13.9, 11 tiles of 128 queries 28 -> 34).
        if (n_items <= 256 && n_tiles > 2) {
            if (BQ == 128) FASTAR_ATTN(64, 4, 2);
            else FASTAR_ATTN(64, 2, 4);
        } else {
            if (BQ == 128) FASTAR_ATTN(64, 4, 1);
            else FASTAR_ATTN(64, 2, 1);
        }
#undef FASTAR_ATTN
    } else {
        if (BQ > 128 || BK > 64) return FASTAR_ERR_UNSUPPORTED;
        return launch_attn_f32(Q, n_q, K, V, cnt, len, H, C, d, sel, nsel, BQ, BK, n_sel, scale_log2, O, lse, s);
    }
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}
