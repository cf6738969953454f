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
// This kernel serves 64-wide heads (and scales too small to divide by); few query blocks: attention_waves.hip, 128-wide heads:
// attention_d128.hip and attention_d128_pp.hip, fp32: attention_f32.hip.  Which call takes which: attn_route below.
#include <algorithm>

#include "common.hpp"

namespace fastar {

constexpr int TK = 64;  // keys per tile
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

struct __attribute__((aligned(16))) TileMeta {
    int idx[TK];     // cache row of each tile position, -1 = masked
    float bias[TK];  // log2(cnt) of that row, -inf when masked
};

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
    static constexpr int TILE_BYTES = (K_BYTES + V_BYTES) > O_BYTES ? (K_BYTES + V_BYTES) : O_BYTES;
};

template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_bf16_kernel(
    const unsigned short *__restrict__ Q, const unsigned short *__restrict__ K, const unsigned short *__restrict__ V,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ len, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ nsel, int n_q, int C, int bk_shift, int n_sel, int n_qb, int H, float scale_log2,
    unsigned short *__restrict__ O, float *__restrict__ lse) {
    typedef AttnCfg<D, NW> Cfg;
    constexpr int NT = Cfg::NT, KSTR = Cfg::KSTR, VSTR = Cfg::VSTR, CPR = Cfg::CPR;
    __shared__ __attribute__((aligned(16))) unsigned char tile_mem[Cfg::TILE_BYTES];
    __shared__ TileMeta meta[3];
    unsigned short *Ks = (unsigned short *)tile_mem;
    unsigned short *Vt = (unsigned short *)(tile_mem + Cfg::K_BYTES);

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
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, g = lane >> 5;
    const int L = min(len[h], C);
    const int n_listed = min(nsel[(size_t)h * n_qb + b], n_sel);
    const int32_t *sel_row = sel + ((size_t)h * n_qb + b) * n_sel;
    const int32_t *cnt_h = cnt ? cnt + (size_t)h * C : nullptr;
    const unsigned short *Kh = K + (size_t)h * C * D;
    const unsigned short *Vh = V + (size_t)h * C * D;
    const int nt = ((n_listed << bk_shift) + TK - 1) / TK;

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

    // The row table of a tile is filled by the first wavefront, a lane per position, in three stages (list entry, multiplicity,
    // table), of which a step does one for each of three tiles: nothing is waited for in the step that asks for it, nor behind
    // that step's tile loads.  1160 blocks of 128 queries x 90 tiles 430 -> 394 us, 512 x 64 131 -> 122.
    const bool filler = __builtin_amdgcn_readfirstlane(wave) == 0;
    auto entry = [&](int t) { return sel_row[max(min((t * TK + lane) >> bk_shift, n_listed - 1), 0)]; };
    auto resolve = [&](int t, int kb) {   // the position's row, -1: masked
        const int listpos = t * TK + lane;
        const int key = (kb << bk_shift) + (listpos & ((1 << bk_shift) - 1));
        return (listpos >> bk_shift) < n_listed && kb >= 0 && key < L ? key : -1;
    };
    auto multiplicity = [&](int key) { return cnt_h ? cnt_h[max(key, 0)] : 1; };
    auto fill = [&](int t, int key, int n) {
        meta[t % 3].idx[lane] = key;
        meta[t % 3].bias[lane] = key < 0 ? -INFINITY : cnt_h ? __log2f((float)n) : 0.0f;
    };
    int key2 = -1, n2 = 1, kb3 = -1;
    if (nt > 0) {
        if (filler) {
            const int kb0 = entry(0);
            int kb1 = -1, kb2 = -1, key1 = -1, n1 = 1;
            if (nt > 1) {   // uniform; a single tile's chain is all there is to such a launch
                kb1 = entry(1);
                kb2 = entry(2);
                kb3 = entry(3);
            }
            const int key0 = resolve(0, kb0), n0 = multiplicity(key0);
            if (nt > 1) {
                key1 = resolve(1, kb1);
                key2 = resolve(2, kb2);
                n1 = multiplicity(key1);
                n2 = multiplicity(key2);
            }
            fill(0, key0, n0);
            if (nt > 1) fill(1, key1, n1);
        }
        __syncthreads();
        issue_loads(meta[0]);
    }
    for (int t = 0; t < nt; ++t) {
        __syncthreads();  // tile t-1 fully consumed; row table of tile t+1 visible
        store_tiles();
        __syncthreads();
        if (filler && t + 2 < nt) {
            fill(t + 2, key2, n2);
            key2 = resolve(t + 3, kb3);
            n2 = multiplicity(key2);
            kb3 = entry(t + 4);
        }
        if (t + 1 < nt) issue_loads(meta[(t + 1) % 3]);
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

int launch_attn_bf16_waves(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len, int H, int C,
                           int d, const int32_t *sel, const int32_t *nsel, int BQ, int bk_shift, int n_sel, float scale_log2, int S,
                           void *O, float *lse, hipStream_t s);

size_t attn_sk_ws_bytes();
int launch_attn_bf16_d128_sk(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len,
                             int H, int C, const int32_t *sel, const int32_t *nsel, int bk_shift, int n_sel,
                             float scale_log2, void *O, float *lse, void *ws, int full_per, hipStream_t s);

}  // namespace fastar

using namespace fastar;

// Whether a launch of n_items query blocks takes the kernel whose wavefronts share a group of 32 queries, and then their number
// per group (0: the other kernels).  Time of this kernel over that of the others by query blocks and list entries of 64 keys, the
// two in turn, lists a tenth of the cache (differences of 0.02 are noise); us where they say more.
//   d = 64, BQ = 64     4 to 256 blocks 0.95 (1 entry) to 0.2 (128); 700 x 2 1.02, x 3 0.97, x 16 0.73; 1024 x 3 1.01, x 64 0.77; 1100 x 3 1.03,
//                       x 5 0.97; 1300 x 4 1.03, x 5 1.00, x 8 0.95; 1500 x 6 1.02, x 8 1.00, x 16 0.97 (the others' one round is full);
//                       1540 to 2040 x 3 0.89 to 0.93, x 64 0.67 to 0.75; 2060 to 4000 x 3 0.95 to 0.99, x 4 0.93 to 0.98, x 64 0.78 to 0.92,
//                       x 128 0.88 to 1.02; 6000 x 4 0.99, x 64 0.98, x 128 1.09
//   d = 64, BQ = 128    4 to 128 blocks 0.98 (1) to 0.2; 160 x 1 1.07, x 2 0.99; 240 x 2 1.05, x 3 1.00, x 64 0.67; 320 x 3 0.95; 328 to 448 x 8
//                       0.97 to 1.01, x 16 0.86 to 0.97, x 128 0.75 to 0.87; 512 x 16 1.00, x 32 0.96; 640 to 760 x 16 1.02 to 1.16
//   d = 128, BQ = 64    4 to 128 blocks 0.89 (2) to 0.4; 160 to 256 x 2 1.16, x 4 1.06, x 6 0.98 to 1.01, x 8 0.90 to 0.94, x 128 0.74; 288 to 384
//                       x 2 1.00, x 3 0.97, x 32 0.81, x 128 0.84 to 0.89, x 300 1.00; 448 x 2 1.12, x 8 1.01, x 32 0.97, x 200 1.18
//   d = 128, BQ = 128   2 to 64 blocks 0.82 (2) to 0.5 (1000); 68 to 128 x 2 1.09, x 4 1.00 to 1.03, x 6 0.95, x 20 0.97 to 0.99, x 32 0.99 to
//                       1.00; 96 x 400 358 -> 384 us, 128 x 1000 868 -> 1005 (every group fetches its rows for itself, here from HBM)
//     with a workspace, where the others leave fragments, the last entry count that is no slower: 12 blocks 22, 16 24, 20 28, 28 32,
//     40 32, 48 36, 64 40; 72 x 20 25.1 against 26.5 us, x 24 28.7 against 24.8.  Below 12 blocks the change comes between 16 and 20
//     (4 x 16 12.8 against 13.6, x 20 14.9 against 14.4); their lists of 9 entries and more keep the fragments they had.
// Where a call with a workspace leaves no fragments, one without takes the same kernel.
static int waves_per_group(int d, int BQ, int BK, int n_items, int n_sel, bool ws) {
    const long long groups = (long long)n_items * (BQ / 32), tiles = ((long long)n_sel * BK + 31) / 32;
    if (d == 64) {
        if (BQ == 64) {
            const int least = groups <= 640 ? 1 : groups <= 2048 ? 5 : groups <= 2600 ? 10 : groups <= 3072 ? 16 : groups <= 4096 ? 5 : 8;
            if (groups > 8192 || tiles < least || (groups > 4096 && tiles > 128)) return 0;
        } else {
            const int least = groups <= 512 ? 1 : groups <= 640 ? 3 : groups <= 1280 ? 5 : 32;
            if (groups > 1792 || tiles < least) return 0;
            if (groups > 1280) return 4;
        }
        if (tiles <= 2) return 2;
        if (groups > 512) return tiles >= 64 ? 4 : 2;
        return tiles >= (groups <= 256 ? 24 : 64) ? 8 : 4;
    }
    if (BK != 64 || tiles < 4) return 0;   // rows by way of a table, and single tiles: no gain
    if (BQ == 64) {
        if (groups > 512) return groups <= 768 && tiles >= 6 ? 2 : 0;
        if (groups > 256) return tiles >= 16 ? 4 : 0;
        return tiles >= 48 ? 8 : 4;
    }
    if (groups > 512) return 0;
    const bool many = n_items > 64, fragments = ws && attn_parts(n_items, (int)((tiles + 1) / 2), 2, 1.65f, 0.0f) > 1;
    if (many && (tiles < 12 || tiles > (fragments ? 40 : 64))) return 0;
    if (!many && fragments && tiles > (n_items < 12 ? 16 : std::min(64, 28 + n_items))) return 0;
    return groups <= 256 && tiles >= 48 ? 8 : 4;
}

// Which kernel a bf16 call of n_items (head, query block) pairs takes.  `n`: wavefronts per group of queries (ATTN_WAVES), pairs
// per XCD that are taken whole (ATTN_ONE_SHARED), runs of tiles per query block (ATTN_PAIR_SPLIT).
struct AttnRoute {
    int kernel, n;
};
static AttnRoute attn_route(int d, int BQ, int BK, int n_items, int n_sel, float scale_log2, bool ws) {
    // The other kernels start a tile's sums from log2(cnt) / scale, and let a reference maximum lag by octaves / scale; this
    // one adds the bias behind the scaling, so that no scale is too small for it.
    if (scale_log2 < ATTN_LEAST_SCALE_LOG2) return {ATTN_PLAIN, 0};
    // With a workspace, and more query blocks than the chip holds at once in a number that leaves a short last
    // round (an XCD holds 64 workgroups of the one-block kernel; a round that only a few of them take part in lasts
    // half as long as a full one, with most of the chip idle): the one-block kernel on whole rounds, then the query
    // blocks left over cut into equal shares of their tiles for all resident workgroups (long enough shares to pay for
    // the fragments and their combination).
    const int n_tiles = (int)(((long long)n_sel * BK + 63) / 64);
    const int full_per = attn_split_full_per(n_items, n_tiles);
    if (ws && d == 128 && BQ == 128 && full_per > 0) return {ATTN_ONE_SHARED, full_per};
    if (const int S = waves_per_group(d, BQ, BK, n_items, n_sel, ws)) return {ATTN_WAVES, S};
    // At most one query block per compute unit: both groups of the two-block kernel on one block (156 blocks of 48 tiles
    // 85 -> 51 us, one-block workgroups take 67), with a workspace several workgroups per block where that pays
    // (8 blocks of 96 tiles 161 -> 21 us).  Very short lists stay with the one-block kernel (3 tiles: 8.5 us against 9.5,
    // 6 tiles 12.2 against 12.1), also beyond 256 blocks (444 blocks of 64 single keys 9.9 us against 11.2).
    if (d == 128 && BQ == 128 && n_items <= 256 && n_tiles > 5)
        return {ATTN_PAIR_SPLIT, ws ? attn_parts(n_items, n_tiles, 2, 1.65f, 0.0f) : 1};
    if (d == 128 && BQ == 128 && n_items <= 512 && n_tiles <= 5 && (n_items <= 256 || n_tiles <= 2)) return {ATTN_ONE, 0};
    // Two query blocks per workgroup in anti-phase (matrix | vector) on each SIMD; one workgroup fills a CU, so the
    // work comes in rounds of 512 query blocks: when the last round would be less than half full, the kernel with
    // one block per workgroup (two workgroups per CU, started as slots free up) finishes earlier.
    if (d == 128 && BQ == 128 && (n_items <= 512 || n_items % 512 == 0 || n_items % 512 >= 256)) return {ATTN_PAIR, 0};
    return {d == 128 ? ATTN_ONE : ATTN_PLAIN, 0};
}

extern "C" int fastar_probe_attn_route(int n_items, int d, int BQ, int BK, int n_sel, int with_workspace, int *n) {
    if (n_items <= 0 || n_sel <= 0 || !n) return FASTAR_ERR_INVALID_ARG;
    if ((d != 64 && d != 128) || (BQ != 64 && BQ != 128) || BK <= 0 || BK > 64 || (BK & (BK - 1))) return FASTAR_ERR_UNSUPPORTED;
    const AttnRoute r = attn_route(d, BQ, BK, n_items, n_sel, 1.0f, with_workspace != 0);
    *n = r.n;
    return r.kernel;
}

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
#define FASTAR_ATTN(DD, NW)                                                                                        \
    hipLaunchKernelGGL((attn_bf16_kernel<DD, NW>), grid, dim3(NW * 64), 0, s, (const unsigned short *)Q,                 \
                       (const unsigned short *)K, (const unsigned short *)V, cnt, len, sel, nsel, n_q, C, bk_shift, \
                       n_sel, n_qb, H, scale_log2, (unsigned short *)O, lse)
        const AttnRoute route = attn_route(d, BQ, BK, n_qb * H, n_sel, scale_log2, ws != nullptr);
        switch (route.kernel) {
            case ATTN_ONE_SHARED:
                return launch_attn_bf16_d128_sk(Q, n_q, K, V, cnt, len, H, C, sel, nsel, bk_shift, n_sel, scale_log2, O, lse, ws,
                                                route.n, s);
            case ATTN_WAVES:
                return launch_attn_bf16_waves(Q, n_q, K, V, cnt, len, H, C, d, sel, nsel, BQ, bk_shift, n_sel, scale_log2, route.n,
                                              O, lse, s);
            case ATTN_PAIR_SPLIT:
                return launch_attn_bf16_d128_pp(Q, n_q, K, V, cnt, len, H, C, sel, nsel, bk_shift, n_sel, scale_log2, O, lse,
                                                route.n, ws, s);
            case ATTN_PAIR:
                return launch_attn_bf16_d128_pp(Q, n_q, K, V, cnt, len, H, C, sel, nsel, bk_shift, n_sel, scale_log2, O, lse, 0,
                                                nullptr, s);
            case ATTN_ONE:   // direct-to-LDS tiles, LDS transpose loads
                return launch_attn_bf16_d128(Q, n_q, K, V, cnt, len, H, C, sel, nsel, BQ, bk_shift, n_sel, scale_log2, O, lse, s);
        }
        if (d == 128 && BQ == 128) FASTAR_ATTN(128, 4);
        else if (d == 128) FASTAR_ATTN(128, 2);
        else if (BQ == 128) FASTAR_ATTN(64, 4);
        else FASTAR_ATTN(64, 2);
#undef FASTAR_ATTN
    } else {
        if (BQ > 128 || BK > 64) return FASTAR_ERR_UNSUPPORTED;
        return launch_attn_f32(Q, n_q, K, V, cnt, len, H, C, d, sel, nsel, BQ, BK, n_sel, scale_log2, O, lse, s);
    }
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}
