// Block-sparse attention in fp32 (sparse_attn_fwd with FASTAR_F32): fp32 products, sums, softmax and outputs, on the
// fp32 matrix instructions.
//
// v_mfma_f32_16x16x4_f32 multiplies and adds in fp32 like a chain of fma, at twice the rate of the vector ALU, and needs
// no operand broadcast: a wavefront owns 16 queries and walks tiles of 32 listed keys, with both contractions transposed
// so that everything that belongs to a query stays in its lane (lane l: query l % 16):
//     S^T = K Q^T    A = K rows straight from global memory (lane l: key l % 16, coordinates 16 c + 4 (l / 16) .. + 3),
//                    B = Q in registers; accumulator register v of lane l is key 4 (l / 16) + v
//     O^T = V^T P^T  B = the S^T registers as they are (k slot l / 16 of step v is key 4 (l / 16) + v),
//                    A = V rows straight from global memory: which output column a row of A stands for is free, so block db
//                    of D / 16 takes columns (D / 16) (l % 16) + db and a lane's elements of one V row are consecutive
// No tile is shared inside a workgroup, so there is no LDS staging and no barrier in the loop; K of the next tile is in
// flight under the second product and V under the first.
//
// What bounds it: a wavefront's chain of tiles (128 matrix instructions of 32 cycles per 32 keys at d = 128) while the launch
// leaves compute units empty, the K and V rows every group fetches through L2 (8 flop per byte) where it fills the chip.
// Hence 16 queries per wavefront, not 32, and KS = 4 wavefronts of a workgroup per query group: they take every fourth
// tile and combine their partial sums through LDS.  Measured, d = 128, 15 key blocks of 64 per query block, us with 8 / 4 /
// 2 / 1 wavefronts per group: 196 groups 35 / 32 / 52 / 97, 512 groups 72 / 64 / 59 / 104, 1076 groups 161 / 132 / 149 / 196,
// 3516 groups (77 TFLOP/s) 455 / 357 / 359 / 385; one query per thread on the vector ALU took 1700 for the 196 groups.
#include "common.hpp"

namespace fastar {

namespace f32a {

constexpr int QW = 16;    // queries per wavefront
constexpr int TKF = 32;   // listed keys per step
constexpr float LN2 = 0.6931471805599453f;

__device__ __forceinline__ f32x4 mfma_f32_16x16x4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// What masked positions (padding, rows past len, the end of the list) fetch: a row of the cache that nothing selects need not
// be finite, and inf + -inf or 0 * inf would reach the output.  Offsets instead of row numbers in the table, so that the
// choice costs nothing per load: 33 us at 196 groups x 15 key blocks against 32 with masked positions on row 0 (a branch that
// clears their operands instead: 35).
__device__ float zero_row[128];

constexpr int KS = 4;     // wavefronts of a workgroup: they share one query group and split its tiles

template <int D>
__global__ __launch_bounds__(KS * 64, 2) void attn_f32_kernel(
    const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V, const int32_t *__restrict__ cnt,
    const int32_t *__restrict__ len, const int32_t *__restrict__ sel, const int32_t *__restrict__ nsel, int n_q, int C,
    int BQ, int BK, int n_sel, int n_qb, int groups_per_block, int n_groups, float scale_log2, float *__restrict__ O,
    float *__restrict__ lse) {
    constexpr int CH = D / 16;   // 16-coordinate chunks of a row, and V columns per lane
    __shared__ __attribute__((aligned(16))) long long tvrows[KS][TKF];
    __shared__ __attribute__((aligned(16))) float tbiases[KS][TKF];
    __shared__ float po[KS][4 * CH][64];       // partial O^T, as it sits in the registers
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
    float m_run = -INFINITY, l_run = 0.0f;   // of this lane's query; l_run over this lane's keys only

    // this wavefront's row table: V row and bias of the 32 positions of a tile (rows as byte offsets from the head's own)
    long long *tvrow = tvrows[ks];
    float *tbias = tbiases[ks];
    struct Position {
        long long k, v;
        float bias;
    };
    const Position masked = {(const char *)zero_row - (const char *)Kh, (const char *)zero_row - (const char *)Vh, -INFINITY};
    auto lookup = [&](int t) {   // position lane % 32 of tile t
        Position pos = masked;
        const int p = t * TKF + (lane & 31);
        if (p < n_pos) {
            const int e = p / BK;
            const int kb = sel_row[e];
            const int k = kb * BK + (p - e * BK);
            if (kb >= 0 && k < L) {
                pos.k = pos.v = (long long)k * (D * 4);
                pos.bias = cnt_h ? log2f((float)cnt_h[k]) : 0.0f;
            }
        }
        return pos;
    };
    f32x4 kf[2][CH];
    auto load_k = [&](long long krow) {   // the key of this lane's row of either half tile: lanes 0..31 hold positions 0..31
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const float *kp = (const float *)((const char *)(Kh + 4 * quarter) + __shfl(krow, 16 * hh + qc, WAVE));
#pragma unroll
            for (int c = 0; c < CH; ++c) kf[hh][c] = *(const f32x4 *)(kp + 16 * c);
        }
    };
    Position next = masked;
    if (ks < nt) {
        next = lookup(ks);
        load_k(next.k);
    }
    for (int t = ks; t < nt; t += KS) {
        if (lane < TKF) {
            tvrow[lane] = next.v;
            tbias[lane] = next.bias;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // V rows of this lane's keys 16 hh + 4 quarter + v
        float vf[2][4][CH];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float *vp = (const float *)((const char *)(Vh + CH * qc) + tvrow[16 * hh + 4 * quarter + v]);
#pragma unroll
                for (int c = 0; c < CH; c += 4) {
                    const f32x4 w = *(const f32x4 *)(vp + c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) vf[hh][v][c + e] = w[e];
                }
            }
        }
        if (t + KS < nt) next = lookup(t + KS);
        f32x4 s[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) s[hh] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) s[hh] = mfma_f32_16x16x4(kf[hh][c][e], q[c][e], s[hh]);
        if (t + KS < nt) load_k(next.k);
        float mx = -INFINITY;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const f32x4 bv = *(const f32x4 *)(tbias + 16 * hh + 4 * quarter);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[hh][v] = fmaf(s[hh][v], scale_log2, bv[v]);
                mx = fmaxf(mx, s[hh][v]);
            }
        }
        mx = fmaxf(mx, shfl_xor(mx, 16));
        mx = fmaxf(mx, shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = m_new == -INFINITY ? 0.0f : m_new;   // every key so far masked
        const float alpha = exp2f(m_run - m_safe);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[hh][v] = exp2f(s[hh][v] - m_safe);
                l_run += s[hh][v];
            }
#pragma unroll
        for (int c = 0; c < CH; ++c) o[c] *= alpha;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int c = 0; c < CH; ++c) o[c] = mfma_f32_16x16x4(vf[hh][v][c], s[hh][v], o[c]);
    }
    float l_tot = l_run + shfl_xor(l_run, 16);
    l_tot += shfl_xor(l_tot, 32);

    // The partial sums meet in LDS; each wavefront finishes its share of the columns.  o[c][v]: column
    // CH * (4 quarter + v) + c of query qc.
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < CH; ++c) po[ks][v * CH + c][lane] = o[c][v];
    if (quarter == 0) {
        pm[ks][qc] = m_run;
        pl[ks][qc] = l_tot;
    }
    __syncthreads();
    float m_all = -INFINITY;
#pragma unroll
    for (int k = 0; k < KS; ++k) m_all = fmaxf(m_all, pm[k][qc]);
    float wgt[KS], l_all = 0.0f;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        wgt[k] = m_all == -INFINITY ? 0.0f : exp2f(pm[k][qc] - m_all);
        l_all += wgt[k] * pl[k][qc];
    }
    if (qc >= nq_here) return;
    const float inv = l_all > 0.0f ? 1.0f / l_all : 0.0f;
    float *orow = O + ((size_t)h * n_q + q0 + qc) * D + CH * (4 * quarter + ks);   // register v = ks is this wavefront's share
#pragma unroll
    for (int c = 0; c < CH; c += 4) {
        f32x4 r = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < KS; ++k) r[e] += wgt[k] * po[k][ks * CH + c + e][lane];
        *(f32x4 *)(orow + c) = r * inv;
    }
    if (lse && quarter == 0 && ks == 0)
        lse[(size_t)h * n_q + q0 + qc] = l_all > 0.0f ? (m_all + log2f(l_all)) * LN2 : -INFINITY;
}

}  // namespace f32a

int launch_attn_f32(const void *Q, int n_q, const void *K, const void *V, const int32_t *cnt, const int32_t *len, int H, int C,
                    int d, const int32_t *sel, const int32_t *nsel, int BQ, int BK, int n_sel, float scale_log2, void *O,
                    float *lse, hipStream_t s) {
    using namespace f32a;
    const int n_qb = (n_q + BQ - 1) / BQ, gpb = (BQ + QW - 1) / QW;
    const long long n_groups = (long long)H * n_qb * gpb;
    if (n_groups >= (1ll << 30)) return FASTAR_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)((n_groups + 7) / 8 * 8));
    hipLaunchKernelGGL(d == 128 ? attn_f32_kernel<128> : attn_f32_kernel<64>, grid, dim3(KS * 64), 0, s, (const float *)Q,
                       (const float *)K, (const float *)V, cnt, len, sel, nsel, n_q, C, BQ, BK, n_sel, n_qb, gpb, (int)n_groups,
                       scale_log2, (float *)O, lse);
    if (hipGetLastError() != hipSuccess) return FASTAR_ERR_HIP;
    return FASTAR_OK;
}

}  // namespace fastar
