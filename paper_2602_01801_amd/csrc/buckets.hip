// Prompt-induced buckets for self-attention (Sec. 5.4, first paragraph: AnnSA reuses the semantic buckets that
// cross-attention pruning found; a query belongs to one or more buckets and attends only to keys of the same bucket(s)).
//
// The prompt tokens are the buckets.  Four small kernels, all on exact integers:
//   prompt_bucket_kernel   the m nearest prompt tokens of every code (the products AnnCA ranks prompt tokens by, on
//                          the int8 matrix cores; one packed 32-bit key per product keeps "largest product, then
//                          smallest token" under a plain unsigned comparison)
//   bucket_mask_kernel     one bit per prompt token: the buckets a query block / key block owns, stored word-major so
//                          that the scoring reads them coalesced
//   bucket_score_kernel    shared buckets of every (query block, key block) pair: AND + bit count
//   bucket_topk_kernel     candidates (at least one shared bucket, or forced) counted, then the exact top-k of select.hip
#include <algorithm>

#include "common.hpp"
#include "topk_dev.hpp"

namespace fastar {

constexpr int BUCKET_MAX_PROMPT = 2048;   // 11 bits of a packed key hold the token id
constexpr int BUCKET_MAX = 8;             // buckets of a code
constexpr int MASK_BLOCKS_PER_WG = 8;
constexpr int SCORE_QB = 8;               // query blocks a thread of the scoring kernel counts for
constexpr int SCORE_THREADS = 128;

// ---- nearest prompt tokens ---------------------------------------------------------------------------------------
// D = A x B with A rows = 32 prompt tokens, B columns = 32 codes: a lane ends with 16 products of ONE code (column
// lane % 32) with prompt tokens pb*32 + 8(v/4) + 4(lane/32) + v%4.
// key = (product + 2^20) * 2^11 + (2047 - token): |product| <= 64 * 127^2 < 2^20, token < 2^11; keys differ and are not 0.
// A lane keeps its M largest keys in order (a minimum and a maximum per place); the two lane halves and, split, the four
// wavefronts then merge theirs.
// Bound by the vector instructions per product (2 + 2M - 1) and, with few codes, by how few wavefronts there are: a frame's
// 12 x 1560 codes in wavefronts of 32 that each walk the whole prompt are 588 chains on 1024 SIMDs.  So with a prompt of at
// least four blocks the wavefronts of a workgroup split the prompt (block p to wavefront p % 4) and share 32 codes; below,
// each takes 32 codes of its own, or there would be idle ones.
// 12 x 1560 codes, 512 prompt tokens, two buckets: 11.5 us with a pass over the products per bucket and 128 codes per
// workgroup, 5.5 us; 12 x 4680 codes: 13.7 and 8.5 us.
template <int M>
__device__ __forceinline__ void insert_key(unsigned (&top)[M], unsigned x) {
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const unsigned lo = min(top[k], x);
        top[k] = max(top[k], x);
        x = lo;
    }
}

template <int R, int M>
__global__ __launch_bounds__(256) void prompt_bucket_kernel(const int8_t *__restrict__ code, int C,
                                                            const int32_t *__restrict__ idx, int n,
                                                            const int8_t *__restrict__ pcode, int n_p, int m, int split,
                                                            int32_t *__restrict__ bucket) {
    constexpr int KS = R / 32;
    __shared__ unsigned part[3][M][32];   // keys of wavefronts 1 .. 3 (split)
    const int h = blockIdx.y;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    const int li = (split ? blockIdx.x : blockIdx.x * 4 + wave) * 32 + col;
    int slot = -1;
    if (li < n) slot = idx ? idx[(size_t)h * n + li] : li;
    if (slot >= C) slot = -1;
    const int8_t *crow = code + ((size_t)h * C + max(slot, 0)) * R;
    i32x4 bfrag[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) bfrag[ks] = *(const i32x4 *)(crow + ks * 32 + 16 * g);
    const int8_t *ph = pcode + (size_t)h * n_p * R;
    const int n_pb = (n_p + 31) / 32;
    const int pb0 = split ? wave : 0, step = split ? 4 : 1;

    unsigned top[M];
#pragma unroll
    for (int k = 0; k < M; ++k) top[k] = 0u;
    for (int pb = pb0; pb < n_pb; pb += 4 * step) {
        // four blocks of prompt tokens per step: their rows are loaded together, then multiplied
        i32x4 afrag[4][KS];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int prow = min((pb + u * step) * 32 + col, n_p - 1);   // rows past the end: any row, masked below
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) afrag[u][ks] = *(const i32x4 *)(ph + (size_t)prow * R + ks * 32 + 16 * g);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int blk = pb + u * step;
            if (blk < n_pb) {   // wave-uniform
                i32x16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = mfma_i8_32x32x32(afrag[u][ks], bfrag[ks], acc);
                const unsigned first = 0x80000000u + 2047u - 32u * (unsigned)blk - 4u * (unsigned)g;
                const int rows_left = n_p - 32 * blk - 4 * g;   // < 32 in a ragged last block only
                if (n_p - 32 * blk >= 32) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        insert_key<M>(top, ((unsigned)acc[v] << 11) + (first - (unsigned)(8 * (v / 4) + v % 4)));
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = 8 * (v / 4) + v % 4;
                        insert_key<M>(top, row < rows_left ? ((unsigned)acc[v] << 11) + (first - (unsigned)row) : 0u);
                    }
                }
            }
        }
    }
    unsigned other[M];
#pragma unroll
    for (int k = 0; k < M; ++k) other[k] = (unsigned)__shfl_xor((int)top[k], 32, WAVE);
#pragma unroll
    for (int k = 0; k < M; ++k) insert_key<M>(top, other[k]);
    if (split) {   // uniform
        if (wave > 0 && g == 0) {
#pragma unroll
            for (int k = 0; k < M; ++k) part[wave - 1][k][col] = top[k];
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int k = 0; k < M; ++k) insert_key<M>(top, part[w][k][col]);
    }
    if (g == 0 && slot >= 0) {
        int32_t *dst = bucket + ((size_t)h * C + slot) * m;
#pragma unroll
        for (int k = 0; k < M; ++k)
            if (k < m) dst[k] = top[k] ? 2047 - (int)(top[k] & 2047u) : -1;   // none left: fewer prompt tokens than m
    }
}

// ---- bucket masks of blocks ----------------------------------------------------------------------------------------
// mask[w][blk] bit t%32 of word w = t/32: some live row of block blk (BS consecutive rows of `bucket`) owns prompt
// token t.  Both sides in one launch: workgroups below q_groups take query blocks, the others key blocks.
// Bound by the latency of load -> LDS atomic chains: a wavefront has two blocks (64 per workgroup left a launch over 37
// query blocks on 12 compute units), four loads of one block in flight.
// 12 x (37 blocks of 128 queries + 585 of 64 keys), two buckets each: 16 + 19 us in two launches, 5.3 us in one.
struct MaskSide {
    const int32_t *bucket;
    const int32_t *len;   // null: all N rows
    int N, BS, n_blocks;
    unsigned *mask;
};
__global__ __launch_bounds__(256) void bucket_mask_kernel(MaskSide q, MaskSide k, int q_groups, int m, int n_p, int W) {
    extern __shared__ unsigned words[];   // [MASK_BLOCKS_PER_WG][W + 1]
    const bool is_q = (int)blockIdx.x < q_groups;
    const MaskSide s = is_q ? q : k;
    const int h = blockIdx.y;
    const int blk0 = ((int)blockIdx.x - (is_q ? 0 : q_groups)) * MASK_BLOCKS_PER_WG;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int L = s.len ? min(s.len[h], s.N) : s.N;
    const int WP = W + 1;
    for (int t = threadIdx.x; t < MASK_BLOCKS_PER_WG * WP; t += 256) words[t] = 0;
    __syncthreads();
    for (int e = wave; e < MASK_BLOCKS_PER_WG; e += 4) {
        const long long row0 = (long long)(blk0 + e) * s.BS;
        const int rows = (int)max(0ll, min((long long)s.BS, (long long)L - row0));
        const int32_t *src = s.bucket + ((size_t)h * s.N + (size_t)row0) * m;
        const long long n = (long long)rows * m;
        for (long long t = lane; t < n; t += 4 * WAVE) {
            int tok[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) tok[i] = t + i * WAVE < n ? src[t + i * WAVE] : -1;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (tok[i] >= 0 && tok[i] < n_p) atomicOr(&words[e * WP + (tok[i] >> 5)], 1u << (tok[i] & 31));
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < MASK_BLOCKS_PER_WG * W; t += 256) {
        const int w = t / MASK_BLOCKS_PER_WG, e = t % MASK_BLOCKS_PER_WG;
        if (blk0 + e < s.n_blocks) s.mask[((size_t)h * W + w) * s.n_blocks + blk0 + e] = words[e * WP + w];
    }
}

// ---- shared buckets of (query block, key block) pairs ---------------------------------------------------------------
// score[h][b][kb] = number of prompt tokens owned by both.  A thread owns a key block and eight query blocks, whose words
// lie next to each other in LDS (two 16-byte reads, the same address for every lane, per word of the masks).
// A workgroup per 128 key blocks and 8 query blocks: with all query blocks in one, 12 heads x 585 key blocks were 36
// workgroups on 256 compute units.
// 12 x 37 x 585 pairs, 16 words: 12.6 us, now 4.7.
__global__ __launch_bounds__(SCORE_THREADS) void bucket_score_kernel(const unsigned *__restrict__ qmask,
                                                                     const unsigned *__restrict__ kmask, int W, int n_qb,
                                                                     int n_kb_cap, int32_t *__restrict__ score) {
    extern __shared__ __attribute__((aligned(16))) unsigned own[];   // [W][SCORE_QB], zero padded
    const int h = blockIdx.y, b0 = blockIdx.z * SCORE_QB;
    for (int t = threadIdx.x; t < SCORE_QB * W; t += SCORE_THREADS) {
        const int w = t / SCORE_QB, b = b0 + t % SCORE_QB;
        own[t] = b < n_qb ? qmask[((size_t)h * W + w) * n_qb + b] : 0u;
    }
    __syncthreads();
    const int kb = blockIdx.x * SCORE_THREADS + threadIdx.x;
    if (kb >= n_kb_cap) return;
    const unsigned *km = kmask + (size_t)h * W * n_kb_cap + kb;
    int acc[SCORE_QB];
#pragma unroll
    for (int e = 0; e < SCORE_QB; ++e) acc[e] = 0;
#pragma unroll 4
    for (int w = 0; w < W; ++w) {
        const unsigned mw = km[(size_t)w * n_kb_cap];
        const u32x4 lo = *(const u32x4 *)(own + w * SCORE_QB), hi = *(const u32x4 *)(own + w * SCORE_QB + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[e] += __popc(mw & lo[e]);
            acc[4 + e] += __popc(mw & hi[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < SCORE_QB; ++e)
        if (b0 + e < n_qb) score[((size_t)h * n_qb + b0 + e) * n_kb_cap + kb] = acc[e];
}

// ---- candidates, then the exact top-k -------------------------------------------------------------------------------
// ALONE: rows of up to TOPK_WAVE_MAX entries, a wavefront each; otherwise four.
template <bool ALONE>
__global__ __launch_bounds__(ALONE ? 64 : 256) void bucket_topk_kernel(const int32_t *__restrict__ score, int n_kb_cap,
                                                          const int32_t *__restrict__ len, int C, int BK, int n_qb,
                                                          int n_sel, int n_sink, int n_local, int32_t *__restrict__ sel,
                                                          int32_t *__restrict__ nsel) {
    extern __shared__ unsigned keys[];   // four wavefronts: min(n_kb_cap, TOPK_LDS_CAP) words, staging of the row's keys
    const int b = blockIdx.x, h = blockIdx.y;
    const int n = min((min(len[h], C) + BK - 1) / BK, n_kb_cap);
    const int32_t *row = score + ((size_t)h * n_qb + b) * n_kb_cap;
    int32_t *out = sel + ((size_t)h * n_qb + b) * n_sel, *n_out = nsel + (size_t)h * n_qb + b;
    __shared__ __attribute__((aligned(16))) unsigned scratch[ALONE ? TOPK_WAVE_BINS : TOPK_SCRATCH];
    if constexpr (ALONE) topk_row_wave<TOPK_WAVE_MAX>(row, n, n_sel, out, n_out, scratch, n_sink, n_local, 1);
    else topk_row(row, n, n_sel, out, n_out, keys, scratch, n_sink, n_local, 1);
}

struct BucketWs {
    size_t qmask_off, kmask_off, score_off, total;
};
static inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }
static BucketWs bucket_ws(int H, int n_q, int C, int n_p, int BQ, int BK) {
    const size_t W = (size_t)(n_p + 31) / 32;
    const size_t n_qb = (size_t)(n_q + BQ - 1) / BQ, n_kb = (size_t)(C + BK - 1) / BK;
    BucketWs w;
    w.qmask_off = 0;
    w.kmask_off = al256((size_t)H * W * n_qb * 4);
    w.score_off = w.kmask_off + al256((size_t)H * W * n_kb * 4);
    w.total = w.score_off + al256((size_t)H * n_qb * n_kb * 4);
    return w;
}
size_t select_buckets_ws_bytes(int H, int n_q, int C, int n_p, int BQ, int BK) {
    if (H <= 0 || n_q <= 0 || C <= 0 || n_p <= 0 || BQ <= 0 || BK <= 0) return 0;
    return bucket_ws(H, n_q, C, n_p, BQ, BK).total;
}

}  // namespace fastar

using namespace fastar;

extern "C" int ann_prompt_buckets(const int8_t *code, int C, const int32_t *idx, int n, const int8_t *pcode, int n_p,
                                  int H, int r, int m, int32_t *bucket, void *stream) {
    if (!code || !pcode || !bucket) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || C <= 0 || n < 0 || n_p <= 0 || m <= 0) return FASTAR_ERR_INVALID_ARG;
    if (!idx && n > C) return FASTAR_ERR_INVALID_ARG;
    if (((uintptr_t)code & 15) || ((uintptr_t)pcode & 15)) return FASTAR_ERR_INVALID_ARG;
    if ((r != 32 && r != 64) || n_p > BUCKET_MAX_PROMPT || m > BUCKET_MAX) return FASTAR_ERR_UNSUPPORTED;
    if (n == 0) return FASTAR_OK;
    const int split = n_p > 96;   // at least four blocks of 32 prompt tokens
    const dim3 grid((unsigned)(split ? (n + 31) / 32 : (n + 127) / 128), (unsigned)H);
#define FASTAR_BUCKETS(R, M)                                                                                              \
    hipLaunchKernelGGL((prompt_bucket_kernel<R, M>), grid, dim3(256), 0, (hipStream_t)stream, code, C, idx, n, pcode, n_p, m, \
                       split, bucket)
#define FASTAR_BUCKETS_M(R)                     \
    do {                                        \
        if (m == 1) FASTAR_BUCKETS(R, 1);       \
        else if (m == 2) FASTAR_BUCKETS(R, 2);  \
        else if (m <= 4) FASTAR_BUCKETS(R, 4);  \
        else FASTAR_BUCKETS(R, BUCKET_MAX);     \
    } while (0)
    if (r == 32) FASTAR_BUCKETS_M(32);
    else FASTAR_BUCKETS_M(64);
#undef FASTAR_BUCKETS_M
#undef FASTAR_BUCKETS
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

extern "C" int ann_select_buckets(const int32_t *qbucket, int n_q, const int32_t *kbucket, const int32_t *len, int H,
                                  int C, int m, int n_p, int BQ, int BK, int n_sel, int n_sink, int n_local,
                                  int32_t *sel, int32_t *nsel, void *ws, size_t ws_bytes, void *stream) {
    if (!qbucket || !kbucket || !len || !sel || !nsel || !ws) return FASTAR_ERR_INVALID_ARG;
    if (H <= 0 || n_q <= 0 || C <= 0 || m <= 0 || n_p <= 0 || BQ <= 0 || BK <= 0 || n_sel <= 0)
        return FASTAR_ERR_INVALID_ARG;
    if (n_sink < 0 || n_local < 0 || n_sink + n_local > n_sel || ((uintptr_t)ws & 255)) return FASTAR_ERR_INVALID_ARG;
    if (n_p > BUCKET_MAX_PROMPT) return FASTAR_ERR_UNSUPPORTED;
    const int W = (n_p + 31) / 32;
    const int n_qb = (n_q + BQ - 1) / BQ, n_kb_cap = (C + BK - 1) / BK;
    if ((size_t)((n_qb + 7) & ~7) * W * 4 > 48 * 1024) return FASTAR_ERR_UNSUPPORTED;   // the interface's limit
    const BucketWs w = bucket_ws(H, n_q, C, n_p, BQ, BK);
    if (ws_bytes < w.total) return FASTAR_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    unsigned *qmask = (unsigned *)((char *)ws + w.qmask_off);
    unsigned *kmask = (unsigned *)((char *)ws + w.kmask_off);
    int32_t *score = (int32_t *)((char *)ws + w.score_off);
    const int q_groups = (n_qb + MASK_BLOCKS_PER_WG - 1) / MASK_BLOCKS_PER_WG;
    const int k_groups = (n_kb_cap + MASK_BLOCKS_PER_WG - 1) / MASK_BLOCKS_PER_WG;
    const MaskSide qs = {qbucket, nullptr, n_q, BQ, n_qb, qmask}, ks = {kbucket, len, C, BK, n_kb_cap, kmask};
    hipLaunchKernelGGL(bucket_mask_kernel, dim3(q_groups + k_groups, H), dim3(256), (size_t)MASK_BLOCKS_PER_WG * (W + 1) * 4, s,
                       qs, ks, q_groups, m, n_p, W);
    FASTAR_LAUNCH_CHECK();
    hipLaunchKernelGGL(bucket_score_kernel,
                       dim3((n_kb_cap + SCORE_THREADS - 1) / SCORE_THREADS, H, (n_qb + SCORE_QB - 1) / SCORE_QB),
                       dim3(SCORE_THREADS), (size_t)SCORE_QB * W * 4, s, qmask, kmask, W, n_qb, n_kb_cap, score);
    FASTAR_LAUNCH_CHECK();
    const bool alone = n_kb_cap <= TOPK_WAVE_MAX;
    auto kernel = alone ? bucket_topk_kernel<true> : bucket_topk_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(n_qb, H), dim3(alone ? 64 : 256), alone ? 0 : (size_t)std::min(n_kb_cap, TOPK_LDS_CAP) * 4, s, score,
                       n_kb_cap, len, C, BK, n_qb, n_sel, n_sink, n_local, sel, nsel);
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}
