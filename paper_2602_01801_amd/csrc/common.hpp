// Shared device helpers of libfastar (gfx950 only): vector types, MFMA wrappers, bf16 handling,
// the 8-bit quantiser and wave-level primitives.  Wavefronts are 64 lanes wide throughout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "../../include/fastar.h"

namespace fastar {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int WAVE = 64;

// ---- MFMA ---------------------------------------------------------------------------------------
// 32x32 tiles: lane l supplies row (A) / column (B) l%32 and the k-slots of half g = l/32; the
// accumulator register v of lane l is element (row 8*(v/4) + 4*g + v%4, column l%32).
// 16x16 tiles: lane l supplies row / column l%16 and the k-slots of quarter l/16; accumulator
// register v is element (row 4*(l/16) + v, column l%16).
// Which k a slot stands for is free as long as A and B agree, so operands are loaded with whatever
// k order suits the memory layout.

__device__ __forceinline__ f32x16 mfma_bf16_32x32x16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ i32x16 mfma_i8_32x32x32(i32x4 a, i32x4 b, i32x16 c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ i32x4 mfma_i8_16x16x64(i32x4 a, i32x4 b, i32x4 c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// ---- bf16 ---------------------------------------------------------------------------------------

__device__ __forceinline__ float bf16_bits_to_f32(unsigned short b) { return __uint_as_float(((unsigned)b) << 16); }
__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// float -> bfloat16 bits, nearest with ties to even (inputs are finite here).
__device__ __forceinline__ unsigned f32_to_bf16_bits(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
    return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

// The same by the conversion instruction: one for the pair.
__device__ __forceinline__ unsigned cvt_bf16x2(float lo, float hi) {
    const bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(unsigned, v);
}
// Transposing LDS read: in each group of 16 lanes, lane 4q + m receives element m of the 8-byte pieces that the lanes q,
// q + 4, q + 8 and q + 12 address.
__device__ __forceinline__ bf16x4 ds_read_tr16(const void *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)p);
}

// ---- quantiser of the ANN code ----------------------------------------------------------------------
// One float32 multiply, round half to even, saturate to [-127, 127]; four values as packed bytes.  The saturation comes
// first (its bounds are whole numbers, so the order does not matter; a NaN becomes -127); the rounding is the addition of
// 1.5 * 2^23, after which the low byte of the float's bits is the rounded value: three instructions per value and three
// byte selections per word, where round, two-sided clamp, conversion and packing took seven per value.
__device__ __forceinline__ unsigned quant8x4(float x0, float x1, float x2, float x3, float qscale) {
    const float x[4] = {x0, x1, x2, x3};
    unsigned u[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        u[e] = __float_as_uint(__fadd_rn(__builtin_amdgcn_fmed3f(__fmul_rn(x[e], qscale), -127.0f, 127.0f), 12582912.0f));
    return __builtin_amdgcn_perm(u[1], u[0], 0x0C0C0400u) | __builtin_amdgcn_perm(u[3], u[2], 0x04000C0Cu);
}
__device__ __forceinline__ unsigned pack_i8x4(int a, int b, int c, int d) {
    return (unsigned)(a & 0xFF) | ((unsigned)(b & 0xFF) << 8) | ((unsigned)(c & 0xFF) << 16) | ((unsigned)(d & 0xFF) << 24);
}

// ---- wave primitives ------------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return threadIdx.x & (WAVE - 1); }

template <typename T>
__device__ __forceinline__ T shfl_xor(T v, int mask) {
    return __shfl_xor(v, mask, WAVE);
}

__device__ __forceinline__ int dot4_i8(unsigned a, unsigned b, int acc) {
    return __builtin_amdgcn_sdot4((int)a, (int)b, acc, false);
}

// Inclusive prefix over a wavefront's lanes, on the vector ALU (six shuffles by way of the LDS queue took 0.3 us).
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8: prefix of 16 lanes
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast 15: rows 1 and 3 add the row below
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast 31: the upper half adds the lower
    return v;
}
// The word of lane ^ 1, lane ^ 2 (STEP 0, 1) or of the mirror lane of the other four of eight (STEP 2): three steps combine eight
// neighbouring lanes on the vector ALU.
template <int STEP>
__device__ __forceinline__ unsigned lane_of_eight(unsigned v) {
    constexpr int CTRL = STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : 0x141;   // quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
// Maximum over a wavefront's lanes, in its last lane.
__device__ __forceinline__ unsigned wave_max_last(unsigned v) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));
    return v;
}

// Group records of the live slots (tempcache_compress), for workgroups of the encode launch to clear; win = nullptr: none.
struct ClearRecords {
    unsigned long long *win;
    int32_t *grp;
    const int32_t *len;
    int H, C;
};

// One-time set-up per device (kernel attributes, symbol addresses), safe to reach from several host threads: run(f)
// calls f once per device ordinal, with that device current, and remembers a success.  It is the only process-wide data
// the library keeps, and it never influences a result.
struct DeviceOnce {
    static constexpr int MAX_DEVICES = 64;
    std::atomic<unsigned long long> done{0};
    std::mutex mu;
    template <class F>
    int run(F &&f) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return FASTAR_ERR_HIP;
        if (dev < 0 || dev >= MAX_DEVICES) return FASTAR_ERR_UNSUPPORTED;
        const unsigned long long bit = 1ull << dev;
        if (done.load(std::memory_order_acquire) & bit) return FASTAR_OK;
        std::lock_guard<std::mutex> lock(mu);
        if (done.load(std::memory_order_relaxed) & bit) return FASTAR_OK;
        const int rc = f(dev);
        if (rc == FASTAR_OK) done.fetch_or(bit, std::memory_order_release);
        return rc;
    }
};

// ---- split attention launches (sparse_attn_fwd_ws, sparse_attn_fwd_fp8_ws) ---------------------------------------
// The (head, query block) pairs are dealt to the 8 XCDs in contiguous ranges of `per`; the first `full_per` pairs of every
// range are taken by one workgroup each, the others are cut into equal shares of their tiles (attention_d128.hip).
constexpr int ATTN_SHARE_WORKGROUPS = 512;   // the most workgroups that take the shares: as many as are resident, two per CU
struct TailMap {
    int per, full_per, total;   // pairs per XCD range, of them taken whole, pairs in all
    __host__ __device__ __forceinline__ int tail_per() const { return per - full_per; }
    __host__ __device__ __forceinline__ long long tiles(int NT) const { return (long long)8 * tail_per() * NT; }
    // workgroups that share them: a tile each at least, as a share without one leaves no fragment (a multiple of 8 either way)
    int shares(int NT) const { return (int)(tiles(NT) < ATTN_SHARE_WORKGROUPS ? tiles(NT) : ATTN_SHARE_WORKGROUPS); }
    // position in the left-over sequence -> (head, block) pair; pairs >= total do not exist (the last range may be short)
    __host__ __device__ __forceinline__ int item(int vi) const { return (vi / tail_per()) * per + full_per + vi % tail_per(); }
};
// Least scale * log2(e) of the kernels that divide by it: 31 / scale (the largest multiplicity's bias) plus a score stays
// far from the largest float.  Subnormal scales gave 0 * infinity.
constexpr float ATTN_LEAST_SCALE_LOG2 = 0x1p-100f;
constexpr int ATTN_PART_O_FLOATS = (128 / 32) * 16 * 64;        // O^T accumulators of one wavefront (d = 128)
constexpr int ATTN_PART_FLOATS = 4 * (ATTN_PART_O_FLOATS + 2 * 64);   // one fragment of a query block: four wavefronts' accumulators, reference maxima, row sums
// Whether a launch of n_items pairs with n_tiles 64-key tiles each is split, and how many pairs per range are taken
// whole then (0: not split).  What the split saves: a last round of n_tiles tiles at a lone workgroup's pace (about 1.2 us
// per tile) against tail_per / 64 of a round at the pace of a full chip (2.4 us per tile) plus about 30 us of fragments and
// launches (an XCD holds 64 workgroups of the one-block kernels).
inline int attn_split_full_per(int n_items, int n_tiles) {
    const int per_xcd = (n_items + 7) / 8, tail_per = per_xcd % 64;
    if (per_xcd > 64 && tail_per > 0 && tail_per <= 24 && (float)n_tiles * (1.2f - 0.0375f * (float)tail_per) > 30.0f)
        return per_xcd - tail_per;
    return 0;
}
// Few query blocks (at most one per compute unit): into how many runs of tiles each is cut, a workgroup (and a fragment)
// each.  one_us / two_us: time of a workgroup per step of tiles_per_step tiles with one / two of them on a compute unit
// (two_us = 0: only one fits).  One run costs its steps and about 4 us; several cost the longest run's steps and, measured
// with 1 .. 224 blocks of 3 .. 192 tiles, 8 us + 0.25 us per run + 0.03 us per workgroup for the fragments, which are
// written, read back and combined by one more launch.  At most 512 fragments: half of the workspace.
inline int attn_parts(int n_items, int n_tiles, int tiles_per_step, float one_us, float two_us) {
    int best = 1;
    float best_us = 1e30f;
    for (int p = 1; p <= 32 && p * n_items <= (two_us > 0.0f ? 512 : 256) && (p == 1 || p * tiles_per_step <= n_tiles); ++p) {
        const int steps = (n_tiles + p * tiles_per_step - 1) / (p * tiles_per_step);
        const float us = (p * n_items <= 256 ? one_us : two_us) * (float)steps +
                         (p == 1 ? 4.0f : 8.0f + 0.25f * (float)p + 0.03f * (float)(p * n_items));
        if (us < best_us) {
            best_us = us;
            best = p;
        }
    }
    return best;
}
// Kernels of bf16 attention (fastar_probe_attn_route returns these numbers).
enum AttnKernel {
    ATTN_PLAIN,        // attention.hip: a block per workgroup, tiles staged by way of registers
    ATTN_WAVES,        // attention_waves.hip: groups of 32 queries whose wavefronts share the tiles
    ATTN_ONE,          // attention_d128.hip: a block per workgroup
    ATTN_ONE_SHARED,   // ... the last round's blocks cut into equal shares
    ATTN_PAIR,         // attention_d128_pp.hip: two blocks per workgroup
    ATTN_PAIR_SPLIT,   // ... one block for both halves of a workgroup, or for several workgroups
};
int launch_attn_combine_parts(const void *ws, int n_parts, int n_q, int n_qb, int H, float scale_log2, float lse_offset, void *O,
                              float *lse, hipStream_t s);
int launch_attn_combine(const void *ws, int n_q, int n_qb, TailMap tm, int NT, float scale_log2, float lse_offset, void *O,
                        float *lse, hipStream_t s);

// Per-file set-up, all of it run by fastar_init() (api.hip) and each lazily by the first launch that needs it.
int attn_d128_pp_setup();
int attn_d128_setup();
int select_setup();
int tempcache_setup();
int attn_fp8_setup();

// Host-side launch check shared by the entry points.
#define FASTAR_LAUNCH_CHECK()                          \
    do {                                               \
        if (hipGetLastError() != hipSuccess) return FASTAR_ERR_HIP; \
    } while (0)

}  // namespace fastar
