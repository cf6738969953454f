// Device pieces of the ANN code (Sec. 5.1 of the paper), shared by the encode kernels and by the TempCache
// match kernel that encodes its own probes:
//   xq = clamp(rint(x * qscale), +-127);  y = R^T xq (int32);  c = clamp((y + 2^(sh-1)) >> sh, +-127)
// One wavefront owns 16 vectors at a time: B operand = their quantised coordinates (column = vector), A operand =
// R^T (rows = code coordinates), accumulator row 4*(lane/16)+v / column lane%16, so a lane ends up with 4 entries per
// block of 16 rows of one vector's code.
#pragma once
#include "common.hpp"

namespace fastar {

// Coordinate t that k-slot e (0..15) of quarter g stands for in k-step ks.  Chosen so that each
// 16-byte load of a lane is contiguous and the four quarters of a row tile the row.
template <bool BF16>
__device__ __forceinline__ int slot_coord(int ks, int g, int e) {
    if (BF16) return ks * 64 + (e >> 3) * 32 + 8 * g + (e & 7);
    return ks * 64 + (e >> 2) * 16 + 4 * g + (e & 3);
}

// One lane's coordinates of one vector: raw bits while its loads are in flight, then the 16 int8 k-slots of every k-step.
template <bool BF16, int D>
struct RawVector {
    static constexpr int N = BF16 ? 2 : 4;   // 16-byte loads per k-step
    u32x4 w[D / 64][N];
    __device__ __forceinline__ void load(const void *row, int g) {
#pragma unroll
        for (int ks = 0; ks < D / 64; ++ks)
#pragma unroll
            for (int m = 0; m < N; ++m)
                w[ks][m] = BF16 ? *(const u32x4 *)((const unsigned short *)row + ks * 64 + m * 32 + 8 * g)
                                : *(const u32x4 *)((const float *)row + ks * 64 + m * 16 + 4 * g);
    }
    __device__ __forceinline__ void quantise(float qscale, i32x4 (&out)[D / 64]) const {
#pragma unroll
        for (int ks = 0; ks < D / 64; ++ks)
#pragma unroll
            for (int m = 0; m < N; ++m) {
                const u32x4 x = w[ks][m];
                if (BF16) {
                    out[ks][(2 * m) & 3] = (int)quant8x4(bf16_lo(x[0]), bf16_hi(x[0]), bf16_lo(x[1]), bf16_hi(x[1]), qscale);
                    out[ks][(2 * m + 1) & 3] = (int)quant8x4(bf16_lo(x[2]), bf16_hi(x[2]), bf16_lo(x[3]), bf16_hi(x[3]), qscale);
                } else {
                    out[ks][m] = (int)quant8x4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]),
                                               __uint_as_float(x[3]), qscale);
                }
            }
    }
};
// Quantised coordinates of one vector, loaded at once.
template <bool BF16, int D>
__device__ __forceinline__ void load_quantised(const void *row, int g, float qscale, i32x4 (&out)[D / 64]) {
    RawVector<BF16, D> v;
    v.load(row, g);
    v.quantise(qscale, out);
}

// A operand of one wavefront: rows of R^T for every (k-step of 64 coordinates, block of CB rows).  Row i of block cb is
// code coordinate CB * i + cb: a lane's CB rows are then neighbours in a row of R, which one load of CB bytes brings
// (byte loads, 64 of them per lane at d = 128 and r = 32, were most of what an encode launch issued), and the results of
// a lane's CB blocks interleave to 4 * CB consecutive code coordinates.
template <bool BF16, int D, int R>
struct CodeMatrix {
    static constexpr int KS = D / 64, CB = R / 16;
    static_assert(CB == 2 || CB == 4, "R = 32 or 64");
    i32x4 a[KS][CB];
    __device__ __forceinline__ void load(const int8_t *__restrict__ Rm, int lane) {
        const int col = lane & 15, g = lane >> 4;
        const bool aligned = ((uintptr_t)Rm & (CB - 1)) == 0;   // uniform
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            unsigned w[16];   // CB neighbouring entries of 16 coordinates
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int8_t *p = Rm + slot_coord<BF16>(ks, g, e) * R + CB * col;
                if (aligned) {
                    w[e] = CB == 2 ? (unsigned)*(const unsigned short *)p : *(const unsigned *)p;
                } else {
                    w[e] = 0u;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) w[e] |= (unsigned)(uint8_t)p[cb] << (8 * cb);
                }
            }
            // byte cb of four words into one: pairs of words side by side first, two byte selections per word of the operand
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const unsigned w0 = w[4 * m], w1 = w[4 * m + 1], w2 = w[4 * m + 2], w3 = w[4 * m + 3];
                const unsigned l0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), l1 = __builtin_amdgcn_perm(w3, w2, 0x05010400u);
                a[ks][0][m] = (int)__builtin_amdgcn_perm(l1, l0, 0x05040100u);
                a[ks][1][m] = (int)__builtin_amdgcn_perm(l1, l0, 0x07060302u);
                if constexpr (CB == 4) {
                    const unsigned h0 = __builtin_amdgcn_perm(w1, w0, 0x07030602u), h1 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
                    a[ks][CB - 2][m] = (int)__builtin_amdgcn_perm(h1, h0, 0x05040100u);
                    a[ks][CB - 1][m] = (int)__builtin_amdgcn_perm(h1, h0, 0x07060302u);
                }
            }
        }
    }
    // Entries 4 * CB * (lane / 16) .. of the code of the vector whose quantised coordinates are b (column lane % 16),
    // saturated to +-lim; f(i, c) takes entry i of them.
    template <class F>
    __device__ __forceinline__ void entries(const i32x4 (&b)[KS], int shift, int lim, F &&f) const {
        i32x4 acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            acc[cb] = i32x4{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc[cb] = mfma_i8_16x16x64(a[ks][cb], b[ks], acc[cb]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                f(CB * v + cb, min(max((acc[cb][v] + (1 << (shift - 1))) >> shift, -lim), lim));   // floor division
    }
    // The same as bytes: 4 * CB consecutive ones.
    struct Words {
        unsigned w[CB];
    };
    __device__ __forceinline__ Words code_words(const i32x4 (&b)[KS], int shift) const {
        int c[4 * CB];
        entries(b, shift, 127, [&](int i, int v) { c[i] = v; });
        Words out;
#pragma unroll
        for (int k = 0; k < CB; ++k) out.w[k] = pack_i8x4(c[4 * k], c[4 * k + 1], c[4 * k + 2], c[4 * k + 3]);
        return out;
    }
    // ... stored as this lane's part of a row of R bytes (16-byte aligned rows unless WORDS: 4-byte aligned ones)
    template <bool WORDS = false>
    __device__ static __forceinline__ void store(int8_t *row, const Words &x, int lane) {
        unsigned *dst = (unsigned *)(row + 4 * CB * (lane >> 4));
        if (WORDS) {
#pragma unroll
            for (int k = 0; k < CB; ++k) dst[k] = x.w[k];
        } else if (CB == 2) {
            *(u32x2 *)dst = u32x2{x.w[0], x.w[1]};
        } else {
            *(u32x4 *)dst = u32x4{x.w[0], x.w[1], x.w[2 & (CB - 1)], x.w[3 & (CB - 1)]};
        }
    }
    // The same entries at BITS (2 or 4) bits each, saturated to +-(2^(BITS-1) - 1), entry i in bits [BITS*i, +BITS).
    template <int BITS>
    __device__ __forceinline__ unsigned code_bits(const i32x4 (&b)[KS], int shift) const {
        static_assert(4 * CB * BITS <= 32, "one word");
        unsigned w = 0;
        entries(b, shift, (1 << (BITS - 1)) - 1, [&](int i, int v) { w |= ((unsigned)v & ((1u << BITS) - 1u)) << (BITS * i); });
        return w;
    }
};

}  // namespace fastar
