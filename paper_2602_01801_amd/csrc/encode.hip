// ANN codes (Sec. 5.1 of the paper: shared low-dimensional random projection + 8-bit quantisation).
//
//   xq = clamp(rint(x * qscale), +-127);  y = R^T xq (int32);  c = clamp((y + 2^(sh-1)) >> sh, +-127)
//
// HBM-bound: d*es bytes in, r bytes out per vector; the d x r contraction (2*d*r integer ops per
// vector) runs on the int8 matrix cores so that it stays off the critical path.  One wavefront owns
// 16 vectors at a time: B operand = their quantised coordinates (column = vector), A operand = R^T
// (rows = code coordinates, encode_dev.hpp), so a lane ends up with r / 4 consecutive code bytes of one vector.
#include "encode_dev.hpp"

namespace fastar {

constexpr int CLEAR_RUN = 4096;   // slots per workgroup that clears group records
template <bool BF16, int D, int R, bool CLEAR>
__global__ __launch_bounds__(256) void encode_kernel(const void *__restrict__ x, int64_t n_vec,
                                                     const int8_t *__restrict__ Rm, float qscale, int shift,
                                                     int8_t *__restrict__ code, unsigned long long *zero_fill,
                                                     int64_t zero_n, unsigned enc_blocks, ClearRecords clear) {
    if (CLEAR && blockIdx.x >= enc_blocks) {   // uniform: the records of a run of slots
        const int per_head = (clear.C + CLEAR_RUN - 1) / CLEAR_RUN, at = (int)(blockIdx.x - enc_blocks);
        const int h = at / per_head, j0 = (at - h * per_head) * CLEAR_RUN;
        const int j1 = min(j0 + CLEAR_RUN, min(clear.len[h], clear.C));
        for (int j = j0 + (int)threadIdx.x; j < j1; j += 256) {
            clear.win[(size_t)h * clear.C + j] = 0ull;
            clear.grp[(size_t)h * clear.C + j] = 0;
        }
        return;
    }
    constexpr int KS = D / 64;   // k-steps of 64 coordinates
    const int lane = lane_id();
    const int col = lane & 15, g = lane >> 4;
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t gthreads = (int64_t)(CLEAR ? enc_blocks : gridDim.x) * blockDim.x;
    // optional: clear a 64-bit array for a later kernel of the same call
    for (int64_t i = gtid; i < zero_n; i += gthreads) zero_fill[i] = 0ull;

    // A operand: rows of R^T for every (k-step, code block), gathered once per wavefront
    CodeMatrix<BF16, D, R> cm;
    cm.load(Rm, lane);

    const int64_t wave = gtid >> 6, n_waves = gthreads >> 6;
    const int64_t n_groups = (n_vec + 15) >> 4;
    const size_t row_bytes = (size_t)D * (BF16 ? 2 : 4);
    for (int64_t grp = wave; grp < n_groups; grp += n_waves) {
        const int64_t vec = grp * 16 + col;
        const int64_t vload = vec < n_vec ? vec : n_vec - 1;
        const char *row = (const char *)x + (size_t)vload * row_bytes;
        i32x4 b[KS];
        load_quantised<BF16, D>(row, g, qscale, b);
        const auto w = cm.code_words(b, shift);
        if (vec < n_vec) {
            if (((uintptr_t)code & 15) == 0) cm.store(code + vec * R, w, lane);   // uniform
            else cm.template store<true>(code + vec * R, w, lane);                // the entry point asks for 4-byte alignment
        }
    }
}

template <bool BF16, int D, int R>
static void launch_encode(const void *x, int64_t n_vec, const fastar_codec *codec, int8_t *code,
                          unsigned long long *zero_fill, int64_t zero_n, hipStream_t s, ClearRecords clear) {
    int64_t groups = (n_vec + 15) / 16;
    int64_t blocks = (groups + 3) / 4;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    if (clear.win) {
        const int64_t clearing = (int64_t)clear.H * ((clear.C + CLEAR_RUN - 1) / CLEAR_RUN);
        hipLaunchKernelGGL((encode_kernel<BF16, D, R, true>), dim3((unsigned)(blocks + clearing)), dim3(256), 0, s, x, n_vec,
                           codec->R, codec->qscale, codec->shift, code, zero_fill, zero_n, (unsigned)blocks, clear);
    } else {
        hipLaunchKernelGGL((encode_kernel<BF16, D, R, false>), dim3((unsigned)blocks), dim3(256), 0, s, x, n_vec, codec->R,
                           codec->qscale, codec->shift, code, zero_fill, zero_n, (unsigned)blocks, clear);
    }
}

// Internal launcher shared with tempcache_compress: encodes and optionally zero-fills an array.
int encode_launch(const void *x, int dtype, int64_t n_vec, int d, const fastar_codec *codec, int r, int8_t *code,
                  unsigned long long *zero_fill, int64_t zero_n, hipStream_t s, ClearRecords clear = {}) {
    if (!x || !codec || !codec->R || !code || n_vec < 0) return FASTAR_ERR_INVALID_ARG;
    if (dtype != FASTAR_F32 && dtype != FASTAR_BF16) return FASTAR_ERR_INVALID_ARG;
    if (codec->shift < 1 || codec->shift > 16) return FASTAR_ERR_INVALID_ARG;
    if ((d != 64 && d != 128) || (r != 32 && r != 64)) return FASTAR_ERR_UNSUPPORTED;
    if (((uintptr_t)x & 15) || ((uintptr_t)code & 3)) return FASTAR_ERR_INVALID_ARG;
    if (n_vec == 0 && zero_n == 0) return FASTAR_OK;
#define FASTAR_ENC(B, DD, RR) launch_encode<B, DD, RR>(x, n_vec, codec, code, zero_fill, zero_n, s, clear)
    const bool bf = dtype == FASTAR_BF16;
    if (d == 64 && r == 32) { if (bf) FASTAR_ENC(true, 64, 32); else FASTAR_ENC(false, 64, 32); }
    else if (d == 64 && r == 64) { if (bf) FASTAR_ENC(true, 64, 64); else FASTAR_ENC(false, 64, 64); }
    else if (d == 128 && r == 32) { if (bf) FASTAR_ENC(true, 128, 32); else FASTAR_ENC(false, 128, 32); }
    else { if (bf) FASTAR_ENC(true, 128, 64); else FASTAR_ENC(false, 128, 64); }
#undef FASTAR_ENC
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

// ---- codes of 2 or 4 bits per entry, packed (appendix, "Quantization precision for ANN matching") -------------------
// Same operands as encode_kernel; a lane ends with eight entries of one vector = BITS bytes.
template <bool BF16, int D, int R, int BITS>
__global__ __launch_bounds__(256) void encode_packed_kernel(const void *__restrict__ x, int64_t n_vec,
                                                            const int8_t *__restrict__ Rm, float qscale, int shift,
                                                            uint8_t *__restrict__ packed) {
    static_assert(R == 32, "eight entries per lane");
    constexpr int KS = D / 64;
    constexpr int ROWB = R * BITS / 8;
    const int lane = lane_id();
    const int col = lane & 15, g = lane >> 4;
    CodeMatrix<BF16, D, R> cm;
    cm.load(Rm, lane);
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t wave = gtid >> 6, n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t n_groups = (n_vec + 15) >> 4;
    const size_t row_bytes = (size_t)D * (BF16 ? 2 : 4);
    for (int64_t grp = wave; grp < n_groups; grp += n_waves) {
        const int64_t vec = grp * 16 + col;
        const int64_t vload = vec < n_vec ? vec : n_vec - 1;
        const char *row = (const char *)x + (size_t)vload * row_bytes;
        i32x4 b[KS];
        load_quantised<BF16, D>(row, g, qscale, b);
        const unsigned w = cm.template code_bits<BITS>(b, shift);
        if (vec < n_vec) {
            uint8_t *dst = packed + vec * ROWB + g * BITS;
            if (BITS == 4) *(unsigned *)dst = w;
            else *(unsigned short *)dst = (unsigned short)w;
        }
    }
}

// ---- sign codes (LSH paragraph of Sec. 5.1): bit j = [ (R^T xq)_j >= 0 ] --------------------------------------
// HBM-bound: d*es bytes in, NB/8 out per vector.  Same operand layout as encode_kernel with NB/16 blocks of 16 rows of
// R^T; row i of block cb is hash bit NB/16 * i + cb.  A lane's NB/16 neighbouring entries of a row of R are then one load
// (byte loads, 256 of them per lane at d = 128 and 128 bits for fewer than two groups of vectors, were most of what the
// launch issued), and the signs of its 4 * NB/16 sums are consecutive bits of one vector: one funnel shift each, no lane
// exchange.  Few enough wavefronts that each hashes many groups with its operand, the next group's rows in flight:
// 128 bits of 449280 bf16 vectors of d = 128 (122 MB) 51.6 -> 27 us = 4.5 TB/s, of 56160 vectors 13.1 -> 11.5 us.
template <bool BF16, int D, int NB>
__global__ __launch_bounds__(256) void encode_sign_kernel(const void *__restrict__ x, int64_t n_vec,
                                                          const int8_t *__restrict__ Rm, float qscale,
                                                          uint32_t *__restrict__ bits) {
    constexpr int KS = D / 64;
    constexpr int CB = NB / 16;      // 4, 8 or 16
    const int lane = lane_id();
    const int col = lane & 15, g = lane >> 4;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6, n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t n_groups = (n_vec + 15) >> 4;
    const size_t row_bytes = (size_t)D * (BF16 ? 2 : 4);
    if (wave >= n_groups) return;
    RawVector<BF16, D> raw;
    auto load = [&](int64_t grp) {   // groups and vectors past the end re-read the last one
        const int64_t vec = grp * 16 + col;
        raw.load((const char *)x + (size_t)(vec < n_vec ? vec : n_vec - 1) * row_bytes, g);
    };
    load(wave);
    i32x4 a[KS][CB];
    const bool aligned = ((uintptr_t)Rm & 3) == 0;   // uniform
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            unsigned w[4][CB / 4];   // CB neighbouring entries of four coordinates
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int8_t *p = Rm + slot_coord<BF16>(ks, g, 4 * m + e) * NB + CB * col;
#pragma unroll
                for (int k = 0; k < CB / 4; ++k) {
                    if (aligned) {
                        w[e][k] = ((const unsigned *)p)[k];
                    } else {
                        w[e][k] = 0u;
#pragma unroll
                        for (int i = 0; i < 4; ++i) w[e][k] |= (unsigned)(uint8_t)p[4 * k + i] << (8 * i);
                    }
                }
            }
            // 4 x 4 bytes transposed: coordinates become the bytes of a word
#pragma unroll
            for (int k = 0; k < CB / 4; ++k) {
                const unsigned lo01 = __builtin_amdgcn_perm(w[1][k], w[0][k], 0x05010400u), hi01 = __builtin_amdgcn_perm(w[1][k], w[0][k], 0x07030602u);
                const unsigned lo23 = __builtin_amdgcn_perm(w[3][k], w[2][k], 0x05010400u), hi23 = __builtin_amdgcn_perm(w[3][k], w[2][k], 0x07030602u);
                a[ks][4 * k + 0][m] = (int)__builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
                a[ks][4 * k + 1][m] = (int)__builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
                a[ks][4 * k + 2][m] = (int)__builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
                a[ks][4 * k + 3][m] = (int)__builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
            }
        }
    for (int64_t grp = wave; grp < n_groups; grp += n_waves) {
        i32x4 b[KS];
        raw.quantise(qscale, b);
        load(grp + n_waves < n_groups ? grp + n_waves : grp);
        i32x4 acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            acc[cb] = i32x4{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc[cb] = mfma_i8_16x16x64(a[ks][cb], b[ks], acc[cb]);
        }
        const int64_t vec = grp * 16 + col;
        if (vec < n_vec) {
            // sum (v, cb) is bit CB * (4 g + v) + cb: 4 * CB bits of this lane, shifted in from the highest
            if constexpr (CB == 4) {
                unsigned neg = 0;
#pragma unroll
                for (int i = 15; i >= 0; --i) neg = __builtin_amdgcn_alignbit(neg, (unsigned)acc[i & 3][i >> 2], 31);
                ((uint16_t *)(bits + vec * (NB / 32)))[g] = (uint16_t)~neg;
            } else {
#pragma unroll
                for (int k = 0; k < CB / 8; ++k) {
                    unsigned neg = 0;
#pragma unroll
                    for (int i = 31; i >= 0; --i)
                        neg = __builtin_amdgcn_alignbit(neg, (unsigned)acc[(32 * k + i) % CB][(32 * k + i) / CB], 31);
                    bits[vec * (NB / 32) + g * (CB / 8) + k] = ~neg;
                }
            }
        }
    }
}

constexpr int SIGN_WORKGROUPS = 768;
template <bool BF16, int D, int NB>
static void launch_encode_sign(const void *x, int64_t n_vec, const int8_t *R, float qscale, uint32_t *bits,
                               hipStream_t s) {
    int64_t groups = (n_vec + 15) / 16;
    int64_t blocks = (groups + 3) / 4;
    // more workgroups than are resident (two to four per compute unit, by the operand's registers) would only repeat
    // the operand's set-up
    if (blocks > SIGN_WORKGROUPS) blocks = SIGN_WORKGROUPS;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL((encode_sign_kernel<BF16, D, NB>), dim3((unsigned)blocks), dim3(256), 0, s, x, n_vec, R, qscale,
                       bits);
}

}  // namespace fastar

extern "C" int fastar_encode(const void *x, int dtype, int64_t n_vec, int d, const fastar_codec *codec, int r,
                             int8_t *code_out, void *stream) {
    return fastar::encode_launch(x, dtype, n_vec, d, codec, r, code_out, nullptr, 0, (hipStream_t)stream);
}

extern "C" int fastar_encode_packed(const void *x, int dtype, int64_t n_vec, int d, const fastar_codec *codec, int r,
                                    int bits, uint8_t *packed_out, void *stream) {
    using namespace fastar;
    if (bits == 8) return encode_launch(x, dtype, n_vec, d, codec, r, (int8_t *)packed_out, nullptr, 0, (hipStream_t)stream);
    if (!x || !codec || !codec->R || !packed_out || n_vec < 0) return FASTAR_ERR_INVALID_ARG;
    if (dtype != FASTAR_F32 && dtype != FASTAR_BF16) return FASTAR_ERR_INVALID_ARG;
    if (bits != 2 && bits != 4) return FASTAR_ERR_INVALID_ARG;
    if (codec->shift < 1 || codec->shift > 16) return FASTAR_ERR_INVALID_ARG;
    if ((d != 64 && d != 128) || r != 32) return FASTAR_ERR_UNSUPPORTED;
    if (((uintptr_t)x & 15) || ((uintptr_t)packed_out & 3)) return FASTAR_ERR_INVALID_ARG;
    if (n_vec == 0) return FASTAR_OK;
    hipStream_t s = (hipStream_t)stream;
    int64_t blocks = ((n_vec + 15) / 16 + 3) / 4;
    if (blocks > 4096) blocks = 4096;
#define FASTAR_ENCP(B, DD, BB)                                                                                       \
    hipLaunchKernelGGL((encode_packed_kernel<B, DD, 32, BB>), dim3((unsigned)blocks), dim3(256), 0, s, x, n_vec, codec->R, \
                       codec->qscale, codec->shift, packed_out)
    const bool bf = dtype == FASTAR_BF16;
    if (d == 64) {
        if (bits == 4) { if (bf) FASTAR_ENCP(true, 64, 4); else FASTAR_ENCP(false, 64, 4); }
        else { if (bf) FASTAR_ENCP(true, 64, 2); else FASTAR_ENCP(false, 64, 2); }
    } else {
        if (bits == 4) { if (bf) FASTAR_ENCP(true, 128, 4); else FASTAR_ENCP(false, 128, 4); }
        else { if (bf) FASTAR_ENCP(true, 128, 2); else FASTAR_ENCP(false, 128, 2); }
    }
#undef FASTAR_ENCP
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}

extern "C" int fastar_encode_sign(const void *x, int dtype, int64_t n_vec, int d, const int8_t *R, float qscale,
                                  int n_bits, uint32_t *bits_out, void *stream) {
    using namespace fastar;
    if (!x || !R || !bits_out || n_vec < 0) return FASTAR_ERR_INVALID_ARG;
    if (dtype != FASTAR_F32 && dtype != FASTAR_BF16) return FASTAR_ERR_INVALID_ARG;
    if ((d != 64 && d != 128) || (n_bits != 64 && n_bits != 128 && n_bits != 256)) return FASTAR_ERR_UNSUPPORTED;
    if (((uintptr_t)x & 15) || ((uintptr_t)bits_out & 3)) return FASTAR_ERR_INVALID_ARG;
    if (n_vec == 0) return FASTAR_OK;
    hipStream_t s = (hipStream_t)stream;
    const bool bf = dtype == FASTAR_BF16;
#define FASTAR_ENCS(DD, NB)                                                              \
    do {                                                                                 \
        if (bf) launch_encode_sign<true, DD, NB>(x, n_vec, R, qscale, bits_out, s);      \
        else launch_encode_sign<false, DD, NB>(x, n_vec, R, qscale, bits_out, s);        \
    } while (0)
    if (d == 64 && n_bits == 64) FASTAR_ENCS(64, 64);
    else if (d == 64 && n_bits == 128) FASTAR_ENCS(64, 128);
    else if (d == 64) FASTAR_ENCS(64, 256);
    else if (n_bits == 64) FASTAR_ENCS(128, 64);
    else if (n_bits == 128) FASTAR_ENCS(128, 128);
    else FASTAR_ENCS(128, 256);
#undef FASTAR_ENCS
    FASTAR_LAUNCH_CHECK();
    return FASTAR_OK;
}
