// Integer GEMM with fused dequant / bias / GELU / requant epilogue (reordered linear, Eq. 2).
//
//   acc[m][c] = sum_k xq[m][k] * wq[c][k]      int8 MFMA (v_mfma_i32_32x32x32_i8), int32 exact
//   y         = fma((float)acc, s_x*s_w[c], b[c]);  optional GELU;  optional requantization
//
// Both operands stay PACKED (b-bit fields) in HBM and in LDS; a lane unpacks its fragment to
// int8 in registers right before the MFMA (2^(8-b)-scaled values, see vitq_dev.h), and the
// epilogue removes the scale exactly.
//
// MFMA roles: the A operand (32 rows) carries WEIGHT rows (output channels), the B operand
// (32 columns) carries TOKEN rows, so a lane of the 32x32 result holds 16 output channels of
// ONE token.  Weight rows are placed in LDS in a permuted slot order so that those 16 channels
// are consecutive: the lane then packs them into one 8-byte (4-bit) store of the token's
// output row, which is exactly the packed operand layout the next linear reads.
//
// Epilogues.  The definition of a requantized output is level = clamp(rint(y / s)) with an IEEE
// division.  The throughput epilogues evaluate a cheaper expression (multiplication by 1/s,
// hardware exp2/rcp inside GELU) whose distance from the definition is bounded; an element
// whose cheap value lies within that bound of a rounding boundary is recomputed with the exact
// operation sequence.  The result is therefore always the definition's, bit for bit.
#include "gemm.h"
#include <type_traits>
#include "launch_util.h"
#include "vitq_dev.h"

namespace vitq {

namespace {

#ifndef VITQ_TC
#define VITQ_TC 128
#define VITQ_TT 256
#define VITQ_WC 2
#define VITQ_WT 4
#define VITQ_BK44 128
#define VITQ_S44 3
#define VITQ_OCC44 4
#endif
#ifndef VITQ_BK88
#define VITQ_BK88 64
#define VITQ_S88 3
#define VITQ_OCC88 3
#endif
#ifndef VITQ_BK84
#define VITQ_BK84 128
#define VITQ_S84 2
#define VITQ_OCC84 4
#endif
enum Epi { kEpiGeneric = 0, kEpiF32 = 1, kEpiQuant = 2, kEpiQuantGelu = 3, kEpiHeadNorm = 4, kEpiAbsorbed = 5, kEpiAbsorbedBig = 6 };   // Big: more than 15 references per channel

// channel c (0..31 within a 32-block) -> MFMA row slot, chosen so that a lane's sixteen
// accumulator registers (rows 8*(r/4) + 4*(lane/32) + r%4) are channels 16*(lane/32) + r
__device__ __forceinline__ int slot_of_channel(int c) {
    return 8 * ((c & 15) >> 2) + 4 * (c >> 4) + (c & 3);
}

template <int WB, int AB>
struct Shift {
    // (8,4): weights expanded to plain int8 beforehand, activations unpacked to 16*x
    static constexpr int value = (WB == 4 && AB == 4) ? 8 : (WB == 2 && AB == 4) ? 10 : (WB == 8 && AB == 4) ? 4 : 0;
};

template <int SB>
__device__ __forceinline__ void store_packed16(uint8_t *dst, const int (&q)[16]) {
    u32 w[4];
    pack16<SB>(q, w);
    if constexpr (SB == 4) {
        *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
    } else if constexpr (SB == 8) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        *reinterpret_cast<u32 *>(dst) = w[0];
    }
}

// Destination of a lane's 16 packed levels = yq + token part + channel part (the address is
// linear in both).  Head-major mode: channel -> (q/k/v, head, d), token -> (image, n).  The two
// divisions avoid the integer-division expansion: the channel one by comparisons (3D channels)
// and a shift when the head size is a power of two; the token one by an fp32 reciprocal with a
// one-step correction (exact for m < 2^22).  A negative part marks "nothing to store".
__device__ __forceinline__ int64_t packed_token_part(const GemmParams &p, int m) {
    if (m >= p.M) return -1;
    if (p.head_major) {
        int b = (int)((float)m * p.inv_ntok);
        int n = m - b * p.Ntok;
        if (n < 0) { b -= 1; n += p.Ntok; }
        if (n >= p.Ntok) { b += 1; n -= p.Ntok; }
        return ((int64_t)b * p.Hh * p.Ntok + n) * p.yq_stride;
    }
    return (int64_t)m * p.yq_stride;
}
__device__ __forceinline__ int64_t packed_channel_part(const GemmParams &p, int cb, int &which) {
    which = 0;
    if (p.head_major) {
        if (cb >= p.Nout) return -1;
        which = (cb >= p.D ? 1 : 0) + (cb >= 2 * p.D ? 1 : 0);
        const int rem = cb - which * p.D;
        int h, d;
        if (p.dh_shift >= 0) { h = rem >> p.dh_shift; d = rem & (p.dh - 1); }
        else { h = rem / p.dh; d = rem - h * p.dh; }
        return (((int64_t)which * p.Bimg * p.Hh + h) * p.Ntok) * p.yq_stride + ((d * p.yq_sb) >> 3);
    }
    if (((cb * p.yq_sb) >> 3) >= p.yq_row_bytes16) return -1;
    return (cb * p.yq_sb) >> 3;
}
__device__ __forceinline__ uint8_t *packed_dst(const GemmParams &p, int m, int cb, int &which) {
    const int64_t t = packed_token_part(p, m), c = packed_channel_part(p, cb, which);
    if (t < 0 || c < 0) return nullptr;
    return p.yq + t + c;
}

// ---- exact epilogue: every output kind, the definition's operation sequence ------------------
__device__ __forceinline__ void epilogue_generic(const GemmParams &p, const v16i &acc, int shift,
                                                 int m, int cb) {
    if (m >= p.M) return;
    const int nvalid = p.Nout - cb;  // may be <= 0 for a group that only exists as padding
    const bool full = nvalid >= 16;
    float y[16];
    int a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int c = cb + r;
        const bool ok = c < p.Nout;
        // (an accumulators-only call carries no scales)
        const float sc = p.s_x * ((ok && p.s_w) ? p.s_w[p.s_w_per_channel ? c : 0] : 1.0f);
        const float bsr = (ok && p.bias) ? p.bias[c] : 0.0f;
        a[r] = acc[r] >> shift;
        float v = fmaf((float)a[r], sc, bsr);
        if (p.act == 1) v = gelu_tanh(v);
        if (p.res && ok && m < p.M) v = v + p.res[(int64_t)m * p.Nout + c];
        y[r] = v;
    }
    const bool vec = full && p.vec_ok;
    if (p.acc_out) {
        int32_t *dst = p.acc_out + (int64_t)m * p.Nout + cb;
        if (vec) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                reinterpret_cast<int4 *>(dst)[j] = make_int4(a[4 * j], a[4 * j + 1], a[4 * j + 2], a[4 * j + 3]);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (r < nvalid) dst[r] = a[r];
        }
    }
    if (p.y_out) {
        float *dst = p.y_out + (int64_t)m * p.Nout + cb;
        if (vec) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                reinterpret_cast<float4 *>(dst)[j] = make_float4(y[4 * j], y[4 * j + 1], y[4 * j + 2], y[4 * j + 3]);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (r < nvalid) dst[r] = y[r];
        }
    }
    if (p.yq) {
        int which;
        uint8_t *dst = packed_dst(p, m, cb, which);
        if (!dst) return;
        const float sy0 = p.s_y[0], sy1 = p.s_y[1], sy2 = p.s_y[2];
        const float s_y = which == 0 ? sy0 : (which == 1 ? sy1 : sy2);
        int q[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            int lv = quantize_level(y[r], s_y, p.qminf, p.qmaxf);
            q[r] = (r < nvalid) ? lv : 0;
        }
        if (p.yq_sb == 4) store_packed16<4>(dst, q);
        else if (p.yq_sb == 8) store_packed16<8>(dst, q);
        else store_packed16<2>(dst, q);
    }
}

// ---- fp32-only epilogue (Nout % 16 == 0) -------------------------------------------------------
// This epilogue runs with the MFMA roles SWAPPED (tokens on the A side, weight rows on the B
// side, weight rows unpermuted in LDS): a lane then holds ONE channel of sixteen tokens, and
// register r of the wave is 32 consecutive channels (one full 128-byte line) of tokens
// m0 + 8*(r/4) + r%4 (+4 for the upper half-wave).  Every store instruction therefore writes
// two complete lines instead of 64 scattered 16-byte pieces.
// The caller passes the folded scale (sc * 2^-shift exactly, so fma((float)acc_scaled, scs, b) ==
// fma((float)acc, sc, b)) with shift 0, or, when the fold was inexact, the plain one and the shift.
template <bool FULL, bool RES>   // FULL: the whole tile lies inside the matrix (no per-element tests); RES: residual given
__device__ __forceinline__ void epilogue_f32(const GemmParams &p, const v16i &acc, int shift, int m0, int ch,
                                             float sc, float bs, const float (&rv)[16]) {
    if (!FULL && ch >= p.Nout) return;
    float *out = p.y_out + (int64_t)m0 * p.Nout + ch;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int dm = 8 * (r >> 2) + (r & 3);
        if (FULL || m0 + dm < p.M) {
            float y = fmaf((float)(acc[r] >> shift), sc, bs);
            if constexpr (RES) y = y + rv[r];               // residual stream
            out[(int64_t)dm * p.Nout] = y;
        }
    }
}
// The residual elements of one 32x32 block, in the register order of epilogue_f32 (each element
// is read by the lane that later writes it, so the stream may be updated in place).
template <bool FULL>
__device__ __forceinline__ void load_residual(const GemmParams &p, int m0, int ch, float (&rv)[16]) {
    if (!FULL && ch >= p.Nout) return;
    const float *res = p.res + (int64_t)m0 * p.Nout + ch;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int dm = 8 * (r >> 2) + (r & 3);
        if (FULL || m0 + dm < p.M) rv[r] = res[(int64_t)dm * p.Nout];
    }
}

// Packs sixteen levels (floats holding level - qmin, i.e. 0 .. qmax - qmin) into 4- or 8-bit
// two's-complement fields and stores them: 8 or 16 bytes at dst.
__device__ __forceinline__ void pack_store16(const GemmParams &p, uint8_t *dst, const float (&lv)[16], float bias8) {
    if (p.yq_sb == 4) {
        // even-indexed levels in the low nibbles of one word, odd-indexed shifted into the high
        u32 ev0 = 0, od0 = 0, ev1 = 0, od1 = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ev0 = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i], i, ev0);
            od0 = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i + 1], i, od0);
            ev1 = __builtin_amdgcn_cvt_pk_u8_f32(lv[8 + 2 * i], i, ev1);
            od1 = __builtin_amdgcn_cvt_pk_u8_f32(lv[8 + 2 * i + 1], i, od1);
        }
        // stored levels are biased by -qmin = 2^(bits-1); remove it per nibble, modulo 16 and
        // without borrows across nibbles (for 4-bit levels this is a flip of bit 3)
        const u32 a0 = ev0 | (od0 << 4), a1 = ev1 | (od1 << 4);
        u32 w0, w1;
        if (bias8 == 8.0f) {                 // (uniform) 4-bit levels: subtracting 8 modulo 16 flips bit 3
            w0 = a0 ^ 0x88888888u;
            w1 = a1 ^ 0x88888888u;
        } else {
            const u32 fix = 0x11111111u * ((u32)bias8 & 0xFu);
            w0 = ((a0 | 0x88888888u) - (fix & 0x77777777u)) ^ ((a0 ^ ~fix) & 0x88888888u);
            w1 = ((a1 | 0x88888888u) - (fix & 0x77777777u)) ^ ((a1 ^ ~fix) & 0x88888888u);
        }
        *reinterpret_cast<uint2 *>(dst) = make_uint2(w0, w1);
    } else {
        // 8-bit storage: the bias -qmin = 2^(bits-1) is removed modulo 256
        const u32 fix = 0x01010101u * ((u32)bias8 & 0xFFu);
        u32 w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u32 v = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) v = __builtin_amdgcn_cvt_pk_u8_f32(lv[4 * j + i], i, v);
            // per-byte subtraction of the bias: (v - fix) without borrows across bytes
            w[j] = ((v | 0x80808080u) - (fix & 0x7F7F7F7Fu)) ^ ((v ^ ~fix) & 0x80808080u);
        }
        *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Eight levels (floats holding level - qmin) -> one word of 4-bit fields (w[0]) or two words of
// 8-bit fields, two's complement, bias removed.
__device__ __forceinline__ void pack8(const GemmParams &p, const float (&lv)[8], float bias8, u32 (&w)[2]) {
    if (p.yq_sb == 4) {
        u32 ev = 0, od = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ev = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i], i, ev);
            od = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i + 1], i, od);
        }
        const u32 a = ev | (od << 4);
        if (bias8 == 8.0f) {                 // (uniform) 4-bit levels: subtracting 8 modulo 16 flips bit 3
            w[0] = a ^ 0x88888888u;
        } else {
            const u32 fix = 0x11111111u * ((u32)bias8 & 0xFu);
            w[0] = ((a | 0x88888888u) - (fix & 0x77777777u)) ^ ((a ^ ~fix) & 0x88888888u);
        }
        w[1] = 0;
    } else {
        const u32 fix = 0x01010101u * ((u32)bias8 & 0xFFu);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            u32 v = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) v = __builtin_amdgcn_cvt_pk_u8_f32(lv[4 * j + i], i, v);
            w[j] = ((v | 0x80808080u) - (fix & 0x7F7F7F7Fu)) ^ ((v ^ ~fix) & 0x80808080u);
        }
    }
}

// A 16-channel group that lies wholly beyond the last output channel but inside the 16-byte
// padded row: the packed format wants zero bytes there.
__device__ __forceinline__ void store_zero_group(const GemmParams &p, uint8_t *dst) {
    if (!dst) return;
    if (p.yq_sb == 4) *reinterpret_cast<uint2 *>(dst) = make_uint2(0u, 0u);
    else *reinterpret_cast<uint4 *>(dst) = make_uint4(0u, 0u, 0u, 0u);
}

// ---- guarded fast requantization (Nout % 16 == 0; 4- or 8-bit storage) ------------------------
// Definition: level = clamp(rint(T)), T = RN(y / s).  Cheap value: with r = RN(1/s), g = eps0 =
// 2^(bits-22) and C = -qmin + 1/2 - g (exactly representable),
//     u = fma(y, r, C),   |u - (T - qmin + 1/2 - g)| <= |T| * 2^-23 + ulp(u)/2  <  g   for |T| <= qmax + 2.
// If fract(u) < 1 - 2g then T - qmin + 1/2 lies strictly inside (floor(u), floor(u) + 1): it is not
// a tie and rint(T) - qmin = floor(u) = u - fract(u) (an exact subtraction).  Otherwise the element
// sits within the error bound of a rounding boundary and is redone with the definition's own
// operations.  Beyond |T| = qmax + 2 both clamp to the same level; a NaN or infinity gives a NaN
// fraction, whose bit pattern compares above every threshold, so it is redone too.
// With GELU the cheap activation (gelu_fast: hardware exp2 / rcp) is within kGeluFastBound * |y| of the
// definition's, which widens the guard per element (there the test is on |t - rint(t)|).
// The sixteen channels of a lane are done in two halves of eight (each with its own test and, if
// need be, its own exact redo): the working set stays small enough for four waves per SIMD.
// lscs / lbs: this lane's sixteen folded scales and biases in LDS.
template <bool GELU>
__device__ __forceinline__ void epilogue_quant(const GemmParams &p, const v16i &acc, int shift, uint8_t *dst,
                                               float s_y, float r_y, int cb, const float *lscs, const float *lbs,
                                               bool force_exact) {
    if (!dst) return;
    const float bias8 = -p.qminf;
    const float top = p.qmaxf - p.qminf;
    u32 words[4];
    static_for<2>([&](auto H) {
        constexpr int h = decltype(H)::value;
        float scs[8], bs[8];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float4 a = *reinterpret_cast<const float4 *>(lscs + 8 * h + 4 * j);
            const float4 b = *reinterpret_cast<const float4 *>(lbs + 8 * h + 4 * j);
            scs[4 * j] = a.x; scs[4 * j + 1] = a.y; scs[4 * j + 2] = a.z; scs[4 * j + 3] = a.w;
            bs[4 * j] = b.x; bs[4 * j + 1] = b.y; bs[4 * j + 2] = b.z; bs[4 * j + 3] = b.w;
        }
        float lv[8];
        // worst = max over the elements of a non-negative per-element figure, taken on the bit
        // patterns: there unsigned order is float order and a NaN compares above everything (so
        // it is caught, which a float max would drop)
        u32 worst = force_exact ? 0x7F800000u : 0u;
        u32 fig[8];
        u32 limit;
        if constexpr (GELU) {
            const float gguard = p.gelu_guard * r_y;
            limit = __float_as_uint(0.5f - p.eps0);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float y = fmaf((float)acc[8 * h + r], scs[r], bs[r]);        // the definition's y, exactly
                const float g = gelu_fast(y);
                const float t8 = fmaf(g, r_y, bias8);
                const float q8 = rintf(t8);
                fig[r] = __float_as_uint(fmaf(fabsf(y), gguard, fabsf(t8 - q8)));
                lv[r] = __builtin_amdgcn_fmed3f(q8, 0.0f, top);
            }
        } else {
            const float C = (bias8 + 0.5f) - p.eps0;
            limit = __float_as_uint(1.0f - 2.0f * p.eps0) - 1u;              // risky: fract(u) >= 1 - 2g
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float y = fmaf((float)acc[8 * h + r], scs[r], bs[r]);        // the definition's y, exactly
                const float u = fmaf(y, r_y, C);
                const float z = __builtin_amdgcn_fractf(u);
                fig[r] = __float_as_uint(z);
                lv[r] = __builtin_amdgcn_fmed3f(u - z, 0.0f, top);
            }
        }
#pragma unroll
        for (int r = 0; r < 8; r += 2) worst = max(worst, max(fig[r], fig[r + 1]));
        const bool risky = worst > limit;
        if (__builtin_amdgcn_ballot_w64(risky) != 0) {
            // some element of these eight channels x 32 tokens sits within the error bound of a rounding
            // boundary: redo them with the definition's exact operation sequence (rare)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                // (re-read the channel's step: the folded copy may be inexact when force_exact is set)
                const float sc = p.s_x * p.s_w[p.s_w_per_channel ? cb + 8 * h + r : 0];
                float ye = fmaf((float)(acc[8 * h + r] >> shift), sc, bs[r]);
                if constexpr (GELU) ye = gelu_tanh(ye);
                const float te = rintf(ye / s_y) + bias8;
                lv[r] = __builtin_amdgcn_fmed3f(te, 0.0f, top);
            }
        }
        u32 w2[2];
        pack8(p, lv, bias8, w2);
        words[2 * h] = w2[0];
        words[2 * h + 1] = w2[1];
    });
    if (p.yq_sb == 4) *reinterpret_cast<uint2 *>(dst) = make_uint2(words[0], words[2]);
    else *reinterpret_cast<uint4 *>(dst) = make_uint4(words[0], words[1], words[2], words[3]);
}

// ---- per-head LayerNorm quantizers of Q and K in the QKV epilogue (Sec. IV-C, Table I) ----------
// Heads are 64 channels and a wave's tile is 64 channels x 64 tokens, so a wave holds whole
// (token, head) groups: after the accumulation, lanes l and l+32 own the two 16-channel halves
// of each 32-channel block of token l (first token block) and of token 32+l (second block).
// One v_permlane32_swap per register pair trades those halves, after which lane (l, g) owns all
// 64 channels of ONE token (block g) and can walk them in order, as Eq. 5 requires: the mean and
// the sum of squared deviations are the fp32 recurrences in element order, and every level is
// the sigma-free comparator's: a guess from the hardware reciprocal square root stands when it is
// provably far from every boundary, and otherwise picks which two comparisons are evaluated.
// The fp32 linear output never leaves registers.
// gamma / beta / the folded scales are wave-uniform: staged in LDS once per tile and read as
// broadcasts.  tmp: this lane's column of 64 x 64 floats in LDS.
// Bound by VALU issue at two waves per SIMD.  The attention block with it, us, with a division per element and a verification
// branch per level / with the quotients below and one test per eight levels, the comparator in line / behind them: 256 ViT-B
// images in 4 bits 328 / 276 / 273, in 8 bits 416 / 372 / 362; 50 DeiT-S images, 2-bit weights 54.1 / 45.5 / 44.9.
constexpr float kHnGuard = 0x1p-21f;   // unit of the guard that lets a guessed level stand (see the LayerNorm kernel)
template <int SB, int NTK, int PAIR>   // PAIR: token blocks 2*PAIR and 2*PAIR + 1 of the wave's NTK
__device__ __forceinline__ void epilogue_headnorm(const GemmParams &p, v16i (&acc)[2][NTK], int shift, uint8_t *dst,
                                                  const float *scs64, const float *bs64, float step,
                                                  const float *gp, const float *bp, float *tmp) {
    // trade halves: afterwards sw[0] is channel 32*ci + r and sw[1] channel 32*ci + 16 + r of this
    // lane's token.  The definition's y = fma((float)acc, s_x*s_w[c], b[c]); the caller passes
    // either the folded scales (which carry 2^-shift exactly) with shift 0, or the plain ones.
    float v[64];
    auto to_y = [&](int a, int i) { return fmaf((float)(a >> shift), scs64[i], bs64[i]); };
#pragma unroll
    for (int ci = 0; ci < 2; ++ci) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const auto sw = __builtin_amdgcn_permlane32_swap(acc[ci][2 * PAIR][r], acc[ci][2 * PAIR + 1][r], false, false);
            v[32 * ci + r] = to_y((int)sw[0], 32 * ci + r);
            v[32 * ci + 16 + r] = to_y((int)sw[1], 32 * ci + 16 + r);
        }
        __builtin_amdgcn_sched_barrier(0);   // the two accumulator tiles are dead before the next pair is touched
    }
    // The running mean's division by a constant is a multiply and an FMA (a multiply where it is a power of two) with
    // 1/i as a sum hi + lo of two fp32 numbers: the bits of the IEEE quotient for a deviation of zero or at least 2^-98 and
    // a finite mean (proof at the LayerNorm kernel's table).  Any other token is walked again with divisions.
    float mu = 0.0f, m2 = 0.0f;
    u32 least = 0xFFFFFFFFu;                                 // twice the bits of the smallest nonzero deviation, minus one
    static_for<64>([&](auto I) {
        constexpr int i = decltype(I)::value, k = i + 1;
        constexpr float hi = 1.0f / (float)k, lo = (float)((1.0 - (double)hi * (double)k) / (double)k);
        const float d1 = v[i] - mu;
        if constexpr ((k & (k - 1)) == 0) {
            mu = mu + d1 * hi;
        } else {
            const float tq = d1 * lo;
            mu = mu + fmaf(d1, hi, tq);
            least = min(least, (__float_as_uint(d1) << 1) - 1u);         // (zero wraps to the largest value)
        }
        const float d2 = v[i] - mu;
        const float pr = d1 * d2;
        m2 = m2 + pr;
    });
    asm volatile("" : "+v"(m2));   // (or its chain sinks past the branch below, all deviations and means held until there)
    const bool walked = fabsf(mu) <= 3.0e38f && least >= 2u * __float_as_uint(0x1p-98f) - 1u;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!walked) != 0, 0)) {
        // (rare; from LDS and rolled up, so that its divisions cost the others no registers)
        mu = 0.0f;
        m2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 64; ++i) tmp[64 * i] = v[i];
#pragma unroll 1
        for (int i = 0; i < 64; ++i) {
            const float x = tmp[64 * i];
            const float d1 = x - mu;
            mu = mu + d1 / (float)(i + 1);
            const float d2 = x - mu;
            const float pr = d1 * d2;
            m2 = m2 + pr;
        }
    }
    const float nf = 64.0f;
    const float ne = nf * p.hn_eps;
    const float V = m2 + ne;
    const float rstep = __builtin_amdgcn_rcpf(step);         // for the guess only
    const float rsr = __builtin_amdgcn_rsqf(V / nf) * rstep; // for the guess only
    const bool stats_ok = step >= 0x1p-20f && step <= 0x1p10f && V >= 0x1p-40f && V <= 0x1p30f;
    const float qminf = p.qminf, qmaxf = p.qmaxf;
    const int span = (int)(qmaxf - qminf);
    const float bias8 = -qminf;
    // The guess tp is within (|g/(sigma*step)| + |beta/step|) * 2^-21 of the exact-arithmetic value the
    // comparator tests, and the comparator's own fp32 evaluation moves a boundary by at most
    // (2|level| + |beta/step| + 1) * 2^-22: a guess further than 2^-21 * (4|tp| + 3|beta/step| + 3) from every
    // half-integer is the level the comparator would count, and it is not run (stats_ok: the squares stay
    // ordinary numbers, which that error model needs).  Eight channels share one test, with the largest |beta/step|
    // of theirs; the figures are compared as bit patterns, where a NaN is above everything and fails it.
    // Levels leave biased, 0 .. qmax - qmin, one byte each: w8[2*j], w8[2*j + 1] hold channels 8*j .. 8*j + 7.
    u32 w8[16];
    u32 unsure = 0;                                          // groups of eight channels with one to be compared
    static_for<8>([&](auto J) {
        constexpr int j = decltype(J)::value;
        float lv[8];
        u32 worst = 0u, bmax = 0u;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = 8 * j + r;
            const float btr = bp[i] * rstep;
            const float g = (v[i] - mu) * gp[i];
            const float tp = fmaf(g, rsr, btr);
            const float tt = rintf(tp);
            worst = max(worst, __float_as_uint(fmaf(fabsf(tp), 4.0f * kHnGuard, fabsf(tp - tt))));
            bmax = max(bmax, __float_as_uint(fabsf(btr)));
            lv[r] = __builtin_amdgcn_fmed3f(tt, qminf, qmaxf);
        }
        const float fig = __uint_as_float(worst) + fmaf(__uint_as_float(bmax), 3.0f * kHnGuard, 3.0f * kHnGuard);
        if (!(stats_ok && fig <= 0.5f)) {                    // (rare: decided below)
            unsure |= 1u << j;
#pragma unroll
            for (int r = 0; r < 8; ++r) tmp[64 * (8 * j + r)] = v[8 * j + r];
        }
        u32 ev = 0, od = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // 4 bits: even and odd channels apart, as the nibbles are merged; 8 bits: in order
            ev = __builtin_amdgcn_cvt_pk_u8_f32(lv[SB == 4 ? 2 * r : r] + bias8, r, ev);
            od = __builtin_amdgcn_cvt_pk_u8_f32(lv[SB == 4 ? 2 * r + 1 : 4 + r] + bias8, r, od);
        }
        w8[2 * j] = ev;
        w8[2 * j + 1] = od;
        __builtin_amdgcn_sched_barrier(0);
    });
    if (!dst) return;
    if constexpr (SB == 4) {
        const u32 fix = 0x11111111u * ((u32)bias8 & 0xFu);
        u32 w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32 a0 = w8[2 * j] | (w8[2 * j + 1] << 4);
            w[j] = ((a0 | 0x88888888u) - (fix & 0x77777777u)) ^ ((a0 ^ ~fix) & 0x88888888u);
        }
        *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
        *reinterpret_cast<uint4 *>(dst + 16) = make_uint4(w[4], w[5], w[6], w[7]);
    } else {
        const u32 fix = 0x01010101u * ((u32)bias8 & 0xFFu);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32 w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u32 x = w8[4 * q + j];
                w[j] = ((x | 0x80808080u) - (fix & 0x7F7F7F7Fu)) ^ ((x ^ ~fix) & 0x80808080u);
            }
            *reinterpret_cast<uint4 *>(dst + 16 * q) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    // The comparator, for groups with a guess near a boundary: from LDS and over what was stored, when nothing else of this
    // token is held.  (It is not that rare with 8-bit levels: a wave has such a lane in one of twelve groups or so.)
    while (unsure) {
        const int j = __builtin_ctz(unsure);
        unsure &= unsure - 1;
        float L[8], bt[8], lv[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = 8 * j + r;
            bt[r] = bp[i];
            const float a = tmp[64 * i] - mu;
            const float g = a * gp[i];
            const float gs = g * fabsf(g);
            L[r] = gs * nf;
            lv[r] = rintf(fmaf(g, rsr, bt[r] * rstep));
            lv[r] = (lv[r] == lv[r]) ? fminf(fmaxf(lv[r], qminf), qmaxf) : qminf;
        }
        auto above = [&](int r, float k) {
            const float rk = (k - 0.5f) * step;
            const float cc = rk - bt[r];
            const float cs = cc * fabsf(cc);
            const float R = cs * V;
            return L[r] > R;
        };
        for (int it = 0; it <= span; ++it) {
            bool moved = false;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const bool low_ok = (lv[r] <= qminf) || above(r, lv[r]);
                const bool high_ok = (lv[r] >= qmaxf) || !above(r, lv[r] + 1.0f);
                const float d = !low_ok ? -1.0f : (!high_ok ? 1.0f : 0.0f);
                lv[r] = lv[r] + d;
                moved = moved || d != 0.0f;
            }
            if (!moved) break;
        }
        u32 w[2] = {0, 0};
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if constexpr (SB == 4) w[0] |= ((u32)(int)lv[r] & 0xFu) << (4 * r);
            else w[r / 4] |= ((u32)(int)lv[r] & 0xFFu) << (8 * (r % 4));
        }
        if constexpr (SB == 4) *reinterpret_cast<u32 *>(dst + 4 * j) = w[0];
        else *reinterpret_cast<uint2 *>(dst + 8 * j) = make_uint2(w[0], w[1]);
    }
}

// ---- integer-only epilogue: equivalent bias + comparator references with the scales absorbed ----
// (Eq. 2, second form; Sec. IV-B.)  level = qmin + #{t : acc + b_int[c] > T[c][t]}, T non-decreasing
// in t, so the count is found by bisection: 4 integer comparisons for up to 15 references, 8 for up
// to 255, no branch, no floating point.  The tile keeps rows of kAbsRow entries in LDS: the references
// themselves when there are at most 15 per channel, else every sixteenth one (T[15], T[31], ...), which
// settles the first four strides; the last four then probe one 16-entry stretch of the caller's table
// in global memory.
// acc + b_int may leave 32 bits (a near-dead channel's bias lies at the int32 limits), T - b_int too, but there
// saturation changes no comparison: acc is at most 2^30 in size.  So the references are taken relative to
// the bias, and a row in LDS holds them ready to be compared with the accumulator as it is (absorbed_reference).
constexpr int kAbsRow = 17;
// |acc| <= 2^(WB-1) * 2^(AB-1) * K, K <= 65536: with the operand factor 2^shift at most 2^30 for every pair of
// operands.  T - b, held to that range, compares like T - b itself; INT32_MAX is never exceeded.
template <int WB, int AB>
__device__ __forceinline__ int absorbed_reference(int T, int b) {
    constexpr int shift = Shift<WB, AB>::value, most = 1 << (30 - shift);
    static_assert(WB + AB - 2 + 16 <= 30 - shift, "accumulators");
    return min(max(__builtin_elementwise_sub_sat(T, b), -most), most) * (1 << shift);
}
template <bool TBL_LDS>
__device__ __forceinline__ void epilogue_absorbed(const GemmParams &p, const v16i &acc, int shift, uint8_t *dst,
                                                  const int *lds_tbl, const int *glb_tbl, int64_t glb_row, const int *bint) {
    if (!dst) return;
    const int nthr = p.ab_nthr;
    float lv[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int4 b4 = *reinterpret_cast<const int4 *>(bint + 4 * q);
        const int bq[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * q + i;
            int pos = 0;                                // references known to be exceeded
            if constexpr (TBL_LDS) {
#pragma unroll
                for (int step = 8; step >= 1; step >>= 1)
                    pos += acc[r] > lds_tbl[r * kAbsRow + pos + step - 1] ? step : 0;
            } else {
                // strides 128..16 probe T[16(i+1) - 1]: entry i of the LDS row; strides 8..1 finish
                // inside one 16-entry stretch of the caller's table
#pragma unroll
                for (int step = 128; step >= 16; step >>= 1)
                    pos += acc[r] > lds_tbl[r * kAbsRow + ((pos + step) >> 4) - 1] ? step : 0;
#pragma unroll
                for (int step = 8; step >= 1; step >>= 1) {
                    const int t = pos + step - 1;
                    const int v = __builtin_elementwise_sub_sat(glb_tbl[(int64_t)r * glb_row + min(t, nthr - 1)], bq[i]);
                    pos += (acc[r] >> shift) > (t >= nthr ? INT32_MAX : v) ? step : 0;
                }
            }
            lv[r] = (float)pos;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    pack_store16(p, dst, lv, -p.qminf);
}

// The same count where every channel of the tile has nearly evenly spaced references, as absorbed scales give: with the
// reference nearest to the sum, b = rint((v - T[0]) / spacing) kept inside the table, the count is b + (v > T[b]), one LDS
// read per element instead of four dependent ones.  T[t] is within 3/8 of a spacing of T[0] + t * spacing and b's
// argument right within 1/8 (checked and bounded where the biases are staged), so v lies above T[b-1] and not above T[b+1].
// us, four dependent reads / this: 12,608 x 768 -> 768 17.4 / 15.0 (12.6 for the floating-point requantizer), 50,432 rows
// 45.6 / 39.0, 25,216 x 1024 -> 3072 100 / 90.
// row: the tile's table from this lane's first channel on; ca, cb: spacing^-1 * 2^-shift and
// (b_int - T[0]) / spacing + 1/2 of the lane's sixteen channels.
__device__ __forceinline__ void epilogue_absorbed_even(const GemmParams &p, const v16i &acc, uint8_t *dst, const int *row,
                                                       const float *ca, const float *cb) {
    if (!dst) return;
    const float top = (float)p.ab_nthr - 0.5f;
    int lv[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 a4 = *reinterpret_cast<const float4 *>(ca + 4 * q), b4 = *reinterpret_cast<const float4 *>(cb + 4 * q);
        const float aq[4] = {a4.x, a4.y, a4.z, a4.w}, bq[4] = {b4.x, b4.y, b4.z, b4.w};
        int t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            t[i] = (int)__builtin_amdgcn_fmed3f(fmaf((float)acc[4 * q + i], aq[i], bq[i]), 0.0f, top);
#pragma unroll
        for (int i = 0; i < 4; ++i) lv[4 * q + i] = t[i] + (acc[4 * q + i] > row[(4 * q + i) * kAbsRow + t[i]] ? 1 : 0);
    }
    const u32 bias = (u32)(int)(-p.qminf);                       // stored levels are signed: count + qmin
    if (p.yq_sb == 4) {
        u32 w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32 x = (u32)lv[8 * h];
#pragma unroll
            for (int i = 1; i < 8; ++i) x |= (u32)lv[8 * h + i] << (4 * i);
            const u32 fix = 0x11111111u * (bias & 0xFu);
            w[h] = ((x | 0x88888888u) - (fix & 0x77777777u)) ^ ((x ^ ~fix) & 0x88888888u);
        }
        *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
    } else {
        u32 w[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            u32 x = (u32)lv[4 * h];
#pragma unroll
            for (int i = 1; i < 4; ++i) x |= (u32)lv[4 * h + i] << (8 * i);
            const u32 fix = 0x01010101u * (bias & 0xFFu);
            w[h] = ((x | 0x80808080u) - (fix & 0x7F7F7F7Fu)) ^ ((x ^ ~fix) & 0x80808080u);
        }
        *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// ---- direct global -> LDS loads ----------------------------------------------------------------
// global_load_lds_dwordx4: lane i of the wave writes its 16 bytes to LDS address M0 + 16*i; no
// VGPRs are used for the data, so several k-stages can be in flight at once.  The compiler does
// not see these loads: completion is tracked by hand with s_waitcnt vmcnt(n) (loads retire in
// order), followed by a workgroup barrier before any lane reads the stage.
__device__ __forceinline__ u32 lds_address(const void *p) {
    return (u32)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)p;
}
// address = sbase (uniform) + voff (per lane)
__device__ __forceinline__ void dma16(u32 voff, const uint8_t *sbase, u32 lds_dst) {
    u32 keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "v"(voff), "s"(sbase), "s"(lds_dst) : "memory");
}
// address = per-lane pointer
__device__ __forceinline__ void dma16_ptr(const uint8_t *ptr, u32 lds_dst) {
    u32 keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "v"(ptr), "s"(lds_dst) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// sixteen zero bytes: the source of operand chunks that lie beyond the end of a row (K tail)
__device__ __attribute__((aligned(16))) const u32 g_zero16[4] = {0u, 0u, 0u, 0u};

// XOR swizzle of the 16-byte chunk index inside an LDS row of CH chunks (rows are stored without
// padding): spreads the rows that consecutive lanes read over all banks.
template <int CH>
__device__ __forceinline__ int swz(int row) {
    if constexpr (CH == 4) return ((row >> 2) & 3) ^ (row & 2);
    else if constexpr (CH == 8) return row & 7;
    else if constexpr (CH == 2) return (row >> 3) & 1;
    else return 0;
}

// inverse of slot_of_channel
__device__ __forceinline__ int channel_of_slot(int s) {
    return 16 * ((s >> 2) & 1) + 4 * (s >> 3) + (s & 3);
}

// marks every fragment of a set as used (and possibly modified) here: an anchor for the scheduler
template <int N>
__device__ __forceinline__ void pin_frags(v4i (&f)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i]));
}

// LDS of the k-stages; the head-norm epilogue keeps 64 values per lane there afterwards
template <int EPI, int WAVES, int STAGES>
constexpr int pipeline_lds = EPI == kEpiHeadNorm && WAVES * 16384 > STAGES ? WAVES * 16384 : STAGES;

template <int WB, int AB, int TC, int TT, int WAVES_C, int WAVES_T, int BK, int S, int OCC, int EPI>
__global__ __launch_bounds__(WAVES_C *WAVES_T * 64, OCC)
void gemm_kernel(GemmParams p) {
    constexpr int NT = WAVES_C * WAVES_T * 64;                // S = k-stages resident in LDS
    constexpr int WROW = BK * WB / 8, XROW = BK * AB / 8;     // bytes per row per stage
    constexpr int WCH = WROW / 16, XCH = XROW / 16;           // 16-byte chunks per row
    constexpr int W_ITERS = TC * WCH / NT, X_ITERS = TT * XCH / NT;
    static_assert((TC * WCH) % NT == 0 && (TT * XCH) % NT == 0, "tile/threads mismatch");
    constexpr int LOADS = W_ITERS + X_ITERS;                  // loads per lane per stage
    constexpr int WC = TC / WAVES_C, WT = TT / WAVES_T;       // wave tile
    constexpr int NC = WC / 32, NTK = WT / 32;                // 32x32 blocks per wave
    static_assert(WC % 32 == 0 && WT % 32 == 0 && TC % 64 == 0 && BK % 64 == 0, "wave tile");
    constexpr int WBUF = TC * WROW, XBUF = TT * XROW, STAGE = WBUF + XBUF;
    constexpr bool SWAP = (EPI == kEpiF32);   // tokens as the MFMA A operand (see epilogue_f32)
    constexpr bool ABSORBED = (EPI == kEpiAbsorbed || EPI == kEpiAbsorbedBig);   // integer-only epilogue

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    float *s_scs = reinterpret_cast<float *>(smem + pipeline_lds<EPI, WAVES_C * WAVES_T, S * STAGE>);     // [TC] folded scales
    float *s_bs = s_scs + TC;                                             // [TC] biases
    int *s_fold_bad = reinterpret_cast<int *>(s_bs + TC);                 // [1] flag
    [[maybe_unused]] float *s_raw = s_bs + TC + 4;                        // [TC] plain scales (fp32, head-norm epilogues)
    [[maybe_unused]] float *s_hg = s_raw + TC, *s_hb = s_raw + 2 * TC;    // [TC] each: gamma, beta of the head-norm epilogue

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_c = wave % WAVES_C;
    const int wave_t = wave / WAVES_C;
    const int li = lane & 31;   // MFMA row / column index of this lane
    const int g = lane >> 5;    // k-group of this lane

    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Re-number them so
    // that the workgroups of one XCD walk consecutive tiles: the channel tiles of one token tile
    // then share that XCD's L2 copy of the activations.
    const int n_ct = (p.Nout + TC - 1) / TC;
    int logical;
    {
        const int total = gridDim.x, id = blockIdx.x;
        const int xcd = id & 7, slot = id >> 3;
        const int per = total >> 3, rem = total & 7;
        logical = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + slot;
    }
    const int ct = logical % n_ct;
    const int tt = logical / n_ct;
    const int c0 = ct * TC;
    const int t0 = tt * TT;

    // ---- stage loads: what each lane fetches is fixed; only the k offset (uniform) advances ----
    // LDS position pos (16-byte units) of a tile holds row pos / CH, chunk (pos % CH) ^ swz(row).
    // Weight rows sit in permuted slots (slot_of_channel) unless the roles are swapped.  Rows
    // beyond the matrix are clamped to its last row: their products land in accumulators that
    // are never stored.
    const int nk = (p.K + BK - 1) / BK;
    const bool ktail = (nk * WROW > p.kbytes_w16) || (nk * XROW > p.kbytes_x16);
    const uint8_t *wbase = p.w + (int64_t)c0 * p.w_stride;
    const uint8_t *xbase = p.x + (int64_t)t0 * p.x_stride;
    u32 w_off[W_ITERS], x_off[X_ITERS];
    int w_kb[W_ITERS], x_kb[X_ITERS];
#pragma unroll
    for (int it = 0; it < W_ITERS; ++it) {
        const int pos = it * NT + tid;
        const int slot = pos / WCH;
        const int chunk = (pos % WCH) ^ swz<WCH>(slot);
        int row = SWAP ? slot : ((slot & ~31) | channel_of_slot(slot & 31));
        row = min(row, p.Nout - 1 - c0);
        w_off[it] = (u32)row * (u32)p.w_stride + (u32)chunk * 16u;
        w_kb[it] = chunk * 16;
    }
#pragma unroll
    for (int it = 0; it < X_ITERS; ++it) {
        const int pos = it * NT + tid;
        int row = pos / XCH;
        const int chunk = (pos % XCH) ^ swz<XCH>(row);
        row = min(row, p.M - 1 - t0);
        x_off[it] = (u32)row * (u32)p.x_stride + (u32)chunk * 16u;
        x_kb[it] = chunk * 16;
    }
    const u32 lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem)) + (u32)wave * 1024u;
    // The LOADS loads of a stage (weights first, then tokens) are issued in kParts groups: a burst of
    // all of them from all four waves queues up in the CU's one address path and stalls every wave
    // for hundreds of cycles, so the main loop spreads the groups over several MFMA steps.
    constexpr int kParts = 3;
    constexpr int kPartLoads = (LOADS + kParts - 1) / kParts;
    auto issue_part = [&](int kt, auto PART) {
        constexpr int lo = decltype(PART)::value * kPartLoads;
        constexpr int hi = (lo + kPartLoads < LOADS) ? lo + kPartLoads : LOADS;
        const u32 dst = lds0 + (u32)(kt % S) * STAGE;
        if (ktail && kt == nk - 1) {
            // last stage of a K that does not fill it: chunks past the row end come from zeros
            static_for<(hi > lo ? hi - lo : 0)>([&](auto I) {
                constexpr int l = lo + decltype(I)::value;
                if constexpr (l < W_ITERS) {
                    const uint8_t *src = wbase + (int64_t)kt * WROW + w_off[l];
                    if (kt * WROW + w_kb[l] >= p.kbytes_w16) src = reinterpret_cast<const uint8_t *>(g_zero16);
                    dma16_ptr(src, dst + l * (NT * 16));
                } else {
                    constexpr int it = l - W_ITERS;
                    const uint8_t *src = xbase + (int64_t)kt * XROW + x_off[it];
                    if (kt * XROW + x_kb[it] >= p.kbytes_x16) src = reinterpret_cast<const uint8_t *>(g_zero16);
                    dma16_ptr(src, dst + WBUF + it * (NT * 16));
                }
            });
        } else {
            const uint8_t *wk = wbase + (int64_t)kt * WROW;
            const uint8_t *xk = xbase + (int64_t)kt * XROW;
            static_for<(hi > lo ? hi - lo : 0)>([&](auto I) {
                constexpr int l = lo + decltype(I)::value;
                if constexpr (l < W_ITERS) dma16(w_off[l], wk, dst + l * (NT * 16));
                else dma16(x_off[l - W_ITERS], xk, dst + WBUF + (l - W_ITERS) * (NT * 16));
            });
        }
    };
    auto issue = [&](int kt) {
        static_for<kParts>([&](auto P) { issue_part(kt, P); });
    };
    // Integer-only epilogue: this lane's share of the tile's comparator references, requested when the last operand
    // load has retired (no hand-counted wait follows), so that it arrives behind the last k-stage.  Requested ahead of
    // the operands it was spilled over the main loop: 12,608 x 768 -> 768 18.8 us, 16.2 without any table.  8-bit operands leave
    // registers for it, and their last k-stage is too short to hide it: there it goes ahead (12,608 rows 19.3 / 18.9).
    constexpr int ABS_ITERS = ABSORBED ? TC * 16 / NT : 1;               // sixteen entries per channel (kAbsRow spreads the banks)
    static_assert(!ABSORBED || TC * 16 % NT == 0, "whole rounds");
    [[maybe_unused]] int abs_ref[ABS_ITERS];
    [[maybe_unused]] auto load_references = [&] {
        if constexpr (ABSORBED) {
            const int nthr = p.ab_nthr;
#pragma unroll
            for (int k = 0; k < ABS_ITERS; ++k) {
                const int i = k * NT + tid, c = i >> 4, e = i & 15;          // entry e of channel c
                const int t = (EPI == kEpiAbsorbed) ? e : 16 * e + 15;       // the reference it holds
                const int ch = min(c0 + c, p.Nout - 1);
                abs_ref[k] = p.ab_thr[(int64_t)ch * nthr + min(t, nthr - 1)];           // (pads: replaced when stored)
            }
        }
    };
    if constexpr (WB == 8 && AB == 8) load_references();
#pragma unroll
    for (int st = 0; st < S - 1; ++st)
        if (st < nk) issue(st);

    // Per-channel epilogue constants, staged once per tile while the first operand loads are in
    // flight: sc = s_x*s_w[c] (the definition's exact product) with the operand factor 2^shift
    // folded in.  The fold is exact unless the result is subnormal; a flag then sends the whole
    // tile through the exact operation sequence.
    if constexpr (ABSORBED) {
        // per channel: the equivalent bias
        if (tid == 0) s_fold_bad[0] = 0;
        for (int c = tid; c < TC; c += NT) reinterpret_cast<int *>(s_raw)[c] = p.ab_bint ? p.ab_bint[min(c0 + c, p.Nout - 1)] : 0;
    } else if constexpr (EPI != kEpiGeneric) {
        if (tid == 0) s_fold_bad[0] = 0;
        __syncthreads();
        for (int c = tid; c < TC; c += NT) {
            const int ch = c0 + c;
            const bool ok = ch < p.Nout;
            const float sw = ok ? p.s_w[p.s_w_per_channel ? ch : 0] : 1.0f;
            const float sc = p.s_x * sw;
            const float folded = ldexpf(sc, -Shift<WB, AB>::value);
            s_scs[c] = folded;
            if constexpr (EPI == kEpiHeadNorm || EPI == kEpiF32) s_raw[c] = sc;
            if constexpr (EPI == kEpiHeadNorm) {
                const bool qk = ch < 2 * p.D;          // V channels have no LayerNorm
                s_hg[c] = qk ? p.hn_gamma[ch] : 0.0f;
                s_hb[c] = qk ? p.hn_beta[ch] : 0.0f;
            }
            s_bs[c] = (ok && p.bias) ? p.bias[ch] : 0.0f;
            if (!(ldexpf(folded, Shift<WB, AB>::value) == sc)) s_fold_bad[0] = 1;
        }
    }

    v16i acc[NC][NTK];
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NTK; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // Byte offsets (inside a stage) of this lane's operand reads.  In sub-step ss the lane owns the
    // 32 values [64*ss + 32*g, +32) of its row: two MFMA operands of 16 values each.
    constexpr int NSS = BK / 64;
    constexpr int WRD = (WB == 8) ? 2 : 1, XRD = (AB == 8) ? 2 : 1;      // 16-byte reads per sub-step
    u32 w_rd[NSS][WRD], x_rd[NSS][XRD];
    {
        const int wrow = wave_c * WC + li, xrow = wave_t * WT + li;
#pragma unroll
        for (int ss = 0; ss < NSS; ++ss) {
            const int wbo = ((ss * 64 + g * 32) * WB) / 8, xbo = ((ss * 64 + g * 32) * AB) / 8;
#pragma unroll
            for (int j = 0; j < WRD; ++j)
                w_rd[ss][j] = (u32)((wrow * WCH + (((wbo >> 4) + j) ^ swz<WCH>(wrow))) * 16 + (wbo & 15));
#pragma unroll
            for (int j = 0; j < XRD; ++j)
                x_rd[ss][j] = (u32)(WBUF + (xrow * XCH + (((xbo >> 4) + j) ^ swz<XCH>(xrow))) * 16 + (xbo & 15));
        }
    }
    // ---- main loop, software-pipelined by hand -------------------------------------------------
    // A k-stage is NSS sub-steps of 64 values; a sub-step is two MFMA steps s = 0, 1 of 32 values.
    // Per sub-step a lane fetches one packed piece per operand block ("raw": 32 values each) and
    // unpacks half of it per MFMA step into int8 fragments ("frag").  Fragments are double
    // buffered: while the NC*NTK MFMAs of one step run on one set, the VALU fills the other set,
    // and the LDS reads of the next sub-step are issued as soon as the current raw registers have
    // been unpacked, so their latency hides behind the MFMAs that follow.  The wait for the next
    // k-stage, the workgroup barrier and the issue of the stage after it sit in the middle of the
    // last sub-step (not between k-steps), where the matrix pipe still holds queued work.
    constexpr int WRAW = WB, XRAW = AB;                           // dwords of raw data per lane, block and sub-step
    u32 wr[NC][WRAW], xr[NTK][XRAW];
    v4i wf[2][NC], xf[2][NTK];
    auto load_raw = [&](int buf, auto SS) {
        constexpr int ss = decltype(SS)::value;
        const uint8_t *stage = smem + buf * STAGE;
#pragma unroll
        for (int ci = 0; ci < NC; ++ci) {
            const uint8_t *src = stage + w_rd[ss][0] + ci * 32 * WROW;
            if constexpr (WB == 4) {
                uint4 v = *reinterpret_cast<const uint4 *>(src);
                wr[ci][0] = v.x; wr[ci][1] = v.y; wr[ci][2] = v.z; wr[ci][3] = v.w;
            } else if constexpr (WB == 2) {
                uint2 v = *reinterpret_cast<const uint2 *>(src);
                wr[ci][0] = v.x; wr[ci][1] = v.y;
            } else {
                uint4 v0 = *reinterpret_cast<const uint4 *>(src);
                uint4 v1 = *reinterpret_cast<const uint4 *>(stage + w_rd[ss][WRD - 1] + ci * 32 * WROW);
                wr[ci][0] = v0.x; wr[ci][1] = v0.y; wr[ci][2] = v0.z; wr[ci][3] = v0.w;
                wr[ci][4] = v1.x; wr[ci][5] = v1.y; wr[ci][6] = v1.z; wr[ci][7] = v1.w;
            }
        }
#pragma unroll
        for (int ti = 0; ti < NTK; ++ti) {
            const uint4 v = *reinterpret_cast<const uint4 *>(stage + x_rd[ss][0] + ti * 32 * XROW);
            xr[ti][0] = v.x; xr[ti][1] = v.y; xr[ti][2] = v.z; xr[ti][3] = v.w;
        }
    };
    // raw -> fragment set `fb` for MFMA step s of the current sub-step
    auto unpack = [&](auto S_, auto FB) {
        constexpr int s = decltype(S_)::value, fb = decltype(FB)::value;
#pragma unroll
        for (int ci = 0; ci < NC; ++ci) {
            if constexpr (WB == 4) wf[fb][ci] = unpack4_x16(wr[ci][2 * s], wr[ci][2 * s + 1]);
            else if constexpr (WB == 2) wf[fb][ci] = unpack2_x64(wr[ci][s]);
            else { wf[fb][ci][0] = (int)wr[ci][4 * s]; wf[fb][ci][1] = (int)wr[ci][4 * s + 1];
                   wf[fb][ci][2] = (int)wr[ci][4 * s + 2]; wf[fb][ci][3] = (int)wr[ci][4 * s + 3]; }
        }
#pragma unroll
        for (int ti = 0; ti < NTK; ++ti) {
            if constexpr (WB == 2) xf[fb][ti] = unpack4_x16_order2(xr[ti][2 * s], xr[ti][2 * s + 1]);
            else xf[fb][ti] = unpack4_x16(xr[ti][2 * s], xr[ti][2 * s + 1]);
        }
    };
    auto mma = [&](auto FB) {
        constexpr int fb = decltype(FB)::value;
#pragma unroll
        for (int ci = 0; ci < NC; ++ci)
#pragma unroll
            for (int ti = 0; ti < NTK; ++ti) {
                if constexpr (SWAP)
                    acc[ci][ti] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xf[fb][ti], wf[fb][ci], acc[ci][ti], 0, 0, 0);
                else
                    acc[ci][ti] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[fb][ci], xf[fb][ti], acc[ci][ti], 0, 0, 0);
            }
    };
    // Interleave pattern of one MFMA step: NC*NTK matrix instructions with the unpack arithmetic of
    // the next step spread evenly between them (then, where given, the LDS reads of the next sub-step).
    constexpr int kMma = NC * NTK;
    constexpr int kUnpackOps = (WB == 8 ? 0 : (WB == 4 ? 6 : 7) * NC) + (WB == 2 ? 10 : 6) * NTK;
    constexpr int kValuPerMma = (kUnpackOps + kMma - 1) / kMma;
    constexpr int kRawReads = NC * WRD + NTK * XRD;
    auto pattern = [&](bool reads_after) {
#pragma unroll
        for (int i = 0; i < kMma; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                 // one MFMA
            if (kValuPerMma > 0) __builtin_amdgcn_sched_group_barrier(0x002, kValuPerMma, 0);   // its share of VALU
        }
        if (reads_after) __builtin_amdgcn_sched_group_barrier(0x100, kRawReads, 0);              // DS reads
    };
    // Stage j is complete once all but the loads of the (at most S-2) younger stages have retired;
    // the barrier then also tells that every wave has finished reading stage j-1, whose buffer the
    // next issue overwrites.
    auto sync_stage = [&](int j) {
        const int younger = nk - 1 - j;
        if (younger >= S - 2) wait_vmcnt<(S - 2) * LOADS>();
        else if (younger == 1) wait_vmcnt<LOADS>();
        else wait_vmcnt<0>();
        __syncthreads();
        if (j + S - 1 < nk) {
            if (j == 0) issue(j + S - 1);
            else issue_part(j + S - 1, std::integral_constant<int, 0>{});
        }
    };
    // The fragments of a set are made "used" at the end of the step that fills them, so the
    // compiler cannot sink their arithmetic past the branches of the synchronisation code (where
    // it would no longer overlap with any MFMA).
    auto pin = [&](auto FB) {
        constexpr int fb = decltype(FB)::value;
        pin_frags(wf[fb]);
        pin_frags(xf[fb]);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    if constexpr (AB == 4) {
    sync_stage(0);
    load_raw(0, I0{});
    unpack(I0{}, I0{});
    // One k-stage.  NEXT: another stage follows (its synchronisation, the issue of a later stage and
    // the first raw reads of the next stage are part of this one); the last stage is a separate
    // instantiation, so that neither copy carries a branch between an MFMA step and its unpacking.
    auto kstep = [&](int kt, auto NEXT_) {
        constexpr bool NEXT = decltype(NEXT_)::value;
        const int buf = kt % S;
        static_for<NSS>([&](auto SS) {
            constexpr int ss = decltype(SS)::value;
            constexpr bool last_ss = (ss + 1 == NSS);
            // the rest of the stage whose first loads followed the previous synchronisation
            // (a stage's groups must enter the load queue in order and ahead of the next stage's first
            // group, which the synchronisation below issues: the waits count loads from the youngest.
            // With a single sub-step per stage that leaves no later slot for the last group.)
            if constexpr (ss == 0) {
                if (kt >= 1 && kt + S - 1 < nk) {
                    issue_part(kt + S - 1, I1{});
                    if constexpr (NSS == 1) issue_part(kt + S - 1, std::integral_constant<int, 2>{});
                }
            }
            // step s = 0 runs; step s = 1 is unpacked; then the raw registers are free
            __builtin_amdgcn_sched_barrier(0);
            mma(I0{});
            unpack(I1{}, I1{});
            if constexpr (!last_ss) {
                load_raw(buf, std::integral_constant<int, (last_ss ? 0 : ss + 1)>{});
                pattern(true);
                pin(I1{});
                __builtin_amdgcn_sched_barrier(0);
            } else {
                pattern(false);
                pin(I1{});
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (NEXT) {
                    sync_stage(kt + 1);
                    load_raw((kt + 1) % S, I0{});
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if constexpr (ss == 0 && NSS > 1) {
                if (kt >= 1 && kt + S - 1 < nk) issue_part(kt + S - 1, std::integral_constant<int, 2>{});
                __builtin_amdgcn_sched_barrier(0);
            }
            // step s = 1 runs; step s = 0 of the next sub-step is unpacked
            mma(I1{});
            if constexpr (!last_ss || NEXT) {
                unpack(I0{}, I0{});
                pattern(false);
                pin(I0{});
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    for (int kt = 0; kt < nk - 1; ++kt) kstep(kt, std::true_type{});
    load_references();
    kstep(nk - 1, std::false_type{});
    } else {
        // 8-bit operands need no unpacking: a step of 32 values is one 16-byte read per operand block,
        // straight into the fragment set that the next step's matrix instructions take.
        constexpr int NST = BK / 32;
        auto read_step = [&](int buf, auto ST, auto FB) {
            constexpr int ss = decltype(ST)::value / 2, j = decltype(ST)::value % 2, fb = decltype(FB)::value;
            const uint8_t *stage = smem + buf * STAGE;
#pragma unroll
            for (int ci = 0; ci < NC; ++ci) wf[fb][ci] = *reinterpret_cast<const v4i *>(stage + w_rd[ss][j % WRD] + ci * 32 * WROW);
#pragma unroll
            for (int ti = 0; ti < NTK; ++ti) xf[fb][ti] = *reinterpret_cast<const v4i *>(stage + x_rd[ss][j % XRD] + ti * 32 * XROW);
        };
        auto steps = [&](int kt, auto NEXT_) {
            constexpr bool NEXT = decltype(NEXT_)::value;
            static_for<NST>([&](auto ST) {
                constexpr int st = decltype(ST)::value, fb = st & 1;
                using FB = std::integral_constant<int, fb>;
                using OTHER = std::integral_constant<int, fb ^ 1>;
                constexpr bool more = st + 1 < NST;
                pin(FB{});
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (st == 0) {
                    if (kt >= 1 && kt + S - 1 < nk) {
                        issue_part(kt + S - 1, I1{});
                        if constexpr (NST == 2) issue_part(kt + S - 1, std::integral_constant<int, 2>{});
                    }
                }
                if constexpr (st == 1 && NST > 2) {
                    if (kt >= 1 && kt + S - 1 < nk) issue_part(kt + S - 1, std::integral_constant<int, 2>{});
                }
                if constexpr (!more && NEXT) sync_stage(kt + 1);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (more) read_step(kt % S, std::integral_constant<int, (more ? st + 1 : 0)>{}, OTHER{});
                else if constexpr (NEXT) read_step((kt + 1) % S, I0{}, OTHER{});
                mma(FB{});
#pragma unroll
                for (int i = 0; i < kMma; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if constexpr (more || NEXT) __builtin_amdgcn_sched_group_barrier(0x100, (NC + NTK + kMma - 1) / kMma, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        sync_stage(0);
        read_step(0, I0{}, I0{});
        for (int kt = 0; kt < nk - 1; ++kt) steps(kt, std::true_type{});
        steps(nk - 1, std::false_type{});
    }
    __syncthreads();


    // ---- epilogue -------------------------------------------------------------------------
    constexpr int shift = Shift<WB, AB>::value;
    const bool fold_ok = (EPI != kEpiGeneric && !ABSORBED) && (s_fold_bad[0] == 0);
    if constexpr (SWAP) {
        // Blocks in turn; the residual of the next block is requested before the current block is
        // stored, so its loads never queue behind those stores.
        auto block_pos = [&](int b, int &m0, int &cl) {
            const int ci = b / NTK, ti = b % NTK;
            cl = wave_c * WC + ci * 32 + li;               // this lane's channel inside the tile
            m0 = t0 + wave_t * WT + ti * 32 + 4 * g;
        };
        auto run = [&](auto FULLT, auto REST) {
            constexpr bool FULL = decltype(FULLT)::value, RES = decltype(REST)::value;
            float rbuf[2][16];                 // residual of the current / the next block
#pragma unroll
            for (int r = 0; r < 16; ++r) rbuf[0][r] = rbuf[1][r] = 0.0f;
            if constexpr (RES) {
                int m0, cl;
                block_pos(0, m0, cl);
                load_residual<FULL>(p, m0, c0 + cl, rbuf[0]);
            }
            static_for<NC * NTK>([&](auto BI) {
                constexpr int b = decltype(BI)::value;
                int m0, cl;
                if constexpr (RES && b + 1 < NC * NTK) {
                    block_pos(b + 1, m0, cl);
                    load_residual<FULL>(p, m0, c0 + cl, rbuf[(b + 1) & 1]);
                }
                block_pos(b, m0, cl);
                epilogue_f32<FULL, RES>(p, acc[b / NTK][b % NTK], fold_ok ? 0 : shift, m0, c0 + cl,
                                        fold_ok ? s_scs[cl] : s_raw[cl], s_bs[cl], rbuf[b & 1]);
            });
        };
        // tiles wholly inside the matrix (all but the last row / column of tiles) skip the bounds tests
        const bool full = t0 + TT <= p.M && c0 + TC <= p.Nout;
        if (p.res) { if (full) run(std::true_type{}, std::true_type{}); else run(std::false_type{}, std::true_type{}); }
        else { if (full) run(std::true_type{}, std::false_type{}); else run(std::false_type{}, std::false_type{}); }
    } else {
        if constexpr (EPI == kEpiHeadNorm) {
            // Q and K tiles: per-head LayerNorm quantizer; V tiles fall through to the plain one
            const int cbw = c0 + wave_c * WC;                       // the wave's head starts here
            if (cbw < 2 * p.D) {
                static_assert(EPI != kEpiHeadNorm || (NC == 2 && NTK % 2 == 0 && WC == 64), "one head per wave");
                int which;
                const int64_t ch_part = packed_channel_part(p, cbw, which);
                const float step = which == 0 ? p.s_y[0] : p.s_y[1];
                // folded scales unless folding was inexact somewhere in the tile: then the plain
                // ones (kept behind the flag word) and the explicit shift
                const float *sc64 = (fold_ok ? s_scs : s_raw) + wave_c * WC;
                const int sh = fold_ok ? 0 : shift;
                if constexpr (EPI == kEpiHeadNorm) {
                    float *tmp = reinterpret_cast<float *>(smem) + wave * 4096 + lane;
                    static_for<NTK / 2>([&](auto PI) {
                        constexpr int pair = decltype(PI)::value;
                        const int64_t tk = packed_token_part(p, t0 + wave_t * WT + 64 * pair + 32 * g + li);
                        uint8_t *dst = (ch_part >= 0 && tk >= 0) ? p.yq + tk + ch_part : nullptr;
                        if (p.yq_sb == 4)
                            epilogue_headnorm<4, NTK, pair>(p, acc, sh, dst, sc64, s_bs + wave_c * WC, step, s_hg + wave_c * WC, s_hb + wave_c * WC, tmp);
                        else
                            epilogue_headnorm<8, NTK, pair>(p, acc, sh, dst, sc64, s_bs + wave_c * WC, step, s_hg + wave_c * WC, s_hb + wave_c * WC, tmp);
                    });
                }
                return;
            }
        }
        if constexpr (ABSORBED) {
            // The pipeline buffers are free now: the tile's LDS table (see epilogue_absorbed) goes there.
            const int nthr = p.ab_nthr;
            constexpr bool in_lds = (EPI == kEpiAbsorbed);
            int *s_tbl = reinterpret_cast<int *>(smem);
            static_assert(TC * kAbsRow * 4 <= S * STAGE, "reference table exceeds the pipeline buffers");
#pragma unroll
            for (int k = 0; k < ABS_ITERS; ++k) {
                const int i = k * NT + tid, c = i >> 4, e = i & 15;
                const int t = in_lds ? e : 16 * e + 15;
                s_tbl[c * kAbsRow + e] = t >= nthr ? INT32_MAX : absorbed_reference<WB, AB>(abs_ref[k], reinterpret_cast<const int *>(s_raw)[c]);
            }
            __syncthreads();
            if constexpr (in_lds) {
                // Are they evenly spaced, as epilogue_absorbed_even needs?  Relative to the bias they have to stay within 22 bits
                // (20 with an operand factor above 2^8), the spacing to be 4 or more and each of them within 3/8
                // of it.  (A sum below 2^24 is exact in fp32 and a larger one beyond every reference.  A sum's place, in
                // spacings from the first reference, has to be right within 1/2 - 3/8 = 1/8.  Its offset -T[0] / spacing is at
                // most 2^22 / 4 in size, so rounding it moves the place by up to 2^-4 [2^-5 below 2^20]; the roundings of
                // the spacing's reciprocal and of the quotient add less than 2^-16.  A closer spacing or a farther reach
                // needs that 2^-4 counted again.)
                // Four neighbouring lanes look at a channel's row here, where it is in LDS.  One lane per channel, reading the caller's
                // table ahead of the main loop, held every tile up, and one that is not even had nothing for it.  12,608 x 768 ->
                // 768, us, no look / that one / this one: references at random 19.1 / 21.1 / 17.4, even ones - / 16.4 / 15.0;
                // 197 rows 12.6 / 14.6 / 11.1 and - / 10.7 / 9.2; 8-bit operands 20.2 / 22.9 / 20.4 and - / 19.5 / 18.1.
                static_assert(4 * TC % NT == 0, "whole groups of four lanes");
                constexpr int reach = 1 << (shift > 8 ? 20 : 22);
#pragma unroll
                for (int it = 0; it < 4 * TC / NT; ++it) {
                    const int c = (it * NT + tid) >> 2;
                    const int at = min(4 * (tid & 3), max(nthr - 4, 0));           // this lane's four (the last ones overlap)
                    int ref[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) ref[e] = s_tbl[c * kAbsRow + min(at + e, nthr - 1)];
                    const int low = __builtin_amdgcn_mov_dpp(ref[0], 0x00, 0xF, 0xF, true);      // of the group's first lane
                    const int high = __builtin_amdgcn_mov_dpp(ref[3], 0xFF, 0xF, 0xF, true);     // and its last
                    const int width = (int)((u32)high - (u32)low);       // (wraps only where low or high are out of reach)
                    const float inv = (float)(nthr - 1) * __builtin_amdgcn_rcpf((float)width);
                    bool ok = low > -(reach << shift) && high < (reach << shift) && width >= ((4 * (nthr - 1)) << shift);
#pragma unroll
                    for (int e = 0; e < 4; ++e)                                    // (one reference: not a number)
                        ok = ok & (fabsf((float)(int)((u32)ref[e] - (u32)low) * inv - (float)min(at + e, nthr - 1)) <= 0.375f);
                    if (!ok) s_fold_bad[0] = 1;
                    if ((tid & 3) == 0) {
                        s_scs[c] = inv;
                        s_bs[c] = fmaf(-(float)low, inv, 0.5f);
                    }
                }
                __syncthreads();
            }
            const bool even = in_lds && s_fold_bad[0] == 0;
            int64_t tok_part[NTK];
#pragma unroll
            for (int ti = 0; ti < NTK; ++ti) tok_part[ti] = packed_token_part(p, t0 + wave_t * WT + ti * 32 + li);
            static_for<NC>([&](auto CI) {
                constexpr int ci = decltype(CI)::value;
                const int cl = wave_c * WC + ci * 32 + 16 * g;
                const int cb = c0 + cl;
                int which;
                const int64_t ch_part = packed_channel_part(p, cb, which);
                const int *bint = reinterpret_cast<const int *>(s_raw) + cl;
                static_for<NTK>([&](auto TI) {
                    constexpr int ti = decltype(TI)::value;
                    uint8_t *dst = (ch_part >= 0 && tok_part[ti] >= 0) ? p.yq + tok_part[ti] + ch_part : nullptr;
                    if (cb >= p.Nout)
                        store_zero_group(p, dst);
                    else if (even)
                        epilogue_absorbed_even(p, acc[ci][ti], dst, s_tbl + cl * kAbsRow, s_scs + cl, s_bs + cl);
                    else
                        epilogue_absorbed<in_lds>(p, acc[ci][ti], shift, dst, s_tbl + cl * kAbsRow,
                                                  p.ab_thr + (int64_t)min(cb, p.Nout - 16) * nthr, nthr, bint);
                });
            });
            return;
        }
        constexpr bool QUANT = (EPI == kEpiQuant || EPI == kEpiQuantGelu || EPI == kEpiHeadNorm);
        int64_t tok_part[NTK];
        if constexpr (QUANT) {
#pragma unroll
            for (int ti = 0; ti < NTK; ++ti)
                tok_part[ti] = packed_token_part(p, t0 + wave_t * WT + ti * 32 + li);
        }
        static_for<NC>([&](auto CI) {
            constexpr int ci = decltype(CI)::value;
            const int cl = wave_c * WC + ci * 32 + 16 * g;     // channel offset inside the tile
            const int cb = c0 + cl;
            int64_t ch_part = -1;
            float s_y = 1.0f, r_y = 1.0f;
            if constexpr (EPI != kEpiGeneric) {
                int which;
                ch_part = packed_channel_part(p, cb, which);
                const float sy0 = p.s_y[0], sy1 = p.s_y[1], sy2 = p.s_y[2];
                const float ry0 = p.r_y[0], ry1 = p.r_y[1], ry2 = p.r_y[2];
                s_y = which == 0 ? sy0 : (which == 1 ? sy1 : sy2);
                r_y = which == 0 ? ry0 : (which == 1 ? ry1 : ry2);
            }
            static_for<NTK>([&](auto TI) {
                constexpr int ti = decltype(TI)::value;
                if constexpr (QUANT) {
                    uint8_t *dst = (ch_part >= 0 && tok_part[ti] >= 0) ? p.yq + tok_part[ti] + ch_part : nullptr;
                    if (cb >= p.Nout) store_zero_group(p, dst);
                    else epilogue_quant<EPI == kEpiQuantGelu>(p, acc[ci][ti], shift, dst, s_y, r_y, cb, s_scs + cl, s_bs + cl, !fold_ok);
                } else {
                    const int m = t0 + wave_t * WT + ti * 32 + li;
                    epilogue_generic(p, acc[ci][ti], shift, m, cb);
                }
            });
        });
    }
}

// ---- few tokens: the contraction split over the waves of a workgroup ---------------------------
// One image through a 768-wide linear is 6 to 18 tiles of the kernel above: a handful of the 256 CUs
// walk all of K in turn, each stage a round trip to L2 that nothing hides.  What bounds such a call is
// that chain, so here a workgroup owns one 32x32 block and its waves share K, 64 values per step, each
// loading its operand pieces straight from L2 into registers (no LDS stage, no barrier in the loop;
// kSplitUnroll steps requested ahead).  The int32 partial sums meet in LDS -- integer addition, so the
// split changes no result -- and wave 0 runs the epilogue on the sum.
constexpr int kSplitUnroll = 4;
constexpr int kSplitMaxWaves = 8;

template <int WB, int AB, int EPI>
__global__ __launch_bounds__(kSplitMaxWaves * 64)
void gemm_split_kernel(GemmParams p) {
    static_assert(EPI == kEpiGeneric || EPI == kEpiF32 || EPI == kEpiQuant || EPI == kEpiQuantGelu, "epilogues");
    constexpr bool SWAP = (EPI == kEpiF32);
    constexpr int WBY = 32 * WB / 8, XBY = 32 * AB / 8;       // bytes of a lane's 32 values of a step
    constexpr int WDW = WBY / 4, XDW = XBY / 4;
    __shared__ int4 s_part[kSplitMaxWaves - 1][4][64];
    __shared__ __attribute__((aligned(16))) float s_scs[32], s_bs[32];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int li = lane & 31, g = lane >> 5;
    const int n_ct = (p.Nout + 31) / 32;
    const int ct = blockIdx.x % n_ct;
    const int c0 = ct * 32, t0 = (blockIdx.x / n_ct) * 32;

    // wave 0 requests what its epilogue needs ahead of the operands
    float sc = 1.0f, bs = 0.0f;
    float rv[16];
    const int m0 = t0 + 4 * g;                                // first token of this lane in the fp32 epilogue
    const bool full = t0 + 32 <= p.M && c0 + 32 <= p.Nout;
    if constexpr (EPI != kEpiGeneric) {
        if (wave == 0) {
            const int ch = c0 + li;
            if (ch < p.Nout) {
                sc = p.s_x * p.s_w[p.s_w_per_channel ? ch : 0];
                if (p.bias) bs = p.bias[ch];
            }
            if constexpr (EPI == kEpiF32) {
                if (p.res) {
                    if (full) load_residual<true>(p, m0, c0 + li, rv);
                    else load_residual<false>(p, m0, c0 + li, rv);
                }
            }
        }
    }

    // this lane's operand rows (rows beyond the matrix are clamped: their products are never stored)
    const uint8_t *wrow = p.w + (int64_t)min(c0 + (SWAP ? li : channel_of_slot(li)), p.Nout - 1) * p.w_stride;
    const uint8_t *xrow = p.x + (int64_t)min(t0 + li, p.M - 1) * p.x_stride;
    const int steps = (p.K + 63) / 64;
    v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
    for (int j0 = wave; j0 < steps; j0 += waves * kSplitUnroll) {
        u32 wr[kSplitUnroll][WDW], xr[kSplitUnroll][XDW];
#pragma unroll
        for (int u = 0; u < kSplitUnroll; ++u) {
            const int j = j0 + u * waves;
            // 16-byte pieces (8 bytes of 2-bit weights) past the end of a row, or of a step past the
            // last one, are read from sixteen zero bytes
#pragma unroll
            for (int q = 0; q < (WBY + 15) / 16; ++q) {
                const int off = j * (2 * WBY) + g * WBY + 16 * q;
                const uint8_t *src = (off < p.kbytes_w16) ? wrow + off : reinterpret_cast<const uint8_t *>(g_zero16);
                if constexpr (WB == 2) {
                    const uint2 v = *reinterpret_cast<const uint2 *>(src);
                    wr[u][0] = v.x; wr[u][1] = v.y;
                } else {
                    const uint4 v = *reinterpret_cast<const uint4 *>(src);
                    wr[u][4 * q] = v.x; wr[u][4 * q + 1] = v.y; wr[u][4 * q + 2] = v.z; wr[u][4 * q + 3] = v.w;
                }
            }
#pragma unroll
            for (int q = 0; q < XBY / 16; ++q) {
                const int off = j * (2 * XBY) + g * XBY + 16 * q;
                const uint8_t *src = (off < p.kbytes_x16) ? xrow + off : reinterpret_cast<const uint8_t *>(g_zero16);
                const uint4 v = *reinterpret_cast<const uint4 *>(src);
                xr[u][4 * q] = v.x; xr[u][4 * q + 1] = v.y; xr[u][4 * q + 2] = v.z; xr[u][4 * q + 3] = v.w;
            }
        }
        static_for<kSplitUnroll>([&](auto U) {
            constexpr int u = decltype(U)::value;
            static_for<2>([&](auto S_) {
                constexpr int s = decltype(S_)::value;
                v4i wf, xf;
                if constexpr (WB == 4) wf = unpack4_x16(wr[u][2 * s], wr[u][2 * s + 1]);
                else if constexpr (WB == 2) wf = unpack2_x64(wr[u][s]);
                else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) wf[i] = (int)wr[u][4 * s + i];
                }
                if constexpr (AB == 4) {
                    if constexpr (WB == 2) xf = unpack4_x16_order2(xr[u][2 * s], xr[u][2 * s + 1]);
                    else xf = unpack4_x16(xr[u][2 * s], xr[u][2 * s + 1]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) xf[i] = (int)xr[u][4 * s + i];
                }
                if constexpr (SWAP) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(xf, wf, acc, 0, 0, 0);
                else acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf, xf, acc, 0, 0, 0);
            });
        });
    }

    if (wave > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            s_part[wave - 1][q][lane] = make_int4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    }
    constexpr int shift = Shift<WB, AB>::value;
    const float folded = ldexpf(sc, -shift);
    const bool fold_ok = __builtin_amdgcn_ballot_w64(!(ldexpf(folded, shift) == sc)) == 0;
    if (EPI != kEpiGeneric && wave == 0 && g == 0) { s_scs[li] = folded; s_bs[li] = bs; }
    __syncthreads();
    if (wave > 0) return;
    for (int w = 0; w < waves - 1; ++w) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int4 v = s_part[w][q][lane];
            acc[4 * q] += v.x; acc[4 * q + 1] += v.y; acc[4 * q + 2] += v.z; acc[4 * q + 3] += v.w;
        }
    }

    if constexpr (EPI == kEpiF32) {
        const float scale = fold_ok ? folded : sc;
        const int sh = fold_ok ? 0 : shift;
        if (p.res) {
            if (full) epilogue_f32<true, true>(p, acc, sh, m0, c0 + li, scale, bs, rv);
            else epilogue_f32<false, true>(p, acc, sh, m0, c0 + li, scale, bs, rv);
        } else {
            if (full) epilogue_f32<true, false>(p, acc, sh, m0, c0 + li, scale, bs, rv);
            else epilogue_f32<false, false>(p, acc, sh, m0, c0 + li, scale, bs, rv);
        }
    } else {
        // the lane's sixteen channels (32 four- or eight-bit channels are whole 16-byte units, so the
        // blocks also cover every padding byte of a packed row)
        const int cb = c0 + 16 * g, m = t0 + li;
        if constexpr (EPI == kEpiGeneric) {
            epilogue_generic(p, acc, shift, m, cb);
        } else {
            int which;
            uint8_t *dst = packed_dst(p, m, cb, which);
            const float sy0 = p.s_y[0], sy1 = p.s_y[1], sy2 = p.s_y[2];
            const float ry0 = p.r_y[0], ry1 = p.r_y[1], ry2 = p.r_y[2];
            const float s_y = which == 0 ? sy0 : (which == 1 ? sy1 : sy2);
            const float r_y = which == 0 ? ry0 : (which == 1 ? ry1 : ry2);
            if (cb >= p.Nout) store_zero_group(p, dst);
            else epilogue_quant<EPI == kEpiQuantGelu>(p, acc, shift, dst, s_y, r_y, cb, s_scs + 16 * g, s_bs + 16 * g, !fold_ok);
        }
    }
}

template <int WB, int AB>
hipError_t launch_split(const GemmParams &p, int epi, hipStream_t stream) {
    const int64_t blocks = (int64_t)((p.Nout + 31) / 32) * ((p.M + 31) / 32);
    const int steps = (p.K + 63) / 64;
    // A wave always computes whole rounds of kSplitUnroll steps (a missing one on zeros): as few rounds as
    // eight waves need, then no more waves than those rounds fill.  With four or eight waves for every K,
    // K 256 wasted three quarters of the work and K 1536 and 3072 one: 8 bits, 788 x 256 -> 768 6.9 -> 5.6 us,
    // 788 x 3072 -> 768 22.1 -> 20.4; 4 bits 985 x 384 -> 1024 5.8 -> 4.8 (fp32 out).
    const int rounds = (steps + kSplitMaxWaves * kSplitUnroll - 1) / (kSplitMaxWaves * kSplitUnroll);
    const int waves = (steps + rounds * kSplitUnroll - 1) / (rounds * kSplitUnroll);
    const dim3 grid((unsigned)blocks), block((unsigned)waves * 64);
    switch (epi) {
        case kEpiF32: hipLaunchKernelGGL((gemm_split_kernel<WB, AB, kEpiF32>), grid, block, 0, stream, p); break;
        case kEpiQuant: hipLaunchKernelGGL((gemm_split_kernel<WB, AB, kEpiQuant>), grid, block, 0, stream, p); break;
        case kEpiQuantGelu: hipLaunchKernelGGL((gemm_split_kernel<WB, AB, kEpiQuantGelu>), grid, block, 0, stream, p); break;
        default: hipLaunchKernelGGL((gemm_split_kernel<WB, AB, kEpiGeneric>), grid, block, 0, stream, p); break;
    }
    return hipGetLastError();
}

template <int WB, int AB, int TC, int TT, int WAVES_C, int WAVES_T, int BK, int S, int OCC, int EPI>
hipError_t launch(const GemmParams &p, hipStream_t stream) {
    constexpr size_t lds = pipeline_lds<EPI, WAVES_C * WAVES_T, S * (TC * (BK * WB / 8) + TT * (BK * AB / 8))> + 2 * TC * sizeof(float) + 16 +
                           ((EPI == kEpiHeadNorm || EPI == kEpiF32 || EPI == kEpiAbsorbed || EPI == kEpiAbsorbedBig) ? TC * sizeof(float) : 0) +
                           (EPI == kEpiHeadNorm ? 2 * TC * sizeof(float) : 0);
    auto kern = gemm_kernel<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, EPI>;
    if (lds > 48 * 1024) {
        static std::atomic<uint64_t> allowed{0};        // (one per instantiation)
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, allowed);
        if (e != hipSuccess) return e;
    }
    const int n_ct = (p.Nout + TC - 1) / TC;
    const int n_tt = (p.M + TT - 1) / TT;
    const int64_t blocks = (int64_t)n_ct * n_tt;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(WAVES_C * WAVES_T * 64), lds, stream, p);
    return hipGetLastError();
}

// the epilogues with one output and whole 16-channel groups (fp32: any width)
template <int WB, int AB, int TC, int TT, int WAVES_C, int WAVES_T, int BK, int S, int OCC>
hipError_t launch_main(const GemmParams &p, int epi, hipStream_t stream) {
    constexpr bool kGelu = !(WB == 4 && AB == 4 && TT == 256);      // (4-bit pairs with GELU: small_tile)
    if (epi == kEpiF32) return launch<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, kEpiF32>(p, stream);
    if (epi == kEpiQuant) return launch<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, kEpiQuant>(p, stream);
    if constexpr (kGelu) {
        if (epi == kEpiQuantGelu) return launch<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, kEpiQuantGelu>(p, stream);
    }
    return hipErrorInvalidValue;
}

template <int WB, int AB, int TC, int TT, int WAVES_C, int WAVES_T, int BK, int S, int OCC>
hipError_t launch_epi(const GemmParams &p, int epi, hipStream_t stream) {
    switch (epi) {
        case kEpiF32: case kEpiQuant: case kEpiQuantGelu:
            return launch_main<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC>(p, epi, stream);
        case kEpiHeadNorm: {
            // this epilogue keeps a token's whole 64-channel head in registers on top of the
            // accumulators: it runs with two waves per SIMD (256 registers) on 64x128 wave tiles
            constexpr int stage = 128 * BK * WB / 8 + 256 * BK * AB / 8;
            constexpr int S_HN = (3 * stage <= 80 * 1024) ? 3 : 2;
            return launch<WB, AB, 128, 256, 2, 2, BK, S_HN, 2, kEpiHeadNorm>(p, stream);
        }
        case kEpiAbsorbed: case kEpiAbsorbedBig:
            if constexpr (WB == 8 && AB == 4) return hipErrorInvalidValue;       // (expanded weights: the other epilogues' calls only)
            else if (epi == kEpiAbsorbed) return launch<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, kEpiAbsorbed>(p, stream);
            else return launch<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, kEpiAbsorbedBig>(p, stream);
        default: return launch<WB, AB, TC, TT, WAVES_C, WAVES_T, BK, S, OCC, kEpiGeneric>(p, stream);
    }
}

// Does the call go to the split-contraction kernel?  It re-reads each operand row once per 32x32 block
// (from L2), so its time grows with the number of blocks, while the tiled kernels' stays at one walk of
// K until their tiles fill the chip.  The tiled kernel's time over the split one's, fp32 out / requantized
// (788 to 1,576 rows; 32 rows and more channels, or 32 channels, are ahead by more in fp32, by less packed):
//             500 blocks   800          992          1184         1500
//   4 bits  K  384  1.45 / 1.57  1.36 / 1.47  1.44 / 1.40  1.20 / 1.32  1.07 / 0.92
//           K 1024  1.65 / 1.65  1.20 / 1.28  1.23 / 1.22  1.00 / 1.09  0.94 / 0.91
//           K 3072  1.90 / 1.84  1.15 / 1.20  1.14 / 1.14  0.87 / 0.91  0.84 / 0.77
//   2 bits  K 1024  1.67 / 1.70  1.27 / 1.38  1.27 / 1.27  1.03 / 1.09  0.97 / 1.03
//             500 blocks   600          800          992
//   8 bits  K  384  1.26 / 1.55  1.12 / 1.39  1.00 / 1.26  1.01 / 1.20
//           K 1024  1.44 / 1.62  1.16 / 1.31  0.97 / 1.15  0.97 / 1.10
//           K 4096  1.65 / 1.56  1.20 / 1.16  0.94 / 0.97  0.88 / 0.89
// Eight-bit operands too large for the caches stream from HBM, where the long row pieces of the tiled
// kernel are read faster once every CU has two blocks: 32 x 16,384 -> 22,400 (700 blocks) 115 us tiled,
// 171 split; 32 x 16,384 -> 16,000 (500) 1.2 times ahead as above.
bool use_split(const GemmParams &p, int wb, int ab, int epi) {
    if (!((wb == 4 && ab == 4) || (wb == 2 && ab == 4) || (wb == 8 && ab == 8))) return false;
    if (epi != kEpiGeneric && epi != kEpiF32 && epi != kEpiQuant && epi != kEpiQuantGelu) return false;
    if (p.yq && p.yq_sb == 2) return false;              // (a 2-bit row's padding can reach past a 32-channel block)
    const int64_t blocks = (int64_t)((p.Nout + 31) / 32) * (((int64_t)p.M + 31) / 32);
    const bool from_hbm = ((int64_t)p.Nout + p.M) * p.K * ab / 8 > (128 << 20);
    return blocks <= (ab == 8 ? (from_hbm ? 512 : 700) : 1000);
}

// 4-bit pairs: 128x128 tiles (four waves, two k-stages, four workgroups per CU) or 128x256 (eight
// waves, three stages, two per CU)?  The time follows the busiest CU, so the smaller tile wins where it
// deals the rows out more evenly (12,608 x 3072 -> 768: 300 large tiles leave two on some CUs and one on
// most, 40.7 us; 594 small ones 34.4), where the tiles do not even fill the chip twice (6,304 rows of
// the same: 26.4 -> 24.8 us; 12,608 x 384 -> 384 9.3 -> 9.0) and with the GELU epilogue, whose arithmetic
// overlaps better with more independent workgroups (50,432 x 768 -> 3072: 166 -> 155 us).  On an even deal
// the larger one reads less (12,608 x 4096 -> 1024 in fp32: 53.9 us against 55.6).
// (Of 129 to 160 rows the larger tile's second half is nearly empty and skips its epilogue, which the deal does
// not see: the several-output epilogue, whose stores weigh most, keeps it there, 129 x 384 -> 20,000 24.1 us against
// 31.5; GELU loses 3 to 18 % past 16,384 channels, too rare a call to build its kernel for that tile.)
// Large fp32 results of a long contraction are bound by their stores, and a deal that saves less than a
// sixteenth does not make up for twice the tiles: 28,368 x 1024 -> 3072 113 us on large tiles, 121 on small
// ones, 44,128 rows 181 and 190 (4096 channels: within 2 % either way).
// The integer-only epilogues gain less from more workgroups beside each other: on an even deal they keep the larger tile (us, large
// / small: 6,304 x 768 -> 768 with 15 references 11.15 / 11.42, 50,432 rows 39.0 / 41.3; with 255 145 / 149) and take the
// smaller one on any other (12,608 x 768 -> 768 with 15 16.6 / 14.7, with 31 44.5 / 36.1, with 255 61.5 / 48.8; 513 x 1024 ->
// 3584 28.6 / 21.2 and 35.6 / 24.9; 25,216 x 1024 -> 3072, 20 units to 19, with 63 217 / 205).  With more than 127
// references, a cache line for each probe, 20 to 19 is too little (304 / 311; 6,304 x 768 -> 3072, 6 to 5, 91.2 / 85.3).
bool small_tile(const GemmParams &p, int epi) {
    constexpr int64_t kCUs = 256;
    const int64_t n_ct = (p.Nout + 127) / 128;
    const int64_t small = n_ct * (((int64_t)p.M + 127) / 128), large = n_ct * (((int64_t)p.M + 255) / 256);
    const int64_t cs = (small + kCUs - 1) / kCUs, cl = 2 * ((large + kCUs - 1) / kCUs);   // 128x128 units of the busiest CU
    if (epi == kEpiAbsorbed || epi == kEpiAbsorbedBig) return p.ab_nthr > 127 ? 16 * cs <= 15 * cl : cs < cl;
    if (epi == kEpiGeneric && p.M > 128 && p.M <= 160) return false;
    if (epi == kEpiF32 && p.K >= 1024 && cl > 16) return false;
    return epi == kEpiQuantGelu || cs < cl || cs <= 2;
}

// 8-bit pairs: which tile?  kSmall: 128x128, 64 values per k-stage, three stages, three workgroups per CU.  kDeep: 128
// values per stage, two stages, two workgroups.  kLarge: 256x256 on sixteen waves, 128 values, two stages, one.  A
// stage of 64 values is half a cache line of every operand row, which L2 then sends twice, and a barrier every eight
// MFMAs of a wave; the larger tile reads half the bytes per product but has no other workgroup beside its epilogue (GELU's
// most of all).  What decides is the busiest CU's work in units of 128x128, times what the form takes per unit.  us of
// kSmall / kDeep / kLarge, outputs fp32 (f), requantized (q), GELU (g), calls repeated until the clock is steady, in
// parentheses the units of the small tiles and of the large one:
//   (1, 4)  5,193 x 1024 -> 1024 q 13.8 / 12.5 / 17 (up to two units kDeep is ahead by 2 to 20 %, by 1 to 7 % behind where K up
//           to 192 does not fill its second stage, 2,247 x 192 -> 2368 q 8.4 / 8.8)
//   (3, 4)  12,608 x 3072 -> 768 f 48.5 / 46.2 / 38.2, q 49.4 / 48.4 / 38.6, g 52.1 / 52.7 / 45.3; K 768 f 18.1 / 19.9 / 16.9,
//           q 17.9 / 18.9 / 16.6, g 22.3 / 23.1 / 24.4; 25,216 x 384 -> 384 f 12.8 / 14.1 / 13.4; x 1536 g 31.6 / 34.2 / 33.9
//   (4, 4)  12,608 x 384 -> 1152 f 18.7 / 17.2 / 16.9, q 17.5 / 17.2 / 15.4, g 23.0 / 23.7 / 23.5
//   (5, 8)  25,216 x 3072 -> 768 f 86.2 / 74.3 / 81.7, q 83.4 / 77.4 / 82.8, g 87.1 / 83.7 / 97.3
//   (7, 8)  6,304 x 1024 -> 4096 q, with its quantizer 51.3 / - / 45.4; 12,608 x 768 -> 2304 f 42.0 / 44.8 / 39.2, q 39.6 / 40.8 / 36.2,
//           g 46.3 / 50.5 / 51.8
//   (10, 12)  12,608 x 768 -> 3072 f 57.1 / 61.6 / 59.6, q 51.3 / 53.3 / 55.0, g 60.9 / 64.0 / 75.1
//   (14, 16)  25,216 x 768 -> 2304 f 89.6 / 90.9 / 79.9, q 74.5 / 75.7 / 73.2, g 85.5 / 90.6 / 98.6; x 384 -> 1152 (7, 8)
//           q 27.3 / 29.9 / 28.3
//   (25, 28)  25,216 x 4096 -> 1024 f 150 / 127 / 113, q 149 / 130 / 111, g 152 / 136 / 123
//   (74, 76)  25,216 x 1024 -> 3072 f 147 / 143 / 121, q 118 / 120 / 107, g 136 / 140 / 142
// Of fp32 results on an even deal of several rounds the stores take most of the time up to K 320 (kSmall / kLarge: 34,763 x 256
// -> 2752, 24 units each, 85.5 / 93.8; 12,856 x 128 -> 3520 38.5 / 39.6; 45,892 x 176 -> 960 41.2 / 44.1; from there on kLarge
// is ahead, 16,384 x 336 -> 4096 90.0 / 76.8), and in two rounds up to 512 where rows are whole cache lines, which kSmall does
// not read twice from L2 (8,992 x 384 -> 3264 35.7 / 40.9, x 512 40.0 / 42.5; x 400 44.1 / 40.7).  GELU of K 2048 and more:
// 30,024 x 2249 -> 1952 255 / 203, 47,258 x 2165 -> 1088 176 / 176, 17,989 x 2166 -> 3488 221 / 182.
// Four units are two even rounds of kDeep and one and a third of kSmall, which a long contraction pays for in full (7,446 x 4096 ->
// 2096 f 99.3 / 85.9, q 95.0 / 73.4; 33,721 x 2048 -> 368 f 55.4 / 50.1); five are three rounds against two, ahead only where
// rows are no whole cache lines (9,239 x 3043 -> 2144 f 120 / 103, q 105 / 91.5; 33,935 x 2432 -> 512 f 73.9 / 79.1).
// A dense kernel that holds the chip for long also holds its clock down for the kernels around it: in the ViT-B block of
// 128 images, calls in a row, kLarge for its QKV linear (14, 16) costs the block 385 -> 406 us and kDeep for its fc2 (5, 8) 400,
// although each saves 1 to 12 us by itself (the attention between them goes from 72 to 77).  The same in blocks of other
// sizes with those units: 43 images of 577 tokens 582 -> 612 and 610, 500 of 50 393 -> 411 and 407, 128 of 198 387 -> 407 and
// 402.  It is the power that operands of a real spread draw: with nearly constant levels kDeep gains the same blocks 1 to 2 %.
// So kLarge has to be ahead by a twelfth past eight units (the figures below contain it), and kDeep is for calls too
// small to matter and where kSmall falls behind for good.  A caller of one such linear alone pays for it, the (14, 16) and
// (5, 8) rows of K 768 and 3072 above, by up to 12 and 14 % with the clock up.  The 128x256 tile on four waves that long
// contractions took before is behind by 2 to 25 % but in calls of four units, where kDeep takes up to 5 % longer (37,142 x
// 2176 -> 288 q 44.5 us, 46.3).
enum class Tile8 { kSmall, kDeep, kLarge };
Tile8 tile8(const GemmParams &p, int epi) {
    constexpr int64_t kCUs = 256;
    const int64_t small = (int64_t)((p.Nout + 127) / 128) * (((int64_t)p.M + 127) / 128);
    const int64_t large = (int64_t)((p.Nout + 255) / 256) * (((int64_t)p.M + 255) / 256);
    const int64_t cs = (small + kCUs - 1) / kCUs, cl = 4 * ((large + kCUs - 1) / kCUs);       // units of the busiest CU
    const bool gelu = epi == kEpiQuantGelu, one_round = large <= kCUs;
    const bool lines = p.x_stride % 128 == 0 && p.w_stride % 128 == 0;           // rows of whole cache lines
    if (cs <= 2) return p.K > 192 ? Tile8::kDeep : Tile8::kSmall;
    int unit;                                       // of kLarge, in hundredths of kSmall's
    if (p.K >= (gelu ? 2048 : 1536)) unit = gelu && !one_round ? 76 : 65;
    else if (p.K >= 768) unit = one_round ? (gelu ? 82 : 65) : (gelu ? 108 : (cs <= 8 ? 84 : 91));
    else unit = gelu ? 108 : (one_round ? 82 : (epi == kEpiF32 && p.K >= (lines && cl <= 8 ? 513 : 320) ? 95 : 104));
    if (unit * cl < 100 * cs) return Tile8::kLarge;
    return p.K >= 2048 && (cs == 4 || (cs == 5 && !lines)) ? Tile8::kDeep : Tile8::kSmall;
}

}  // namespace

hipError_t gemm_launch(GemmParams p, int wb, int ab, hipStream_t stream) {
    // pick the epilogue: the specialised ones need full 16-channel groups and a single output
    int epi = kEpiGeneric;
    const bool aligned = (p.Nout % 16 == 0);
    if (!p.acc_out && p.y_out && !p.yq && p.act == 0) epi = kEpiF32;     // any Nout
    if (aligned && !p.acc_out) {
        if (p.yq && !p.y_out && (p.yq_sb == 4 || p.yq_sb == 8)) epi = p.act == 1 ? kEpiQuantGelu : kEpiQuant;
    }
    if (p.ab_thr) {
        // integer-only epilogue: packed output only, whole 16-channel groups, 4- or 8-bit storage
        if (!aligned || p.acc_out || p.y_out || !p.yq || (p.yq_sb != 4 && p.yq_sb != 8) || p.act != 0 ||
            p.ab_nthr < 1 || p.ab_nthr > 255 || p.hn_gamma)
            return hipErrorInvalidValue;
        epi = p.ab_nthr <= 15 ? kEpiAbsorbed : kEpiAbsorbedBig;
    }
    if (p.hn_gamma) {
        // the fused per-head LayerNorm quantizers need whole 64-channel heads per wave tile
        if (epi != kEpiQuant || !p.head_major || p.dh != 64 || p.D % 64 != 0 || p.Nout != 3 * p.D || !p.hn_beta)
            return hipErrorInvalidValue;
        epi = kEpiHeadNorm;
    }
    // per-lane operand offsets inside a tile are kept in 32 bits (255 rows * stride + 112)
    if (p.x_stride >= (1 << 24) || p.w_stride >= (1 << 24) || p.M < 1 || p.Nout < 1) return hipErrorInvalidValue;
    if (p.head_major) {
        p.inv_ntok = 1.0f / (float)p.Ntok;
        p.dh_shift = -1;
        for (int sft = 0; sft < 16; ++sft)
            if ((1 << sft) == p.dh) p.dh_shift = sft;
        if (p.M >= (1 << 22)) return hipErrorInvalidValue;
    }
    if (p.yq && epi != kEpiAbsorbed && epi != kEpiAbsorbedBig) {
        for (int i = 0; i < 3; ++i) p.r_y[i] = 1.0f / p.s_y[i];
        p.eps0 = ldexpf(1.0f, (p.qmaxf > 7.5f ? 8 : 4) - 22);
        p.gelu_guard = kGeluFastBound;
        // a step so small that 1/s overflows, or so large that it underflows, takes the exact path
        for (int i = 0; i < 3; ++i)
            if (!(p.r_y[i] > 0x1p-100f && p.r_y[i] < 0x1p100f)) {
                if (epi == kEpiHeadNorm) return hipErrorInvalidValue;
                epi = (epi == kEpiF32) ? epi : kEpiGeneric;
            }
    }
    if (use_split(p, wb, ab, epi)) {
        if (wb == 4) return launch_split<4, 4>(p, epi, stream);
        if (wb == 2) return launch_split<2, 4>(p, epi, stream);
        return launch_split<8, 8>(p, epi, stream);
    }
    if (wb == 4 && ab == 4) {
        if (small_tile(p, epi)) return launch_epi<4, 4, 128, 128, 2, 2, VITQ_BK44, 2, 4>(p, epi, stream);
        return launch_epi<4, 4, VITQ_TC, VITQ_TT, VITQ_WC, VITQ_WT, VITQ_BK44, VITQ_S44, VITQ_OCC44>(p, epi, stream);
    }
    if (wb == 2 && ab == 4) return launch_epi<2, 4, 128, 128, 2, 2, 128, 2, 4>(p, epi, stream);
    if (wb == 8 && ab == 8) {
        if (epi == kEpiF32 || epi == kEpiQuant || epi == kEpiQuantGelu) {
            const Tile8 tile = tile8(p, epi);
            if (tile == Tile8::kLarge) return launch_main<8, 8, 256, 256, 4, 4, 128, 2, 4>(p, epi, stream);
            if (tile == Tile8::kDeep) return launch_main<8, 8, 128, 128, 2, 2, 128, 2, 2>(p, epi, stream);
        }
        return launch_epi<8, 8, 128, 128, 2, 2, VITQ_BK88, VITQ_S88, VITQ_OCC88>(p, epi, stream);
    }
    if (wb == 8 && ab == 4) return launch_epi<8, 4, VITQ_TC, VITQ_TT, VITQ_WC, VITQ_WT, VITQ_BK84, VITQ_S84, VITQ_OCC84>(p, epi, stream);
    return hipErrorInvalidValue;
}

}  // namespace vitq
