// Attention on quantized operands: S = Q.K^T (Eq. 3), shift-based exponential (Eq. 4), the
// softmax division absorbed into the P quantizer's thresholds (Sec. IV-B), and O = P.V with
// the operand scales applied next to the output quantizer (Sec. IV-B).
//
// One workgroup (4 waves) serves one (image, head): K and V^T are staged as int8 in
// LDS once, then each wave takes blocks of 16 query rows.  Everything between the two
// matmuls stays in registers:
//
//   S^T tile = mfma_16x16x64(A = K rows, B = Q rows)  -> lane (query = lane%16, g = lane/16)
//              holds keys 16t + 4g + r of tile t: a full score row lives in 4 lanes, so the
//              integer row max and row sum are in-register reductions plus two lane swaps.
//   P^T      = the quantized levels, packed 4 per register in exactly the order the second
//              MFMA wants for its B operand (no LDS round trip between the matmuls).
//   O^T tile = mfma_16x16x64(A = V^T rows, B = P^T)   -> lane holds 16 consecutive d of its
//              query: one 8-byte packed store per lane.
//
// All reductions are integer, so lane order cannot change a result.
#include "attention.h"
#include "vitq_dev.h"

#ifndef VITQ_ATT_OCC
#define VITQ_ATT_OCC 4      // workgroups per CU aimed at by the 4-bit kernels of up to 13 key tiles
#endif
#ifndef VITQ_ATT_OCC8
#define VITQ_ATT_OCC8 4     // the same for 8-bit operands or 8-bit P (143 -> 135 us on the W8A8 ViT-B block)
#endif
#ifndef VITQ_ATT_GROUP
#define VITQ_ATT_GROUP 2    // key tiles between scheduling fences (bounds the loads in flight, hence registers)
#endif
namespace vitq {

namespace {

// physical LDS row of V^T column d: the sixteen rows one MFMA reads are consecutive
__device__ __forceinline__ int vt_row(int d) { return 16 * ((d >> 2) & 3) + 4 * (d >> 4) + (d & 3); }
// position of key n inside a V^T row: lane group g = (n%16)/4 owns 16 consecutive bytes of
// every 64-key chunk, ordered (tile within chunk, r)
__device__ __forceinline__ int vt_pos(int n) {
    return (n & ~63) + (((n & 15) >> 2) << 4) + (((n & 63) >> 4) << 2) + (n & 3);
}

// per-nibble a - b (mod 16) of eight packed nibbles, no borrows across nibbles
__device__ __forceinline__ u32 nib_sub(u32 a, u32 b) {
    return ((a | 0x88888888u) - (b & 0x77777777u)) ^ ((a ^ ~b) & 0x88888888u);
}

// LDS byte address of a pointer into shared memory, and a 32-bit read at such an address
typedef __attribute__((address_space(3))) const u32 lds_u32;
__device__ __forceinline__ u32 lds_addr(const void *p) {
    return (u32)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)p;
}
__device__ __forceinline__ u32 lds_read(u32 addr) { return *(lds_u32 *)(uintptr_t)addr; }

// V^T in LDS (int8, one row per d; a dword of a row is four consecutive keys).  An item is four keys x one
// 4-byte piece of their V rows (eight 4-bit or four 8-bit values): the four words are transposed in
// registers (byte permutes) and written as whole dwords, one per value -- byte-wise writes from lanes
// holding one key each serialise four to a dword.  4-bit values are kept as 16 * q (moved to the top of
// their byte without sign extension, like the other operands), so the P.V accumulators carry a factor
// 2^kShift that the epilogue removes with an exact shift.
template <int SB>
struct VRows {
    static constexpr int kPieces = (SB == 4) ? 8 : 16;     // 4-byte pieces per V row
    static constexpr int kShift = (SB == 4) ? 4 : 0;
    static __device__ __forceinline__ void load(const uint8_t *v, int64_t row0, int64_t stride, int N, int item, u32 (&w)[4]) {
        const int kg = item / kPieces, dp = item - kg * kPieces;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = 4 * kg + i;
            w[i] = 0u;
            if (n < N) w[i] = *reinterpret_cast<const u32 *>(v + (row0 + n) * stride + 4 * dp);
        }
    }
    // rows a0..a3 (one word per key) -> o[j] = byte j of each, key 0 in the low byte
    static __device__ __forceinline__ void transpose(u32 a0, u32 a1, u32 a2, u32 a3, u32 (&o)[4]) {
        const u32 t0 = __builtin_amdgcn_perm(a1, a0, 0x05010400u), t1 = __builtin_amdgcn_perm(a1, a0, 0x07030602u);
        const u32 t2 = __builtin_amdgcn_perm(a3, a2, 0x05010400u), t3 = __builtin_amdgcn_perm(a3, a2, 0x07030602u);
        o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
        o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
        o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
        o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
    }
    static __device__ __forceinline__ void store(uint8_t *sVT, int vpitch, int item, const u32 (&w)[4]) {
        const int kg = item / kPieces, dp = item - kg * kPieces;
        uint8_t *col = sVT + vt_pos(4 * kg);
        u32 o[4];
        if constexpr (SB == 4) {
            // even values (low nibbles) and odd values (high nibbles) of the piece: d = 8*dp + 2*j (+1)
            transpose((w[0] << 4) & 0xF0F0F0F0u, (w[1] << 4) & 0xF0F0F0F0u, (w[2] << 4) & 0xF0F0F0F0u,
                      (w[3] << 4) & 0xF0F0F0F0u, o);
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<u32 *>(col + vt_row(8 * dp + 2 * j) * vpitch) = o[j];
            transpose(w[0] & 0xF0F0F0F0u, w[1] & 0xF0F0F0F0u, w[2] & 0xF0F0F0F0u, w[3] & 0xF0F0F0F0u, o);
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<u32 *>(col + vt_row(8 * dp + 2 * j + 1) * vpitch) = o[j];
        } else {
            transpose(w[0], w[1], w[2], w[3], o);
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<u32 *>(col + vt_row(4 * dp + j) * vpitch) = o[j];
        }
    }
};

// K rows in LDS.  EXPAND (the register-resident kernel): int8 MFMA operands whatever the storage, a
// 4-bit row being expanded once per workgroup when it is staged (16 * level per byte, in the value order
// of unpack4_x16, which the query fragments share) instead of once per 16-query block that reads it.
// Otherwise (the streaming kernel, which reads every row three times per query block and is bound by
// those LDS reads) 4-bit rows stay packed and a lane unpacks its fragment.  Piece c is 8 bytes of the
// packed row; the pitches are bank-conflict-free for the fragment reads.
template <int SB, bool EXPAND>
struct KRows {
    static constexpr int pitch = (SB == 4 && !EXPAND) ? 40 : 80;
    static __device__ __forceinline__ void store_piece(uint8_t *row, int c, const uint2 &v) {
        if constexpr (SB == 4 && EXPAND) *reinterpret_cast<v4i *>(row + 16 * c) = unpack4_x16(v.x, v.y);
        else *reinterpret_cast<uint2 *>(row + 8 * c) = v;
    }
    static __device__ __forceinline__ v4i fragment(const uint8_t *row, int g) {
        if constexpr (SB == 4 && !EXPAND) {
            const uint2 v = *reinterpret_cast<const uint2 *>(row + 8 * g);
            return unpack4_x16(v.x, v.y);
        } else {
            return *reinterpret_cast<const v4i *>(row + 16 * g);
        }
    }
};

// (1+r) << floor(alpha*d) in 12.20 fixed point for an integer score difference d <= 0 (Eq. 4)
__device__ __forceinline__ u32 shift_exp_fixed(int d, float alpha) {
    float tt = alpha * (float)d;
    float f = floorf(tt);
    float fr = tt - f;
    u32 u = (u32)((1.0f + fr) * 1048576.0f);
    float nf = -f;
    int sh = (nf >= 31.0f) ? 31 : (int)nf;
    return u >> sh;
}

// TAIL: N > 16*(NT-1), i.e. every key tile but the last holds only real keys (no masking there).
template <int NT, int SB, int MODE, bool P8, bool LUT, bool TAIL>
__global__ __launch_bounds__(256, (NT <= 13 ? ((SB == 4 && !P8) ? VITQ_ATT_OCC : VITQ_ATT_OCC8) : 1)) void attention_kernel(AttnParams p) {
    constexpr int NCH = (NT + 3) / 4;                 // 64-key chunks of the P.V contraction
    constexpr int NKEYP = NCH * 64;                   // padded key count of V^T rows
    constexpr int KROW = 64 * SB / 8;                 // bytes of one packed K row
    using KR = KRows<SB, true>;
    constexpr int KPITCH = KR::pitch;
    constexpr int VPITCH = NKEYP + 16;
    constexpr int SHIFT = (SB == 4) ? 8 : 0;          // both operands of S carry a factor 16 at 4 bits
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint8_t *sK = smem;                               // [NT*16][KPITCH]
    uint8_t *sVT = smem + ((NT * 16 * KPITCH + 15) & ~15);  // [64][VPITCH] int8
    u32 *sLUT = reinterpret_cast<u32 *>(sVT + 64 * VPITCH);  // [lut_n] exponential table (4-bit)
    const int lut_last = p.lut_n - 1;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int li = lane & 15;
    const int g = lane >> 4;
    const int bh = blockIdx.x;
    const int b = bh / p.H;
    const int h = bh - b * p.H;
    const int N = p.N;
    const int64_t row0 = (int64_t)bh * N;             // first row of this head in q/k/v/p

    // ---- stage K and V^T (both int8) ---------------------------------------------------
    // Every global load of this thread is requested before anything waits on one (the table of
    // exponentials is computed while they are in flight): a load -> store loop would pay the memory
    // latency once per trip.
    constexpr int KCH = KROW / 8;                     // 8-byte pieces per K row
    using VR = VRows<SB>;
    constexpr int K_ITEMS = NT * 16 * KCH, V_ITEMS = (NKEYP / 4) * VR::kPieces;   // (V: four keys x one 4-byte piece)
    constexpr bool BATCH = (NT <= 13);                // (the long-row variant keeps the loop: registers)
    constexpr int K_IT = BATCH ? (K_ITEMS + 255) / 256 : 1, V_IT = BATCH ? (V_ITEMS + 255) / 256 : 1;
    [[maybe_unused]] uint2 kreg[K_IT];
    [[maybe_unused]] u32 vreg[V_IT][4];
    if constexpr (BATCH && MODE != kAttnPVOnly) {
#pragma unroll
        for (int it = 0; it < K_IT; ++it) {
            const int id = it * 256 + tid;
            const int n = id / KCH, c = id - n * KCH;
            kreg[it] = make_uint2(0, 0);
            if (id < K_ITEMS && n < N) kreg[it] = *reinterpret_cast<const uint2 *>(p.k + (row0 + n) * p.k_stride + c * 8);
        }
    }
    if constexpr (BATCH && MODE != kAttnQKOnly) {
#pragma unroll
        for (int it = 0; it < V_IT; ++it) {
            const int id = it * 256 + tid;
            VR::load(p.v, row0, p.v_stride, id < V_ITEMS ? N : 0, id, vreg[it]);
        }
    }
    // this lane's packed query row of block qb (zeros beyond the last row); the first block's is
    // requested here and each later one while the block before it is computed
    const int nqb = (N + 15) / 16;
    const int wslot = (wave + bh) & 3;                // rotate which wave gets the odd block
    const int qb_first = blockIdx.y * 4 + wslot, qb_step = 4 * p.qsplit;
    auto load_q = [&](int qb) {
        uint4 v = make_uint4(0, 0, 0, 0);
        const int qrow = qb * 16 + li;
        if (qb < nqb && qrow < N) {
            const uint8_t *src = p.q + (row0 + qrow) * p.q_stride;
            if constexpr (SB == 4) {
                const uint2 t = *reinterpret_cast<const uint2 *>(src + 8 * g);
                v.x = t.x; v.y = t.y;
            } else {
                v = *reinterpret_cast<const uint4 *>(src + 16 * g);
            }
        }
        return v;
    };
    [[maybe_unused]] uint4 qnext = make_uint4(0, 0, 0, 0);
    if constexpr (MODE != kAttnPVOnly) qnext = load_q(qb_first);
    if constexpr (LUT && MODE != kAttnPVOnly) {
        // entry d: the fixed-point exponential of score difference -d, by the exact operation
        // sequence; the last entry stands for every larger difference, where the value is 0
        for (int i = tid; i < p.lut_n; i += 256)
            sLUT[i] = (i == lut_last) ? 0u : shift_exp_fixed(-i, p.alpha);
    }
    if constexpr (MODE != kAttnPVOnly) {
        if constexpr (BATCH) {
#pragma unroll
            for (int it = 0; it < K_IT; ++it) {
                const int id = it * 256 + tid;
                const int n = id / KCH, c = id - n * KCH;
                if (id < K_ITEMS) KR::store_piece(sK + n * KPITCH, c, kreg[it]);
            }
        } else {
            for (int id = tid; id < K_ITEMS; id += 256) {
                int n = id / KCH, c = id - n * KCH;
                uint2 v = make_uint2(0, 0);
                if (n < N) v = *reinterpret_cast<const uint2 *>(p.k + (row0 + n) * p.k_stride + c * 8);
                KR::store_piece(sK + n * KPITCH, c, v);
            }
        }
    }
    if constexpr (MODE != kAttnQKOnly) {
        if constexpr (BATCH) {
#pragma unroll
            for (int it = 0; it < V_IT; ++it) {
                const int id = it * 256 + tid;
                if (id < V_ITEMS) VR::store(sVT, VPITCH, id, vreg[it]);
            }
        } else {
            for (int id = tid; id < V_ITEMS; id += 256) {
                u32 w[4];
                VR::load(p.v, row0, p.v_stride, N, id, w);
                VR::store(sVT, VPITCH, id, w);
            }
        }
    }
    __syncthreads();

    for (int qb = qb_first; qb < nqb; qb += qb_step) {
        const int qrow = qb * 16 + li;                // query row of this lane
        const bool qok = qrow < N;
        u32 pp[NCH * 4];                              // packed P^T: 4 levels per register
#pragma unroll
        for (int i = 0; i < NCH * 4; ++i) pp[i] = P8 ? 0x80808080u : 0u;

        if constexpr (MODE != kAttnPVOnly) {
            // ---- S^T = K . Q^T ------------------------------------------------------------
            v4i qf;
            {
                const uint4 v = qnext;
                qnext = load_q(qb + qb_step);
                if constexpr (SB == 4) {
                    qf = unpack4_x16(v.x, v.y);
                } else {
                    qf[0] = (int)v.x; qf[1] = (int)v.y; qf[2] = (int)v.z; qf[3] = (int)v.w;
                }
            }
            v4i s[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                v4i kf;
                kf = KR::fragment(sK + (16 * t + li) * KPITCH, g);
                v4i z = {0, 0, 0, 0};
                s[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf, qf, z, 0, 0, 0);
            }
            // Tiles t < n_full hold only real keys (known at compile time in the TAIL variant).
            // ---- integer row max (keys >= N excluded) ---------------------------------------
            int mx = INT32_MIN;
            static_for<NT>([&](auto T) {
                constexpr int t = decltype(T)::value;
                if (TAIL && t < NT - 1) {
                    mx = max(mx, max(max(s[t][0], s[t][1]), max(s[t][2], s[t][3])));
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (16 * t + 4 * g + r < N) mx = max(mx, s[t][r]);
                }
            });
            mx = max(mx, __shfl_xor(mx, 16, 64));
            mx = max(mx, __shfl_xor(mx, 32, 64));
            if constexpr (MODE == kAttnQKOnly) {
                if (p.s_acc_out && qok) {
                    int32_t *dst = p.s_acc_out + (row0 + qrow) * N;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int key = 16 * t + 4 * g + r;
                            if (key < N) dst[key] = s[t][r] >> SHIFT;
                        }
                }
            }
            // ---- shift-based exponential in 12.20 fixed point (Eq. 4), integer row sum -------
            // e depends only on the integer difference d = max - S, so at 4 bits (d <= 8192) it is
            // read from a table that this workgroup filled with the exact operation sequence.
            bool direct = !LUT;
            if constexpr (LUT) {
                if (!p.lut_full) {
                    // cut table: a row whose spread max - min reaches past it cannot use it
                    int mn = INT32_MAX;
                    static_for<NT>([&](auto T) {
                        constexpr int t = decltype(T)::value;
                        if (TAIL && t < NT - 1) {
                            mn = min(mn, min(min(s[t][0], s[t][1]), min(s[t][2], s[t][3])));
                        } else {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (16 * t + 4 * g + r < N) mn = min(mn, s[t][r]);
                        }
                    });
                    mn = min(mn, __shfl_xor(mn, 16, 64));
                    mn = min(mn, __shfl_xor(mn, 32, 64));
                    direct = __builtin_amdgcn_ballot_w64(((mx - mn) >> SHIFT) >= lut_last) != 0;
                }
            }
            u32 sum = 0;
            constexpr int LSH = SHIFT >= 2 ? SHIFT - 2 : 0;     // (the table exists at 4 bits only)
            [[maybe_unused]] const u32 lut_hi = lds_addr(sLUT) + (u32)(mx >> LSH);
            [[maybe_unused]] const u32 lut_cap = lds_addr(sLUT) + 4u * (u32)lut_last;
            auto exp_pass = [&](auto DIRECT) {
                auto exp_of = [&](int sv) -> u32 {
                    if constexpr (LUT && !decltype(DIRECT)::value) {
                        // scores carry the operand factor 2^SHIFT, so (mx - sv) >> (SHIFT - 2) is the
                        // byte offset 4*d of entry d directly
                        // (both are multiples of 2^SHIFT, so the shift distributes over the difference;
                        // lut_hi = table address + (mx >> LSH), lut_cap = address of the last entry)
                        return lds_read(min(lut_hi - (u32)(sv >> LSH), lut_cap));
                    } else {
                        return shift_exp_fixed(sv - mx, p.alpha_scaled);
                    }
                };
                static_for<NT>([&](auto T) {
                    constexpr int t = decltype(T)::value;
                    if constexpr (VITQ_ATT_GROUP > 0 && t % (VITQ_ATT_GROUP > 0 ? VITQ_ATT_GROUP : 1) == 0 && t > 0)
                        __builtin_amdgcn_sched_barrier(0);     // bound the table loads in flight (registers)
                    if (TAIL && t < NT - 1) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) { const u32 e = exp_of(s[t][r]); s[t][r] = (int)e; sum += e; }
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            u32 e = 0;
                            if (16 * t + 4 * g + r < N) e = exp_of(s[t][r]);
                            s[t][r] = (int)e;
                            sum += e;
                        }
                    }
                });
            };
            if (direct) exp_pass(std::true_type{});
            else exp_pass(std::false_type{});
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            // ---- P level = #{k : 2*pmax*e > (2k-1)*sum} (division absorbed into the comparator) --
            // Cheap value x = e * (pmax/sum) in fp32 is within pmax*2^-22 of the exact ratio, and the
            // level is that ratio rounded (exact halves down).  Unless x is that close to a half,
            // rint(x) is the level; otherwise the four values are decided in 64-bit integers.
            const float inv = (float)p.pmax / (float)sum;
            const float thr_p = 0.5f - (P8 ? 0x1p-13f : 0x1p-17f);
            const u32 two_pmax = 2u * (u32)p.pmax;
            float worst = 0.0f;            // largest distance of a ratio from its rounded value
            static_for<NT>([&](auto T) {
                constexpr int t = decltype(T)::value;
                if constexpr (VITQ_ATT_GROUP > 0 && t % (VITQ_ATT_GROUP > 0 ? VITQ_ATT_GROUP : 1) == 0 && t > 0)
                    __builtin_amdgcn_sched_barrier(0);
                u32 packed = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = (float)(u32)s[t][r] * inv;
                    const float q = rintf(x);
                    worst = fmaxf(worst, fabsf(x - q));
                    packed = __builtin_amdgcn_cvt_pk_u8_f32(q, r, packed);
                }
                pp[t] = P8 ? (packed ^ 0x80808080u) : packed;
            });
            if (__builtin_amdgcn_ballot_w64(!(worst <= thr_p)) != 0) {
                // some ratio of this 16-query block is within the error bound of a half: decide
                // every level of the block in exact 64-bit integer arithmetic (rare)
                static_for<NT>([&](auto T) {
                    constexpr int t = decltype(T)::value;
                    u32 packed = 0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const u32 e = (u32)s[t][r];
                        u32 c = (u32)rintf((float)e * inv);
                        const uint64_t lhs = (uint64_t)two_pmax * e;
                        const uint64_t up = (uint64_t)(2u * c + 1u) * sum;
                        const uint64_t dn = (uint64_t)(2u * c - 1u) * sum;   // only used when c > 0
                        if (lhs > up) c += 1;
                        else if (c > 0 && lhs <= dn) c -= 1;
                        c = min(c, (u32)p.pmax);
                        packed |= (P8 ? (c ^ 0x80u) : c) << (8 * r);
                    }
                    pp[t] = packed;
                });
            }
            if constexpr (MODE == kAttnQKOnly) {
                if (p.p_out && qok) {
                    uint8_t *dst = p.p_out + (row0 + qrow) * p.p_out_stride;
#pragma unroll
                    for (int t = 0; t < NT + 1; ++t) {
                        const u32 lv = (t < NT) ? (P8 ? (pp[t < NT ? t : 0] ^ 0x80808080u) : pp[t < NT ? t : 0]) : 0u;
                        if (p.p_sb == 4) {
                            const int off = 8 * t + 2 * g;
                            if (off < p.p_out_row_bytes16) {
                                u32 hw = (lv & 0xFu) | ((lv >> 4) & 0xF0u) | ((lv >> 8) & 0xF00u) | ((lv >> 12) & 0xF000u);
                                *reinterpret_cast<uint16_t *>(dst + off) = (uint16_t)hw;
                            }
                        } else {
                            const int off = 16 * t + 4 * g;
                            if (off < p.p_out_row_bytes16) *reinterpret_cast<u32 *>(dst + off) = lv;
                        }
                    }
                }
            }
        } else {
            // ---- P^T from memory (stand-alone P.V) ------------------------------------------
            const uint8_t *src = p.p_in + (row0 + qrow) * p.p_in_stride;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                u32 lv = 0;
                if (p.p_sb == 4) {
                    const int off = 8 * t + 2 * g;
                    if (qok && off < p.p_in_row_bytes16) {
                        u32 hw = *reinterpret_cast<const uint16_t *>(src + off);
                        lv = (hw & 0xFu) | ((hw & 0xF0u) << 4) | ((hw & 0xF00u) << 8) | ((hw & 0xF000u) << 12);
                    }
                } else {
                    const int off = 16 * t + 4 * g;
                    if (qok && off < p.p_in_row_bytes16) lv = *reinterpret_cast<const u32 *>(src + off);
                }
                pp[t] = P8 ? (lv ^ 0x80808080u) : lv;
            }
        }

        if constexpr (MODE != kAttnQKOnly) {
            // ---- O^T = V^T . P^T ------------------------------------------------------------
            v4i o[4], cs[4];
#pragma unroll
            for (int T = 0; T < 4; ++T) { o[T] = v4i{0, 0, 0, 0}; cs[T] = v4i{0, 0, 0, 0}; }
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                v4i pf;
                pf[0] = (int)pp[4 * c]; pf[1] = (int)pp[4 * c + 1];
                pf[2] = (int)pp[4 * c + 2]; pf[3] = (int)pp[4 * c + 3];
#pragma unroll
                for (int T = 0; T < 4; ++T) {
                    v4i vf = *reinterpret_cast<const v4i *>(sVT + (16 * T + li) * VPITCH + 64 * c + 16 * g);
                    o[T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf, pf, o[T], 0, 0, 0);
                    if constexpr (P8) {
                        // levels are stored minus 128; add 128 * (column sum of V) back
                        const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
                        cs[T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf, ones, cs[T], 0, 0, 0);
                    }
                }
            }
            if (qok) {
                float lv[16];            // level - qmin, in [0, qmax - qmin]
                float of[16];
                int oa[16];
                // requantization: cheap value fma(o, 1/s_o, -qmin) with the same guard as the
                // linear epilogue; a block with an element near a rounding boundary is redone
                // with the exact division
                const float bias8 = -p.qminf, top = p.qmaxf - p.qminf;
                const float thr_o = 0.5f - p.eps_o;
                u32 worst_o = 0u;        // max distance to the rounded value, as bit patterns (NaN on top)
#pragma unroll
                for (int T = 0; T < 4; ++T)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        int a = o[T][r];
                        if constexpr (P8) a += 128 * cs[T][r];
                        a >>= VRows<SB>::kShift;         // (V^T holds 16 * q at 4 bits: exact)
                        oa[4 * T + r] = a;
                        const float ov = (float)a * p.spv;
                        of[4 * T + r] = ov;
                        const float t8 = fmaf(ov, p.r_o, bias8);
                        const float q8 = rintf(t8);
                        worst_o = max(worst_o, __float_as_uint(fabsf(t8 - q8)));
                        lv[4 * T + r] = __builtin_amdgcn_fmed3f(q8, 0.0f, top);
                    }
                if (__builtin_amdgcn_ballot_w64(worst_o > __float_as_uint(thr_o)) != 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        lv[i] = __builtin_amdgcn_fmed3f(rintf(of[i] / p.s_o) + bias8, 0.0f, top);
                }
                const int d0 = 16 * g;
                if (p.o_acc_out) {
                    int4 *dst = reinterpret_cast<int4 *>(p.o_acc_out + (row0 + qrow) * 64 + d0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) dst[j] = make_int4(oa[4 * j], oa[4 * j + 1], oa[4 * j + 2], oa[4 * j + 3]);
                }
                const int64_t orow = (int64_t)b * N + qrow;
                if (p.o_out) {
                    float4 *dst = reinterpret_cast<float4 *>(p.o_out + orow * (p.H * 64) + h * 64 + d0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) dst[j] = make_float4(of[4 * j], of[4 * j + 1], of[4 * j + 2], of[4 * j + 3]);
                }
                if (p.oq) {
                    uint8_t *dst = p.oq + orow * p.oq_stride + (((h * 64 + d0) * p.oq_sb) >> 3);
                    if (p.oq_sb == 4) {
                        // even-indexed levels in the low nibbles of one word, odd-indexed shifted into
                        // the high ones; the stored levels are biased by -qmin = 8, and flipping bit 3
                        // turns them into two's complement
                        u32 ev0 = 0, od0 = 0, ev1 = 0, od1 = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            ev0 = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i], i, ev0);
                            od0 = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i + 1], i, od0);
                            ev1 = __builtin_amdgcn_cvt_pk_u8_f32(lv[8 + 2 * i], i, ev1);
                            od1 = __builtin_amdgcn_cvt_pk_u8_f32(lv[8 + 2 * i + 1], i, od1);
                        }
                        const u32 fix = 0x11111111u * ((u32)bias8 & 0xFu);
                        // per-nibble subtraction of the bias (a power of two: 2^(bits-1)) modulo 16
                        const u32 w0 = nib_sub(ev0 | (od0 << 4), fix);
                        const u32 w1 = nib_sub(ev1 | (od1 << 4), fix);
                        *reinterpret_cast<uint2 *>(dst) = make_uint2(w0, w1);
                    } else {
                        const u32 fix = 0x01010101u * ((u32)bias8 & 0xFFu);
                        u32 w[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            u32 v = 0;
#pragma unroll
                            for (int i = 0; i < 4; ++i) v = __builtin_amdgcn_cvt_pk_u8_f32(lv[4 * j + i], i, v);
                            // per-byte subtraction of the bias without borrows across bytes
                            w[j] = ((v | 0x80808080u) - (fix & 0x7F7F7F7Fu)) ^ ((v ^ ~fix) & 0x80808080u);
                        }
                        *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                }
            }
        }
    }
}

template <int NT, int SB, int MODE, bool P8, bool LUT, bool TAIL>
hipError_t launch_tail(const AttnParams &p, hipStream_t stream) {
    constexpr int NCH = (NT + 3) / 4;
    constexpr int KPITCH = KRows<SB, true>::pitch;
    const size_t lds = ((NT * 16 * KPITCH + 15) & ~15) + (size_t)64 * (NCH * 64 + 16) +
                       (LUT ? (size_t)p.lut_n * 4 : 0);
    auto kern = attention_kernel<NT, SB, MODE, P8, LUT, TAIL>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    dim3 grid((unsigned)(p.B * p.H), (unsigned)p.qsplit);
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, stream, p);
    return hipGetLastError();
}

template <int NT, int SB, int MODE, bool P8, bool LUT>
hipError_t launch_one(const AttnParams &p, hipStream_t stream) {
    if (p.N > 16 * (NT - 1)) return launch_tail<NT, SB, MODE, P8, LUT, true>(p, stream);
    return launch_tail<NT, SB, MODE, P8, LUT, false>(p, stream);
}

template <int NT, int SB, int MODE>
hipError_t launch_p(const AttnParams &p, hipStream_t stream) {
    if (p.pmax > 127) return launch_one<NT, SB, MODE, true, false>(p, stream);
    if (SB == 4 && p.lut_n > 0 && MODE != kAttnPVOnly) return launch_one<NT, SB, MODE, false, true>(p, stream);
    return launch_one<NT, SB, MODE, false, false>(p, stream);
}

template <int NT, int SB>
hipError_t launch_mode(const AttnParams &p, AttnMode mode, hipStream_t stream) {
    switch (mode) {
        case kAttnFused: return launch_p<NT, SB, kAttnFused>(p, stream);
        case kAttnQKOnly: return launch_p<NT, SB, kAttnQKOnly>(p, stream);
        case kAttnPVOnly: return launch_p<NT, SB, kAttnPVOnly>(p, stream);
    }
    return hipErrorInvalidValue;
}

// ---- fused attention, streaming form --------------------------------------------------------
// The kernel above keeps a whole score row block (16 queries x all keys) in registers, which
// costs 4 registers per key tile and limits it to one or two waves per SIMD.  The matrix cores
// are nearly idle in this kernel (the work is the softmax arithmetic), so this form RECOMPUTES
// the 16x16 score tiles instead of keeping them: pass A takes the integer row maximum (and
// minimum when the exponential table was cut), pass B the integer sum of the exponentials, pass C
// quantizes each tile to P levels and feeds the P.V matrix cores one 64-key chunk at a time.
// Every value is produced by the same arithmetic as above (integer max and sum, table / exact
// exponential, guarded fp32 quantizer with the 64-bit fallback), so the results are identical;
// only a handful of registers hold scores at any time, and the key count is a run-time value.
constexpr int kStreamThreads = 1024;    // 16 waves share one head's K / V^T in LDS

// KEEP == 0: eight waves per SIMD, i.e. at most 64 registers, so that two workgroups share a CU.
// KEEP > 0: one workgroup's LDS fills a CU, four waves per SIMD have 128 registers, and the exponentials
// of the first KEEP tiles (all of real keys) stay in registers from pass B to pass C.
template <int SB, bool P8, bool LUT, int KEEP>
__global__ __launch_bounds__(kStreamThreads, (KEEP > 0 ? 4 : 8)) void attention_stream_kernel(AttnParams p) {
    static_assert(KEEP % 4 == 0, "whole 64-key chunks are kept");
    constexpr int NTHR = kStreamThreads, NW = NTHR / 64;
    constexpr int KROW = 64 * SB / 8;
    using KR = KRows<SB, false>;
    constexpr int KPITCH = KR::pitch;
    constexpr int SHIFT = (SB == 4) ? 8 : 0;
    const int N = p.N;
    const int nt = (N + 15) / 16;                     // key tiles
    const int nch = (nt + 3) / 4;                     // 64-key chunks
    const int nkeyp = nch * 64;
    const int vpitch = nkeyp + 16;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint8_t *sK = smem;                               // [nch*64][KPITCH] (rows >= N are zero)
    uint8_t *sVT = smem + (((size_t)nkeyp * KPITCH + 15) & ~(size_t)15);   // [64][vpitch] int8
    u32 *sLUT = reinterpret_cast<u32 *>(sVT + 64 * vpitch);
    const int lut_last = p.lut_n - 1;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int li = lane & 15;
    const int g = lane >> 4;
    const int bh = blockIdx.x;
    const int b = bh / p.H;
    const int h = bh - b * p.H;
    const int64_t row0 = (int64_t)bh * N;

    // Every global load of this thread (K, V and the first query row) is requested before anything
    // waits on one; the table of exponentials is computed while they are in flight.
    constexpr int KCH = KROW / 8;                     // 8-byte pieces per K row
    using VR = VRows<SB>;                             // V items: four keys x one 4-byte piece
    constexpr int kMaxKeyp = 640;                     // N <= 592
    constexpr int K_IT = (kMaxKeyp * KCH + NTHR - 1) / NTHR, V_IT = ((kMaxKeyp / 4) * VR::kPieces + NTHR - 1) / NTHR;
    uint2 kreg[K_IT];
    u32 vreg[V_IT][4];
#pragma unroll
    for (int it = 0; it < K_IT; ++it) {
        const int id = it * NTHR + tid;
        const int n = id / KCH, c = id - n * KCH;
        kreg[it] = make_uint2(0, 0);
        if (n < N) kreg[it] = *reinterpret_cast<const uint2 *>(p.k + (row0 + n) * p.k_stride + c * 8);
    }
#pragma unroll
    for (int it = 0; it < V_IT; ++it) {
        const int id = it * NTHR + tid;
        VR::load(p.v, row0, p.v_stride, id < (nkeyp / 4) * VR::kPieces ? N : 0, id, vreg[it]);
    }
    const int nqb = (N + 15) / 16;
    const int wslot = (wave + bh) % NW;
    const int qb_first = blockIdx.y * NW + wslot, qb_step = NW * p.qsplit;
    auto load_q = [&](int qb) {
        uint4 v = make_uint4(0, 0, 0, 0);
        const int qrow = qb * 16 + li;
        if (qb < nqb && qrow < N) {
            const uint8_t *src = p.q + (row0 + qrow) * p.q_stride;
            if constexpr (SB == 4) {
                const uint2 t = *reinterpret_cast<const uint2 *>(src + 8 * g);
                v.x = t.x; v.y = t.y;
            } else {
                v = *reinterpret_cast<const uint4 *>(src + 16 * g);
            }
        }
        return v;
    };
    uint4 qnext = load_q(qb_first);
    if constexpr (LUT) {
        for (int i = tid; i < p.lut_n; i += NTHR)
            sLUT[i] = (i == lut_last) ? 0u : shift_exp_fixed(-i, p.alpha);
    }
#pragma unroll
    for (int it = 0; it < K_IT; ++it) {
        const int id = it * NTHR + tid;
        const int n = id / KCH, c = id - n * KCH;
        if (id < nkeyp * KCH) KR::store_piece(sK + n * KPITCH, c, kreg[it]);
    }
#pragma unroll
    for (int it = 0; it < V_IT; ++it) {
        const int id = it * NTHR + tid;
        if (id < (nkeyp / 4) * VR::kPieces) VR::store(sVT, vpitch, id, vreg[it]);
    }
    __syncthreads();

    const float thr_p = 0.5f - (P8 ? 0x1p-13f : 0x1p-17f);
    const u32 two_pmax = 2u * (u32)p.pmax;
    for (int qb = qb_first; qb < nqb; qb += qb_step) {
        const int qrow = qb * 16 + li;
        const bool qok = qrow < N;
        v4i qf;
        {
            const uint4 v = qnext;
            qnext = load_q(qb + qb_step);
            if constexpr (SB == 4) {
                qf = unpack4_x16(v.x, v.y);
            } else {
                qf[0] = (int)v.x; qf[1] = (int)v.y; qf[2] = (int)v.z; qf[3] = (int)v.w;
            }
        }
        // one 16-key tile of S^T: lane (query li, group g) gets keys 16t + 4g + r
        auto score_tile = [&](int t) -> v4i {
            v4i kf;
            kf = KR::fragment(sK + (16 * t + li) * KPITCH, g);
            v4i z = {0, 0, 0, 0};
            return __builtin_amdgcn_mfma_i32_16x16x64_i8(kf, qf, z, 0, 0, 0);
        };
        const int nfull = N / 16;                      // tiles [0, nfull) hold only real keys

        // ---- pass A: integer row max (and min) -------------------------------------------------
        int mx = INT32_MIN, mn = INT32_MAX;
#pragma unroll 4
        for (int t = 0; t < nfull; ++t) {
            const v4i s = score_tile(t);
            mx = max(mx, max(max(s[0], s[1]), max(s[2], s[3])));
            if (LUT && !p.lut_full) mn = min(mn, min(min(s[0], s[1]), min(s[2], s[3])));
        }
        if (nfull < nt) {
            const v4i s = score_tile(nfull);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * nfull + 4 * g + r < N) { mx = max(mx, s[r]); mn = min(mn, s[r]); }
        }
        mx = max(mx, __shfl_xor(mx, 16, 64));
        mx = max(mx, __shfl_xor(mx, 32, 64));
        bool direct = !LUT;
        if constexpr (LUT) {
            if (!p.lut_full) {
                mn = min(mn, __shfl_xor(mn, 16, 64));
                mn = min(mn, __shfl_xor(mn, 32, 64));
                direct = __builtin_amdgcn_ballot_w64(((mx - mn) >> SHIFT) >= lut_last) != 0;
            }
        }
        constexpr int LSH = SHIFT >= 2 ? SHIFT - 2 : 0;
        const u32 lut_hi = lds_addr(sLUT) + (u32)(mx >> LSH);
        const u32 lut_cap = lds_addr(sLUT) + 4u * (u32)lut_last;
        auto exp_of = [&](int sv) -> u32 {
            if (LUT && !direct) return lds_read(min(lut_hi - (u32)(sv >> LSH), lut_cap));
            return shift_exp_fixed(sv - mx, p.alpha_scaled);
        };
        // exponentials of one tile, zero for keys >= N
        auto exp_tile = [&](int t, u32 (&e)[4]) {
            const v4i s = score_tile(t);
            if (t < nfull) {
#pragma unroll
                for (int r = 0; r < 4; ++r) e[r] = exp_of(s[r]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) e[r] = (16 * t + 4 * g + r < N) ? exp_of(s[r]) : 0u;
            }
        };

        // ---- pass B: integer row sum of the exponentials ---------------------------------------
        u32 sum = 0;
        [[maybe_unused]] u32 keep[KEEP > 0 ? KEEP : 1][4];
        static_for<KEEP>([&](auto T) {
            constexpr int t = decltype(T)::value;
            if constexpr (t % 4 == 0 && t > 0) __builtin_amdgcn_sched_barrier(0);      // (bounds the registers)
            const v4i s = score_tile(t);
#pragma unroll
            for (int r = 0; r < 4; ++r) keep[t][r] = exp_of(s[r]);
            sum += (keep[t][0] + keep[t][1]) + (keep[t][2] + keep[t][3]);
        });
#pragma unroll 4
        for (int t = KEEP; t < nt; ++t) {
            u32 e[4];
            exp_tile(t, e);
            sum += (e[0] + e[1]) + (e[2] + e[3]);
        }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        const float inv = (float)p.pmax / (float)sum;

        // ---- pass C: P levels, one 64-key chunk at a time, into the P.V matrix cores -----------
        v4i o[4], cs[4];
#pragma unroll
        for (int T = 0; T < 4; ++T) { o[T] = v4i{0, 0, 0, 0}; cs[T] = v4i{0, 0, 0, 0}; }
        auto chunk = [&](auto C, int c) {                // C >= 0: chunk number known, its exponentials kept
            constexpr bool KEPT = decltype(C)::value >= 0;
            u32 pp[4];
            float worst = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 4 * c + j;
                u32 packed = 0;
                if (KEPT || t < nt) {
                    u32 e[4];
                    if constexpr (KEPT) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) e[r] = keep[4 * decltype(C)::value + j][r];
                    } else {
                        exp_tile(t, e);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float x = (float)e[r] * inv;
                        const float q = rintf(x);
                        worst = fmaxf(worst, fabsf(x - q));
                        packed = __builtin_amdgcn_cvt_pk_u8_f32(q, r, packed);
                    }
                }
                pp[j] = P8 ? (packed ^ 0x80808080u) : packed;
            }
            if (__builtin_amdgcn_ballot_w64(!(worst <= thr_p)) != 0) {
                // some ratio of this chunk is within the error bound of a half: decide its levels
                // in exact 64-bit integer arithmetic (rare)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 4 * c + j;
                    u32 packed = 0;
                    if (t < nt) {
                        u32 e[4];
                        exp_tile(t, e);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            u32 lvl = (u32)rintf((float)e[r] * inv);
                            const uint64_t lhs = (uint64_t)two_pmax * e[r];
                            const uint64_t up = (uint64_t)(2u * lvl + 1u) * sum;
                            const uint64_t dn = (uint64_t)(2u * lvl - 1u) * sum;   // only used when lvl > 0
                            if (lhs > up) lvl += 1;
                            else if (lvl > 0 && lhs <= dn) lvl -= 1;
                            lvl = min(lvl, (u32)p.pmax);
                            packed |= lvl << (8 * r);
                        }
                    }
                    pp[j] = P8 ? (packed ^ 0x80808080u) : packed;
                }
            }
            v4i pf;
            pf[0] = (int)pp[0]; pf[1] = (int)pp[1]; pf[2] = (int)pp[2]; pf[3] = (int)pp[3];
#pragma unroll
            for (int T = 0; T < 4; ++T) {
                v4i vf = *reinterpret_cast<const v4i *>(sVT + (16 * T + li) * vpitch + 64 * c + 16 * g);
                o[T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf, pf, o[T], 0, 0, 0);
                if constexpr (P8) {
                    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
                    cs[T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf, ones, cs[T], 0, 0, 0);
                }
            }
        };
        static_for<KEEP / 4>([&](auto C) { chunk(C, decltype(C)::value); });
        for (int c = KEEP / 4; c < nch; ++c) chunk(std::integral_constant<int, -1>{}, c);

        // ---- output: scale, requantize (guarded), pack ------------------------------------------
        if (qok) {
            float lv[16];
            float of[16];
            const float bias8 = -p.qminf, top = p.qmaxf - p.qminf;
            const float thr_o = 0.5f - p.eps_o;
            u32 worst_o = 0u;
#pragma unroll
            for (int T = 0; T < 4; ++T)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    int a = o[T][r];
                    if constexpr (P8) a += 128 * cs[T][r];
                    a >>= VRows<SB>::kShift;             // (V^T holds 16 * q at 4 bits: exact)
                    const float ov = (float)a * p.spv;
                    of[4 * T + r] = ov;
                    const float t8 = fmaf(ov, p.r_o, bias8);
                    const float q8 = rintf(t8);
                    worst_o = max(worst_o, __float_as_uint(fabsf(t8 - q8)));
                    lv[4 * T + r] = __builtin_amdgcn_fmed3f(q8, 0.0f, top);
                }
            if (__builtin_amdgcn_ballot_w64(worst_o > __float_as_uint(thr_o)) != 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    lv[i] = __builtin_amdgcn_fmed3f(rintf(of[i] / p.s_o) + bias8, 0.0f, top);
            }
            const int d0 = 16 * g;
            const int64_t orow = (int64_t)b * N + qrow;
            uint8_t *dst = p.oq + orow * p.oq_stride + (((h * 64 + d0) * p.oq_sb) >> 3);
            if (p.oq_sb == 4) {
                u32 ev0 = 0, od0 = 0, ev1 = 0, od1 = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ev0 = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i], i, ev0);
                    od0 = __builtin_amdgcn_cvt_pk_u8_f32(lv[2 * i + 1], i, od0);
                    ev1 = __builtin_amdgcn_cvt_pk_u8_f32(lv[8 + 2 * i], i, ev1);
                    od1 = __builtin_amdgcn_cvt_pk_u8_f32(lv[8 + 2 * i + 1], i, od1);
                }
                const u32 fix = 0x11111111u * ((u32)bias8 & 0xFu);
                *reinterpret_cast<uint2 *>(dst) = make_uint2(nib_sub(ev0 | (od0 << 4), fix), nib_sub(ev1 | (od1 << 4), fix));
            } else {
                const u32 fix = 0x01010101u * ((u32)bias8 & 0xFFu);
                u32 w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    u32 v = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v = __builtin_amdgcn_cvt_pk_u8_f32(lv[4 * j + i], i, v);
                    w[j] = ((v | 0x80808080u) - (fix & 0x7F7F7F7Fu)) ^ ((v ^ ~fix) & 0x80808080u);
                }
                *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
}

template <int SB, bool P8, bool LUT, int KEEP>
hipError_t launch_stream_keep(const AttnParams &p, size_t lds, hipStream_t stream) {
    auto kern = attention_stream_kernel<SB, P8, LUT, KEEP>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    dim3 grid((unsigned)(p.B * p.H), (unsigned)p.qsplit);
    hipLaunchKernelGGL(kern, grid, dim3(kStreamThreads), lds, stream, p);
    return hipGetLastError();
}

template <int SB, bool P8, bool LUT>
hipError_t launch_stream(const AttnParams &p, hipStream_t stream) {
    constexpr int KPITCH = KRows<SB, false>::pitch;
    [[maybe_unused]] constexpr int KEEP = 16;            // (64 of the 128 registers)
    const int nch = ((p.N + 15) / 16 + 3) / 4;
    const size_t lds = (((size_t)nch * 64 * KPITCH + 15) & ~(size_t)15) + (size_t)64 * (nch * 64 + 16) +
                       (LUT ? (size_t)p.lut_n * 4 : 0);
    // Past half a CU's 160 KB a second workgroup would not fit, so the registers it would need are free for
    // the exponentials (8-bit operands from 513 keys, so the first KEEP tiles hold real keys only; 4-bit ones
    // stay below and keep the occupancy, with which they measured the same).  Attention block, 8 bits, 577
    // keys: 9 images x 16 heads 134 -> 126 us with P of 8 bits, 121 -> 116 with 4; 64 x 12 460 -> 420 and
    // 432 -> 398 (513 to 592 keys, 1 to 64 images: 4 to 13 % everywhere).  With 128 registers 14 are spilled
    // (P of 8 bits; 3 otherwise), with the 64 of the other form 18 (2).
    if constexpr (SB == 8) {
        static_assert(16 * KEEP <= 512, "kept tiles of real keys only");
        if (lds > 80 * 1024) return launch_stream_keep<SB, P8, LUT, KEEP>(p, lds, stream);
    }
    return launch_stream_keep<SB, P8, LUT, 0>(p, lds, stream);
}

template <int SB>
hipError_t launch_stream_p(const AttnParams &p, hipStream_t stream) {
    if (p.pmax > 127) return launch_stream<SB, true, false>(p, stream);
    if constexpr (SB == 4) {                              // (the table of exponentials is one of 4-bit operands)
        if (p.lut_n > 0) return launch_stream<SB, false, true>(p, stream);
    }
    return launch_stream<SB, false, false>(p, stream);
}

}  // namespace

#ifndef VITQ_STREAM_MIN_N
#define VITQ_STREAM_MIN_N 209
#endif
hipError_t attention_launch(const AttnParams &p, AttnMode mode, hipStream_t stream) {
    if (p.B * p.H == 0) return hipSuccess;
    // fused attention with packed output only: long rows take the streaming form
    if (mode == kAttnFused && p.oq && !p.o_acc_out && !p.o_out && p.N >= VITQ_STREAM_MIN_N && p.N <= 37 * 16) {
        if (p.sb == 4) return launch_stream_p<4>(p, stream);
        if (p.sb == 8) return launch_stream_p<8>(p, stream);
    }
    if (p.N <= 13 * 16) {
        if (p.sb == 4) return launch_mode<13, 4>(p, mode, stream);
        if (p.sb == 8) return launch_mode<13, 8>(p, mode, stream);
    } else if (p.N <= 37 * 16) {
        if (p.sb == 4) return launch_mode<37, 4>(p, mode, stream);
        if (p.sb == 8) return launch_mode<37, 8>(p, mode, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace vitq
