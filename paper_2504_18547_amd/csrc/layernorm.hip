// LayerNorm followed by a quantizer, without division by sigma and without square root
// (Sec. IV-C, Eq. 5, Fig. 5).
//
// Phase 1 -- row statistics.  They are the incremental recurrences of Eq. 5 in fp32, elements in
// order: that order is part of the definition (fp32 addition does not associate), so one LANE
// walks one row.  What bounds it is the serial chain: a wave issues one VALU instruction per 8.5
// cycles, dependent or not, so the time is (instructions per element of the busiest wave) x 8.5
// cycles x columns whatever the number of rows.  The work of a step is therefore dealt to three
// waves of the workgroup that run one chunk of CH columns apart:
//   walker      mu_i = mu_{i-1} + (x_i - mu_{i-1}) / i        (four instructions; leaves mu_i in LDS)
//   accumulator M_i  = M_{i-1} + (x_i - mu_{i-1}) * (x_i - mu_i)      (four)
//   checker     smallest nonzero |x_i - mu_{i-1}|: is the division-free step exact?   (four)
// while four more waves bring the rows in, coalesced, several chunks ahead.
// Phase 2 -- levels.  The quantizer is the comparator of Fig. 5(b): the level is the number of
// references (k - 1/2)*step that the normalised value exceeds, each decided as
//     ssq((x - mu) * gamma) * n  >  ssq((k - 1/2)*step - beta) * V,      ssq(v) = v * |v|,
// V = M_n + n*eps the (stabilised) sum of squared deviations -- sigma never appears.  Elements
// are independent here, so the workgroup's rows are re-read (from L2; rows of up to 128 columns from
// LDS, where they still are) by all waves with coalesced 16-byte loads, four elements per lane, two to four
// rows of a wave per pass.  The comparisons are monotone in k, so
// instead of all 2^b - 1 of them the kernel makes a guess with the hardware reciprocal square
// root.  A guess that lies further from every half-integer than the proven distance between the
// guess and the comparator's own boundary stands as it is; otherwise the comparator itself is
// evaluated at the guessed level and the one above, stepping the guess until both agree, and
// every decision is the comparator's.
#include "layernorm.h"
#include <type_traits>
#include "launch_util.h"
#include "vitq_dev.h"

namespace vitq {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

// 1/k, k = 1 .. kRkMax, as hi + lo: hi = RN(1/k), lo = RN(1/k - hi), evaluated by the compiler.  Then
//     t = RN(d*lo),  q = RN(d*hi + t)          (a multiply and an FMA)
// equals RN(d/k) for every fp32 d with 2^-98 <= |d| and a finite result, and for d = 0: hi + lo and the
// rounding of t are off by at most 2^-48 of the quotient together (2^-39 where t is subnormal), while d/k is
// never the midpoint of two neighbouring fp32 numbers (a midpoint has a 25-bit odd significand, which would
// have to divide the 24-bit one of d) and never closer to one than 1/(2k) of their distance, i.e. 2^-37 of
// the quotient for k <= 4096.  (tests/test_division_free_mean_update.py runs a slice of that space.)  An infinite or NaN d
// gives a mean that is not finite from then on.
constexpr int kRkMax = 4096;
struct alignas(64) RkTable {       // (hi, lo) of 1/k at 2*(k - 1)
    float v[2 * kRkMax];
    constexpr RkTable() : v{} {
        for (int k = 1; k <= kRkMax; ++k) {
            const float hi = 1.0f / (float)k;
            v[2 * (k - 1)] = hi;
            v[2 * (k - 1) + 1] = (float)((1.0 - (double)hi * (double)k) / (double)k);      // (the difference is exact)
        }
    }
};
__device__ const RkTable g_rk{};
constexpr float kRkMinDev = 0x1p-98f;  // smallest nonzero deviation for which the two-step quotient is proven

constexpr float kLnGuard = 0x1p-21f;   // unit of the guard that lets a guessed level stand without the comparator
constexpr int kLnWaves = 7, kLnLoaders = 4;   // waves per workgroup: walker, accumulator, checker and the loading ones
constexpr int kLnCols = 32;            // columns per chunk (128 bytes of a row)
constexpr int kDepth = 3;              // chunks a loading wave holds in registers (in flight) ahead of LDS
constexpr int kXBufs = 4, kMBufs = 2;  // chunks of rows / of running means in LDS
enum LnMode { kLnVec = 0, kLnRes = 1, kLnScalar = 2 };       // 16-byte loads without / with residual or sum; element loads

// The definition's own walk of one row (division), for rows outside the fast step's range.
__device__ __forceinline__ float2 ln_walk_row(const float *xr, const float *rr, int cols) {
    float mu = 0.0f, m2 = 0.0f;
#pragma unroll 2
    for (int j = 0; j < cols; ++j) {
        float t = xr[j];
        if (rr) t = t + rr[j];
        const float d1 = t - mu;
        mu = mu + d1 / (float)(j + 1);
        const float d2 = t - mu;
        const float pr = d1 * d2;
        m2 = m2 + pr;
    }
    return make_float2(mu, m2);
}

// Levels of columns c0 .. c0 + 3 of a row by the comparator, one byte each, biased by -qmin.  level = qmin +
// #{lv : above(lv)}; above() is monotone in lv, so c is the level iff above(c) (or c == qmin) and not above(c + 1) (or
// c == qmax).  st: mean, guess of 1/(sigma*step), -, V.  For rows without a residual.
__device__ __forceinline__ u32 ln_compare(const LnParams &p, int64_t row, int c0, const float4 &st, float rstep) {
    const int cols = (int)p.cols;
    const float nf = (float)cols, V = st.w, qminf = (float)p.qmin, qmaxf = (float)p.qmax;
    float L[4], bt[4], lv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = min(c0 + i, cols - 1);
        const float a = p.x[row * p.ld + c] - st.x;
        const float g = a * p.gamma[c];
        bt[i] = p.beta[c];
        const float gs = g * fabsf(g);
        L[i] = gs * nf;
        lv[i] = fminf(fmaxf(rintf(fmaf(g, st.y, bt[i] * rstep)), qminf), qmaxf);             // (NaN: qmin)
    }
    auto above = [&](int i, float k) {                    // comparator of Fig. 5(b)
        const float rk = (k - 0.5f) * p.step;
        const float cc = rk - bt[i];
        const float cs = cc * fabsf(cc);
        const float rhs = cs * V;
        return L[i] > rhs;
    };
    for (int it = 0; it <= p.qmax - p.qmin; ++it) {
        bool moved = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool low_ok = (lv[i] <= qminf) || above(i, lv[i]);
            const bool high_ok = (lv[i] >= qmaxf) || !above(i, lv[i] + 1.0f);
            const float d = !low_ok ? -1.0f : (!high_ok ? 1.0f : 0.0f);
            lv[i] = lv[i] + d;
            moved = moved || d != 0.0f;
        }
        if (__builtin_amdgcn_ballot_w64(moved) == 0) break;
    }
    u32 w = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) w |= (u32)(int)(lv[i] - qminf) << (8 * i);
    return w;
}

// What the level pass needs of a row: mean, guess of 1/(sigma*step), 0 (or infinity: no guess), V.  In a row whose V is
// not an ordinary number every element is compared.
__device__ __forceinline__ float4 ln_row_stats(const LnParams &p, float mu, float m2, float rstep) {
    const float nf = (float)(int)p.cols;
    const float ne = nf * p.eps;
    const float V = m2 + ne;
    const bool plain = V >= 0x1p-40f && V <= 0x1p30f && p.step >= 0x1p-20f && p.step <= 0x1p10f;
    return make_float4(mu, __builtin_amdgcn_rsqf(V / nf) * rstep, plain ? 0.0f : __uint_as_float(0x7F800000u), V);
}

// R rows per workgroup: see layernorm_quantize_launch.
// SHORT: rows of at most kXBufs chunks (128 columns).  There the level pass is what bounds the call: three
// round trips to memory for rows that LDS still holds, and 8 to 32 of a wave's 64 lanes at work.  So the rows
// stay in LDS and a wave decides 64 >> gsh of them side by side.  us, one walk per lane on one wave / seven
// waves without this / with it: 400,000 x 16 8-bit 58 / 76 / 41, 400,000 x 128 83 / 93 / 76,
// 100,000 x 31 37 / 40 / 26, 197 x 128 13.1 / 6.2 / 5.8.  (One row of under 32 columns is where the
// first is still ahead, by 0.3 to 1 us: nothing there hides the hand-over between the waves.)
// A chunk in LDS: 16-byte group c (four columns) of row r at c * (R + 1) + r, so that a wave reads one group of
// its rows contiguously, at offsets from one base that are compile-time constants.
template <int MODE, int SB, int R, bool SHORT>
__global__ __launch_bounds__(kLnWaves * 64, 6) void layernorm_quantize_kernel(LnParams p) {
    constexpr int CH = kLnCols, NW = kLnWaves, LW = kLnLoaders;
    constexpr int kGroups = CH / 4, CQ = kGroups * (R + 1);
    constexpr bool VEC = MODE != kLnScalar;
    static_assert(NW == 3 + LW && R <= 64 && CH % 16 == 0 && kRkMax % CH == 0, "roles");
    __shared__ __attribute__((aligned(16))) float4 s_ln[(kXBufs + kMBufs) * CQ];
    float4 *s_x = s_ln;                                   // [kXBufs] chunks of rows
    float4 *s_m = s_ln + kXBufs * CQ;                     // [kMBufs] chunks of running means
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int cols = (int)p.cols;
    const float nf = (float)cols;

    // ---- phase 1: Eq. 5, mu_i = mu_{i-1} + (x_i - mu_{i-1}) / i,
    //                     M_i  = M_{i-1}  + (x_i - mu_{i-1}) * (x_i - mu_i)
    // The roles rotate with the workgroup index (of the workgroups of one XCD, which arrive at a CU in
    // steps of its 32 CUs), so that the workgroups sharing a CU walk their rows on different SIMDs.
    const int role = (int)(((u32)wave + (blockIdx.x >> 3) + (blockIdx.x >> 8)) % (u32)NW);
    const int nch = (cols + CH - 1) / CH;
    const int lr = min(lane, R - 1);
    float mu = 0.0f, m2 = 0.0f;
    u32 least = 0xFFFFFFFFu;                              // bits of the smallest nonzero deviation, minus one
    // Step t, between two barriers: chunk t is walked, chunk t - 1 accumulated and checked, chunk t + 2 put
    // into LDS (chunk t + 1 is there: the walker fetches it into registers as it consumes chunk t).  Every
    // role passes the same nch + 2 barriers.
    if (role == 0) {
        __syncthreads();
        float4 x[kGroups];
#pragma unroll
        for (int c = 0; c < kGroups; ++c) x[c] = s_x[c * (R + 1) + lr];
        typedef __attribute__((address_space(4))) const v16f const_v16f;      // (constant memory: scalar loads)
        uint64_t rk = reinterpret_cast<uint64_t>(g_rk.v);
        asm("" : "+s"(rk));                               // (one address computation, not one per load)
        v16f k16[CH / 8];
        auto load_rk = [&](int g, int t) {                // (a chunk beyond the table divides instead)
            k16[g] = reinterpret_cast<const_v16f *>(rk)[(CH / 8) * min(t, kRkMax / CH - 1) + g];
        };
#pragma unroll
        for (int g = 0; g < CH / 8; ++g) load_rk(g, 0);
        for (int t = 0; t <= nch; ++t) {
            if (t < nch) {
                const float4 *next = s_x + ((t + 1) % kXBufs) * CQ + lr;
                float4 *dst = s_m + (t % kMBufs) * CQ + lr;
                const int n = min(cols - t * CH, CH);
                if (n == CH && (t + 1) * CH <= kRkMax) {
#pragma unroll
                    for (int c = 0; c < kGroups; ++c) {
                        auto step = [&](float xv, int i) {
                            const float d1 = xv - mu;
                            const float tq = d1 * k16[c >> 1][8 * (c & 1) + 2 * i + 1];
                            mu = mu + fmaf(d1, k16[c >> 1][8 * (c & 1) + 2 * i], tq);
                            return mu;
                        };
                        float4 m;
                        m.x = step(x[c].x, 0); m.y = step(x[c].y, 1); m.z = step(x[c].z, 2); m.w = step(x[c].w, 3);
                        __builtin_amdgcn_sched_barrier(0);
                        dst[c * (R + 1)] = m;
                        x[c] = next[c * (R + 1)];
                        if (c & 1) load_rk(c >> 1, t + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {                                  // a last partial chunk, or one beyond the table
                    const float *xs = reinterpret_cast<const float *>(s_x + (t % kXBufs) * CQ + lr);
                    for (int i = 0; i < n; ++i) {
                        const float xv = xs[(i >> 2) * 4 * (R + 1) + (i & 3)];
                        const float d1 = xv - mu;
                        mu = mu + d1 / (float)(t * CH + i + 1);
                        reinterpret_cast<float *>(dst)[(i >> 2) * 4 * (R + 1) + (i & 3)] = mu;
                    }
#pragma unroll
                    for (int c = 0; c < kGroups; ++c) x[c] = next[c * (R + 1)];
                }
            }
            __syncthreads();
        }
    } else if (role == 1 || role == 2) {
        auto run = [&](auto &&f) {
            __syncthreads();
            __syncthreads();
            for (int t = 0; t < nch; ++t) {
                const float4 *src = s_x + (t % kXBufs) * CQ + lr;
                const float4 *msrc = s_m + (t % kMBufs) * CQ + lr;
                const int n = min(cols - t * CH, CH);
                if (n == CH) {
#pragma unroll
                    for (int c = 0; c < kGroups; ++c) {
                        const float4 x = src[c * (R + 1)], m = msrc[c * (R + 1)];
                        f(x.x, m.x); f(x.y, m.y); f(x.z, m.z); f(x.w, m.w);
                    }
                } else {
                    for (int i = 0; i < n; ++i)
                        f(reinterpret_cast<const float *>(src)[(i >> 2) * 4 * (R + 1) + (i & 3)],
                          reinterpret_cast<const float *>(msrc)[(i >> 2) * 4 * (R + 1) + (i & 3)]);
                }
                __syncthreads();
            }
        };
        if (role == 1)
            run([&](float x, float m) {
                const float d1 = x - mu;                  // (mu: the mean before this element)
                const float d2 = x - m;
                const float pr = d1 * d2;
                m2 = m2 + pr;
                mu = m;
            });
        else
            run([&](float x, float m) {
                const float d1 = x - mu;                  // (zero wraps to the largest value)
                least = min(least, (__float_as_uint(d1) & 0x7FFFFFFFu) - 1u);
                mu = m;
            });
    } else {
        // loading waves: each lane brings one or two 16-byte groups of a chunk (chunks of 128-byte row pieces)
        constexpr int ITEMS = R * kGroups, LT = LW * 64, IT = (ITEMS + LT - 1) / LT;
        static_assert(ITEMS % LT == 0 || IT == 1, "items of the loading waves");
        const int lt = (role - 3) * 64 + lane;
        const bool loader = role < 3 + LW && (role - 3) * 64 < ITEMS;      // (wave-uniform)
        // Rows and columns beyond the matrix are clamped (what they bring is never used): unconditional loads
        // keep the compiler's count of what is in flight, so that a put waits for its own chunk only.
        struct Piece { float4 x[IT], r[MODE == kLnRes ? IT : 1]; };
        int64_t at[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it)
            at[it] = min(row0 + (it * LT + lt) / kGroups, p.rows - 1) * p.ld;
        auto fetch = [&](int ch, Piece &v) {
            const int c = min(ch, nch - 1) * CH + 4 * (lt % kGroups);
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                if constexpr (MODE == kLnScalar) {
                    float e[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int64_t i = at[it] + min(c + j, cols - 1);
                        e[j] = p.res ? p.x[i] + p.res[i] : p.x[i];
                    }
                    v.x[it] = make_float4(e[0], e[1], e[2], e[3]);
                } else {
                    const int64_t i = at[it] + min(c, cols - 4);
                    v.x[it] = *reinterpret_cast<const float4 *>(p.x + i);
                    if constexpr (MODE == kLnRes) v.r[it] = *reinterpret_cast<const float4 *>((p.res ? p.res : p.x) + i);
                }
            }
        };
        auto put = [&](int ch, const Piece &v) {
            if (SHORT && ch >= nch) return;
            float4 *dst = s_x + (ch % kXBufs) * CQ;
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int i = it * LT + lt;
                float4 a = v.x[it];
                if (MODE == kLnRes && p.res) {
                    a.x = a.x + v.r[it].x; a.y = a.y + v.r[it].y; a.z = a.z + v.r[it].z; a.w = a.w + v.r[it].w;
                }
                dst[(i % kGroups) * (R + 1) + i / kGroups] = a;
            }
        };
        if (loader) {
            Piece pre[kDepth];
            static_for<kDepth>([&](auto D) { fetch(decltype(D)::value, pre[decltype(D)::value]); });
            put(0, pre[0]);
            fetch(kDepth, pre[0]);
            put(1, pre[1]);
            fetch(kDepth + 1, pre[1]);
            __syncthreads();
            // step t stores chunk t + 2, held in pre[(t + 2) % kDepth] (past the last chunk: into a free buffer,
            // or, if the rows stay, not at all)
            int t = 0;
            for (; t + kDepth <= nch + 1; t += kDepth)
                static_for<kDepth>([&](auto D) {
                    constexpr int d = decltype(D)::value, slot = (d + 2) % kDepth;
                    put(t + d + 2, pre[slot]);
                    fetch(t + d + 2 + kDepth, pre[slot]);
                    __syncthreads();
                });
            static_for<kDepth - 1>([&](auto D) {
                constexpr int d = decltype(D)::value, slot = (d + 2) % kDepth;
                if (t + d <= nch) {
                    put(t + d + 2, pre[slot]);
                    __syncthreads();
                }
            });
        } else {
            for (int t = 0; t < nch + 2; ++t) __syncthreads();
        }
    }
    // ---- phase 2: levels.  A pass covers BL blocks of 256 columns: lane l owns columns c0..c0+3 of each, a
    // wave every NW-th row; a pass's loads go out together, the first pass's before the statistics are
    // exchanged. ----
    constexpr int ROWS = (R + NW - 1) / NW;               // rows of a wave
    constexpr int HALVES = (ROWS + 3) / 4;                // (many rows: a part of them per pass)
    constexpr int NB = SHORT ? 2 : (ROWS + HALVES - 1) / HALVES;      // of them per pass
    constexpr int BL = NB <= 3 && !SHORT ? 2 : 1;
    const int nrows = (int)min((int64_t)R, p.rows - row0);
    const int padded = p.row_bytes16 * 8 / SB;            // columns of the 16-byte padded row
    // (SHORT: a row takes 1 << gsh lanes)
    const int gsh = !SHORT ? 6 : padded <= 16 ? 2 : padded <= 32 ? 3 : padded <= 64 ? 4 : 5;
    const int gl = lane & ((1 << gsh) - 1);               // this lane's group of four columns
    float4 xv[BL][NB], gv[BL], bv[BL];
    auto row_of = [&](int pass, int k) {
        if constexpr (SHORT) return ((wave + NW * (k + NB * pass)) << (6 - gsh)) + (lane >> gsh);
        else return wave + NW * (k + NB * (pass % HALVES));
    };
    auto element = [&](int64_t at, int c) {
        float t = p.x[at + c];
        if (p.res) t = t + p.res[at + c];
        return t;
    };
    // 16 bytes at a uniform base plus a 32-bit lane offset.  (A 16-byte load takes any 4-byte aligned address:
    // gamma and beta need no more, while rows that are not 16-byte aligned go element by element.  With
    // gamma off by 4 bytes, 50,432 x 768: 140 us element by element, 72 like this.)
    typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
    auto load4 = [](const float *base, u32 off) {
        const v4f_any v = *reinterpret_cast<const v4f_any *>(reinterpret_cast<const char *>(base) + off);
        return make_float4(v.x, v.y, v.z, v.w);
    };
    auto load_params = [&](int c0, int bl) {
        if constexpr (VEC) {
            gv[bl] = load4(p.gamma, 4u * (u32)min(c0, cols - 4));
            bv[bl] = load4(p.beta, 4u * (u32)min(c0, cols - 4));
        } else {
            const int c[4] = {min(c0, cols - 1), min(c0 + 1, cols - 1), min(c0 + 2, cols - 1), min(c0 + 3, cols - 1)};
            gv[bl] = make_float4(p.gamma[c[0]], p.gamma[c[1]], p.gamma[c[2]], p.gamma[c[3]]);
            bv[bl] = make_float4(p.beta[c[0]], p.beta[c[1]], p.beta[c[2]], p.beta[c[3]]);
        }
    };
    auto load_pass = [&](int pass) {                      // (columns and rows beyond the matrix: clamped, not used)
        int64_t at[NB];
        int r = min(row_of(pass, 0), nrows - 1);
        at[0] = (row0 + r) * p.ld;
        [[maybe_unused]] const int grp = min(gl, nch * kGroups - 1);
#pragma unroll
        for (int k = 1; k < NB; ++k) {
            const bool more = r + NW < nrows;
            at[k] = at[k - 1] + (more ? NW * p.ld : 0);
            r += more ? NW : 0;
        }
#pragma unroll
        for (int bl = 0; bl < BL; ++bl) {
            const int c0 = 4 * gl + (SHORT ? 0 : 256 * (pass / HALVES * BL + bl));
            [[maybe_unused]] const int c[4] = {min(c0, cols - 1), min(c0 + 1, cols - 1), min(c0 + 2, cols - 1), min(c0 + 3, cols - 1)};
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                float4 &v = xv[bl][k];
                if constexpr (SHORT) {
                    v = s_x[(grp / kGroups) * CQ + (grp % kGroups) * (R + 1) + min(row_of(pass, k), nrows - 1)];
                } else if constexpr (VEC) {
                    const u32 cv = 4u * (u32)min(c0, cols - 4);
                    v = load4(p.x + at[k], cv);
                    if constexpr (MODE == kLnRes) {
                        if (p.res) {
                            const float4 r4 = load4(p.res + at[k], cv);
                            v.x = v.x + r4.x; v.y = v.y + r4.y; v.z = v.z + r4.z; v.w = v.w + r4.w;
                        }
                    }
                } else {
                    v = make_float4(element(at[k], c[0]), element(at[k], c[1]), element(at[k], c[2]), element(at[k], c[3]));
                }
            }
            load_params(c0, bl);
        }
    };
    load_pass(0);

    // the running means are done with: their LDS holds the statistics from here on
    float4 *s_row = s_m;                                  // [R] mean, guess of 1/(sigma*step), 0 (or infinity: no guess), V
    float *s_m2 = reinterpret_cast<float *>(s_m + R);     // [R] sum of squared deviations
    u32 *s_least = reinterpret_cast<u32 *>(s_m2 + R);
    if (lane < R) {
        if (role == 1) s_m2[lane] = m2;
        else if (role == 2) s_least[lane] = least;
    }
    __syncthreads();
    const float rstep = __builtin_amdgcn_rcpf(p.step);    // for the guess only
    if (role == 0 && lane < nrows) {
        m2 = s_m2[lane];
        // (a deviation too small for the two-step quotient, or anything that is not finite: divide)
        const bool ok = fabsf(mu) <= 3.0e38f && s_least[lane] >= __float_as_uint(kRkMinDev) - 1u;
        if (!ok) {
            const float2 st = ln_walk_row(p.x + (row0 + lane) * p.ld, p.res ? p.res + (row0 + lane) * p.ld : nullptr, cols);
            mu = st.x;
            m2 = st.y;
        }
        const float ne = nf * p.eps;
        const float V = m2 + ne;
        // in a row whose V is not an ordinary number every element is compared
        const bool plain = V >= 0x1p-40f && V <= 0x1p30f && p.step >= 0x1p-20f && p.step <= 0x1p10f;
        s_row[lane] = make_float4(mu, __builtin_amdgcn_rsqf(V / nf) * rstep, plain ? 0.0f : __uint_as_float(0x7F800000u), V);
    }
    __syncthreads();

    // The guess.  In exact arithmetic on the fp32 values g, beta, step, V the comparator asks whether
    // t* = (g / sigma + beta) / step exceeds lv - 1/2 (sigma^2 = V/n).  The value tp computed here with the
    // hardware rsq / rcp, tp = g * (rs*rstep) + beta*rstep, differs from t* by at most
    // (|g/(sigma*step)| + |beta/step|) * 2^-21, and the comparator's own fp32 evaluation moves its boundary by at
    // most (2|lv| + |beta/step| + 1) * 2^-22 (five roundings on the two sides, two of them doubled by the
    // squares).  So when tp is further than kLnGuard * (4|tp| + 3|beta/step| + 3) from every half-integer, the
    // rounded tp is the level the comparator would count, and the comparator is not run.  With at most 4-bit
    // fields |tp| is taken as 8.5, which holds wherever a boundary is near (beyond it the level is the clamp on
    // both sides), and the bias -qmin rides in the FMA's addend (two more roundings of values below 16: 2
    // units); with 8-bit fields the lane's largest |tp| is used.  (A NaN tp drops out of the maxima, but then the
    // row's guess is marked infinite, or a gamma or beta is not finite and the limit is NaN.)
    // The relative-error model behind these bounds needs the squares to stay
    // ordinary numbers: the guess is trusted only for 2^-20 <= step <= 2^10 and 2^-40 <= V <= 2^30 (then an
    // underflowing g*|g| can differ from the exact product by 2^-139 at most, against
    // |L - R| >= V * step^2 * d^2 for a value d levels from a boundary, and nothing overflows below the |tp|
    // that the guard itself rejects).
    const float qminf = (float)p.qmin, qmaxf = (float)p.qmax;
    const float top = qmaxf - qminf;
    const u32 unbias = (u32)(p.qmin & ((1 << SB) - 1)) * 0x01010101u;    // added per byte: level - qmin -> field
    [[maybe_unused]] auto d8 = [&](float t) { return rintf(t) - qminf; };      // (rounded first: adding the bias would round again)
    // packs the four levels (one byte each, biased by -qmin) of columns c0.. of a row and stores them
    uint8_t *const out0 = p.out + row0 * p.out_stride;
    auto store_levels = [&](int r, int c0, u32 w) {       // (without SHORT r is uniform, the 64-bit product scalar)
        uint8_t *dst = out0 + r * p.out_stride + (u32)(c0 * SB / 8);
        if constexpr (SB == 8) w = ((w & 0x7F7F7F7Fu) + (unbias & 0x7F7F7F7Fu)) ^ ((w ^ unbias) & 0x80808080u);
        else w = (w + unbias) & (((1u << SB) - 1u) * 0x01010101u);
        if (padded != cols) {                             // zeros beyond the last column
            const int live = cols - c0;
            if (live < 4) w &= live <= 0 ? 0u : ((1u << (8 * live)) - 1u);
        }
        if constexpr (SB == 8) *reinterpret_cast<u32 *>(dst) = w;
        else if constexpr (SB == 4)
            *reinterpret_cast<uint16_t *>(dst) = (uint16_t)__builtin_amdgcn_perm(0u, w | (w >> 4), 0x0C0C0200u);
        else *dst = (uint8_t)(w | (w >> 6) | (w >> 12) | (w >> 18));
    };
    for (int pass = 0; SHORT ? row_of(pass, 0) - (lane >> gsh) < nrows : pass / HALVES * BL * 256 < padded; ++pass) {
        if (pass > 0) load_pass(pass);
        u32 redo = 0;                                     // (wave-uniform) items to be decided by the comparator
        static_for<BL>([&](auto BLK) {
            constexpr int bl = decltype(BLK)::value;
            const int c0 = 4 * gl + (SHORT ? 0 : 256 * (pass / HALVES * BL + bl));
            if (c0 >= padded) return;
            const float gm[4] = {gv[bl].x, gv[bl].y, gv[bl].z, gv[bl].w}, bt[4] = {bv[bl].x, bv[bl].y, bv[bl].z, bv[bl].w};
            float btr[4], bmax = 0.0f, odd = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                btr[i] = SB == 8 ? bt[i] * rstep : fmaf(bt[i], rstep, -qminf);
                bmax = fmaxf(bmax, fabsf(bt[i] * rstep));
                odd = odd + (gm[i] - gm[i]) + (bt[i] - bt[i]);           // NaN unless all of them are finite
            }
            const float limit = (0.5f - kLnGuard * (3.0f * bmax + (SB == 8 ? 3.0f : 39.0f))) + odd;
            static_for<NB>([&](auto K) {
                constexpr int k = decltype(K)::value;
                const int r = row_of(pass, k);
                __builtin_amdgcn_sched_barrier(0);        // (items in turn: bounds the registers)
                if (r < nrows) {
                    const float x[4] = {xv[bl][k].x, xv[bl][k].y, xv[bl][k].z, xv[bl][k].w};
                    const float4 st = s_row[r];
                    float tp[4], d[4];
                    u32 w = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float a = x[i] - st.x;
                        const float g = a * gm[i];
                        tp[i] = fmaf(g, st.y, btr[i]);
                        d[i] = tp[i] - rintf(tp[i]);
                        // (to nearest even, saturates to a byte)
                        const float lv = SB == 8 ? fminf(d8(tp[i]), top) : __builtin_amdgcn_fmed3f(tp[i], 0.0f, top);
                        w = __builtin_amdgcn_cvt_pk_u8_f32(lv, i, w);
                    }
                    const float far = fmaxf(fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fabsf(d[2])), fabsf(d[3]));
                    float fig = far + st.z;
                    if constexpr (SB == 8)
                        fig = fmaf(fmaxf(fmaxf(fmaxf(fabsf(tp[0]), fabsf(tp[1])), fabsf(tp[2])), fabsf(tp[3])), 4.0f * kLnGuard, fig);
                    if (__builtin_amdgcn_ballot_w64(!(fig <= limit)) != 0) redo |= 1u << (bl * NB + k);
                    store_levels(r, c0, w);
                    if constexpr (MODE != kLnVec) {
                        if (p.sum_out) {
                            float *so = p.sum_out + (row0 + r) * p.ld + c0;
                            if constexpr (VEC) {
                                if (c0 < cols) *reinterpret_cast<float4 *>(so) = xv[bl][k];
                            } else {
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    if (c0 + i < cols) so[i] = x[i];
                            }
                        }
                    }
                }
            });
        });
        // Rare: items with an element inside the guard (ln_compare's sequence, written out: calling it from here took this kernel
        // from 68.9 to 77.4 us at 50,432 x 768).  level = qmin + #{lv : above(lv)}; above() is monotone in
        // lv, so c is the level iff above(c) (or c == qmin) and not above(c + 1) (or c == qmax).
        while (redo) {
            const int item = __builtin_ctz(redo);
            redo &= redo - 1;
            const int c0 = 4 * gl + (SHORT ? 0 : 256 * (pass / HALVES * BL + item / NB)), r = row_of(pass, item % NB);
            if (c0 >= padded || r >= nrows) continue;
            const float4 st = s_row[r];
            const float V = st.w;
            const int c[4] = {c0, min(c0 + 1, cols - 1), min(c0 + 2, cols - 1), min(c0 + 3, cols - 1)};
            float L[4], bt[4], lv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t at = (row0 + r) * p.ld + min(c[i], cols - 1);
                const float x = MODE != kLnVec && p.sum_out ? p.sum_out[at] : (p.res ? p.x[at] + p.res[at] : p.x[at]);
                const float a = x - st.x;
                const float g = a * p.gamma[min(c[i], cols - 1)];
                bt[i] = p.beta[min(c[i], cols - 1)];
                const float gs = g * fabsf(g);
                L[i] = gs * nf;
                lv[i] = fminf(fmaxf(rintf(fmaf(g, st.y, bt[i] * rstep)), qminf), qmaxf);             // (NaN: qmin)
            }
            auto above = [&](int i, float k) {            // comparator of Fig. 5(b)
                const float rk = (k - 0.5f) * p.step;
                const float cc = rk - bt[i];
                const float cs = cc * fabsf(cc);
                const float rhs = cs * V;
                return L[i] > rhs;
            };
            for (int it = 0; it <= p.qmax - p.qmin; ++it) {
                bool moved = false;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool low_ok = (lv[i] <= qminf) || above(i, lv[i]);
                    const bool high_ok = (lv[i] >= qmaxf) || !above(i, lv[i] + 1.0f);
                    const float d = !low_ok ? -1.0f : (!high_ok ? 1.0f : 0.0f);
                    lv[i] = lv[i] + d;
                    moved = moved || d != 0.0f;
                }
                if (__builtin_amdgcn_ballot_w64(moved) == 0) break;
            }
            u32 w = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) w |= (u32)(int)(lv[i] - qminf) << (8 * i);
            store_levels(r, c0, w);
        }
    }
}

// ---- rows of 129 to 1152 columns without a residual: the workgroup's rows stay in registers -------------------
// One workgroup of sixteen waves per CU.  Twelve of them request all of the workgroup's rows at once and keep them,
// NP 16-byte pieces per lane, so that the level pass reads no memory, and the even deal of the rows over the CUs
// (up to R = 16, 32 or 64 of them: a wave's lanes walk one each) leaves no second round of workgroups half empty.
// What bounds the call is then the walker's chain, four dependent instructions per column of 4.3 cycles each, and
// everything else is kept off that wave, which issues an instruction per 4.3 cycles whatever it is: the operands of
// the next sixteen columns (row pieces from LDS, 1/i from scalar memory) are requested before the current sixteen
// are walked, and only every fourth mean leaves it, in one 16-byte write per sixteen columns (a wave that does nothing
// else: 17.4 cycles per column; with the reads 19.7, with the scalar loads 20.6, with all means written 27.4,
// with every fourth 22.5).  The lane that holds a piece repeats its four steps.
// A chunk is 1024 / R columns = 256 pieces, one per lane of a set of four loading waves; the three sets take the
// chunks in turn.  In step t chunk t is walked, the set of chunk t + 3 puts it into LDS, that of chunk t - 1 multiplies
// its deviations, and the adder sums the products of chunk t - 2 up in order.
// A chunk in LDS: 16-byte group c (four columns) of row r at c * (R + 1) + r.
// us per call, fp32 -> 4 bits, kernel above / this: 768 columns 197 rows 21.3 / 15.1, 4,096 21.6 / 15.2, 9,900 28.4 / 20.8,
// 12,608 32.3 / 22.0 (of it the walk 10.6, levels 4.1), 16,384 33.6 / 26.2; 384 columns 197 rows 13.0 / 10.0, 9,900
// 16.7 / 13.3; 1,024 columns 12,608 rows 40.0 / 29.4.
constexpr int kResWaves = 16, kResSets = 3;
constexpr int kResMaxCols = 1152;
// LDS: per-column parameters of the level pass, then the chunks, over which the packed rows are laid once they are done with
template <int R>
constexpr size_t kResRings = (size_t)6 * (256 / R) * (R + 1) * 16 + 4 * 1024;
template <int R>
size_t resident_lds(const LnParams &p) {
    const size_t groups = ((size_t)p.cols + 1024 / R - 1) / (1024 / R) * (256 / R), rows = (size_t)R * (p.row_bytes16 + 16);
    return groups * 68 + (rows > kResRings<R> ? rows : kResRings<R>) + 16;
}
template <int SB, int R, int NP>
__global__ __launch_bounds__(kResWaves * 64, 4) void layernorm_resident_kernel(LnParams p, int wg_rows) {
    constexpr int CH = 1024 / R, G = CH / 4, BPC = CH / 16, CQ = G * (R + 1);
    static_assert(R * G == 256 && CH % 16 == 0 && kResMaxCols <= kRkMax, "one piece per lane of a set");
    extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
    __shared__ __attribute__((aligned(16))) float4 s_row[R];
    __shared__ float s_m2[R];                             // sum of squared deviations
    __shared__ u32 s_least[R];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * wg_rows;
    const int nrows = (int)min((int64_t)wg_rows, p.rows - row0);
    const int cols = (int)p.cols;
    const int nch = (cols + CH - 1) / CH;
    float4 *const s_gm = reinterpret_cast<float4 *>(s_dyn), *const s_bt = s_gm + nch * G;     // gamma, beta (see below) of four columns
    float4 *const s_rk = s_bt + nch * G;                                                      // their (hi, lo) of 1/i: two each
    float *const s_limit = reinterpret_cast<float *>(s_rk + 2 * nch * G);
    float4 *const s_x = reinterpret_cast<float4 *>(s_dyn + ((nch * G * 68 + 15) & ~15));      // [4] chunks of rows
    float4 *const s_end = s_x + 4 * CQ;                   // [4] chunks: per batch and row, the mean after columns 4, 8, 12, 16
    float4 *const s_p = s_end + 4 * BPC * R;              // [2] chunks of products
    const float rstep = __builtin_amdgcn_rcpf(p.step);    // for the guess only
    const float qminf = (float)p.qmin;
    const float top = (float)p.qmax - qminf;
    float mu = 0.0f, m2 = 0.0f;
    // The rows of the workgroup, as the loading waves hold them: piece i of a lane is group g of chunk 3 * i + set.
    const int set = (wave >> 2) - 1;
    const int lt = (wave & 3) * 64 + lane;
    const int row = lt / G, g = lt % G;
    float4 x[NP];

    // Every wave passes the same nch + 4 barriers: behind the first three chunks, once more, and behind each of the
    // nch + 2 steps.
    const int steps = nch + 2;
    if (wave == 0) {
        if (lane < R) {
            __builtin_amdgcn_s_setprio(3);
            s_end[(3 * BPC + BPC - 1) * R + lane].w = 0.0f;                   // the mean before chunk 0
            __syncthreads();
            typedef __attribute__((address_space(4))) const v16f const_v16f;  // (constant memory: scalar loads)
            uint64_t rk = reinterpret_cast<uint64_t>(g_rk.v);
            asm("" : "+s"(rk));                           // (one address computation, not one per load)
            struct Batch { float4 x[4]; v16f k[2]; };     // sixteen columns: row pieces and (hi, lo) of 1/i
            Batch even, odd;
            auto fill = [&](int b, Batch &n) {
                const float4 *src = s_x + ((b / BPC) & 3) * CQ + (b % BPC) * 4 * (R + 1) + lane;
                const const_v16f *t = reinterpret_cast<const const_v16f *>(rk) + 2 * b;
                n.k[0] = t[0];
                n.k[1] = t[1];
#pragma unroll
                for (int i = 0; i < 4; ++i) n.x[i] = src[i * (R + 1)];
            };
            auto walk4 = [&](const Batch &n, auto I) {
                constexpr int i = decltype(I)::value;
                const float e[4] = {n.x[i].x, n.x[i].y, n.x[i].z, n.x[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d1 = e[j] - mu;
                    const float tq = d1 * n.k[i >> 1][8 * (i & 1) + 2 * j + 1];
                    mu = mu + fmaf(d1, n.k[i >> 1][8 * (i & 1) + 2 * j], tq);
                }
                return mu;
            };
            // One batch.  The barrier ahead of a chunk's step stands behind the first four columns of the chunk, and the
            // wait for the next batch's operands ahead of the last write: LDS and scalar loads share a counter that can
            // only be waited to zero, and all that it then waits for was sent off twelve columns earlier.
            auto batch = [&](int b, auto FIRST, const Batch &cur, Batch &next) {
                constexpr bool first = decltype(FIRST)::value;                // of its chunk
                const int c = b / BPC;
                float end[4];
                static_for<4>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    end[i] = walk4(cur, I);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (i == 0) {
                        if constexpr (first) __syncthreads();
                        fill(b + 1, next);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
                __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0)
                __builtin_amdgcn_sched_barrier(0);
                s_end[((c & 3) * BPC + b % BPC) * R + lane] = make_float4(end[0], end[1], end[2], end[3]);
                __builtin_amdgcn_sched_barrier(0);
            };
            using T = std::true_type;
            using F = std::false_type;
            const int fast = cols / CH;                   // whole chunks
            int c = 0;
            fill(0, even);
            __builtin_amdgcn_s_waitcnt(0xC07F);           // (here, so that the loop's head does not wait for the writes before it)
            if constexpr (BPC == 1) {
                for (; c + 2 <= fast; c += 2) {
                    batch(c, T{}, even, odd);
                    batch(c + 1, T{}, odd, even);
                }
                if (c < fast) batch(c++, T{}, even, odd);
            } else {
                for (; c < fast; ++c) {
                    const int b = c * BPC;
                    batch(b, T{}, even, odd);
                    batch(b + 1, F{}, odd, even);
                    if constexpr (BPC == 4) {
                        batch(b + 2, F{}, even, odd);
                        batch(b + 3, F{}, odd, even);
                    }
                }
            }
            if (c < nch) {                                // the columns' end inside a chunk
                __syncthreads();
                const int n = cols - c * CH;
                for (int j = 0; j < n / 16; ++j) {
                    fill(c * BPC + j, even);
                    float end[4];
                    static_for<4>([&](auto I) { end[decltype(I)::value] = walk4(even, I); });
                    s_end[((c & 3) * BPC + j) * R + lane] = make_float4(end[0], end[1], end[2], end[3]);
                }
                float *dst = reinterpret_cast<float *>(s_end + (c & 3) * BPC * R + lane);
                const float *src = reinterpret_cast<const float *>(s_x + (c & 3) * CQ + lane);
                for (int i = n & ~15; i < n; ++i) {
                    const float2 k = *reinterpret_cast<const float2 *>(g_rk.v + 2 * (c * CH + i));
                    const float d1 = src[(i >> 2) * 4 * (R + 1) + (i & 3)] - mu;
                    const float tq = d1 * k.y;
                    mu = mu + fmaf(d1, k.x, tq);
                    dst[(i >> 4) * 4 * R + ((i >> 2) & 3)] = mu;              // (the last one of four columns stays)
                }
            }
            __builtin_amdgcn_s_setprio(0);
            for (int t = 0; t < 3; ++t) __syncthreads();
        }
    } else if (wave == 1) {
        const int lr = min(lane, R - 1);
        for (int t = 0; t < 4; ++t) __syncthreads();
        for (int c = 0; c < nch; ++c) {
            const float4 *src = s_p + (c & 1) * CQ + lr;
            const int n = min(cols - c * CH, CH);
            if (n == CH) {
                float4 v[2][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[0][i] = src[i * (R + 1)];
#pragma unroll
                for (int j = 0; j < BPC; ++j) {
                    if (j + 1 < BPC) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[(j + 1) & 1][i] = src[(4 * (j + 1) + i) * (R + 1)];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float4 &a = v[j & 1][i];
                        m2 = m2 + a.x; m2 = m2 + a.y; m2 = m2 + a.z; m2 = m2 + a.w;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                for (int i = 0; i < n; ++i) m2 = m2 + reinterpret_cast<const float *>(src)[(i >> 2) * 4 * (R + 1) + (i & 3)];
            }
            __syncthreads();
        }
        if (lane < R) s_m2[lane] = m2;
    } else if (wave < 4) {
        // The guess of a level, tp = g * (rs*rstep) + beta*rstep, and the distance from every half-integer that makes
        // it the comparator's, are derived at the kernel above; the parts that depend on the column only are laid
        // out here for all rows: gamma, beta in steps (4-bit fields: counted from -qmin) and the limit.
        if (wave == 2) {
            for (int r = lane; r < R; r += 64) s_least[r] = 0xFFFFFFFFu;
        }
        for (int q = (wave & 1) * 64 + lane; q < 2 * nch * G; q += 128) s_rk[q] = reinterpret_cast<const float4 *>(g_rk.v)[q];
        __syncthreads();
        for (int q = (wave & 1) * 64 + lane; q < nch * G; q += 128) {
            float gm[4], bt[4], btr[4], bmax = 0.0f, odd = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                gm[i] = p.gamma[min(4 * q + i, cols - 1)];
                bt[i] = p.beta[min(4 * q + i, cols - 1)];
                btr[i] = SB == 8 ? bt[i] * rstep : fmaf(bt[i], rstep, -qminf);
                bmax = fmaxf(bmax, fabsf(bt[i] * rstep));
                odd = odd + (gm[i] - gm[i]) + (bt[i] - bt[i]);           // NaN unless all of them are finite
            }
            s_gm[q] = make_float4(gm[0], gm[1], gm[2], gm[3]);
            s_bt[q] = make_float4(btr[0], btr[1], btr[2], btr[3]);
            s_limit[q] = (0.5f - kLnGuard * (3.0f * bmax + (SB == 8 ? 3.0f : 39.0f))) + odd;
        }
        for (int t = 0; t < steps + 1; ++t) __syncthreads();
    } else {
        // (columns and rows beyond the matrix: clamped, not used)
        const float *src = p.x + (row0 + min(row, nrows - 1)) * p.ld;
        // A set would otherwise request all of its chunks before the next set requests its first.
        constexpr int PD = NP < 5 ? NP : 5;
        auto request = [&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i < NP)
                x[i] = *reinterpret_cast<const float4 *>(src + min((kResSets * i + set) * CH + 4 * g, cols - 4));
        };
        static_for<PD>([&](auto I) { request(I); });
        const int at = g * (R + 1) + row;
        // the mean before a piece: what the walker left four columns earlier (of the chunk before, for the first piece)
        const float *ends = reinterpret_cast<const float *>(s_end + row);
        const int before_at = g == 0 ? ((BPC - 1) * R * 4 + 3) : ((g - 1) >> 2) * R * 4 + ((g - 1) & 3);
        u32 least = 0xFFFFFFFFu;                          // twice the bits of the smallest nonzero deviation, minus one
        s_x[set * CQ + at] = x[0];
        __syncthreads();
        __syncthreads();
        int t = 0;
        for (; t < set; ++t) __syncthreads();
        // Three steps of the set at a time: chunk t + 3 = piece j + 1 is put, chunk t = piece j multiplied one step later.
        // (Nested rather than in sequence: no path joins another one, so the compiler counts the loads in flight.)
        auto three_steps = [&](auto &&self, auto J) __attribute__((always_inline)) -> void {
            constexpr int j = decltype(J)::value;
            if (t >= steps) return;
            if constexpr (j + 1 < NP) s_x[((t + 3) & 3) * CQ + at] = x[j + 1];
            request(std::integral_constant<int, j + PD>{});
            __syncthreads();
            if (t + 1 >= steps) return;
            if constexpr (j < NP) {
                const float4 v = x[j], k0 = s_rk[2 * (t * G + g)], k1 = s_rk[2 * (t * G + g) + 1];
                float m = ends[((g == 0 ? t - 1 : t) & 3) * BPC * R * 4 + before_at];
                const float e[4] = {v.x, v.y, v.z, v.w}, hi[4] = {k0.x, k0.z, k1.x, k1.z}, lo[4] = {k0.y, k0.w, k1.y, k1.w};
                float pr[4];
                u32 l[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float d1 = e[i] - m;
                    const float tq = d1 * lo[i];
                    m = m + fmaf(d1, hi[i], tq);
                    const float d2 = e[i] - m;
                    pr[i] = d1 * d2;
                    l[i] = (__float_as_uint(d1) << 1) - 1u;                      // (zero wraps to the largest value)
                }
                s_p[(t & 1) * CQ + at] = make_float4(pr[0], pr[1], pr[2], pr[3]);
                const u32 l4 = min(min(l[0], l[1]), min(l[2], l[3]));
                if (t * CH + 4 * g < cols) least = min(least, l4);
            }
            __syncthreads();
            if (t + 2 >= steps) return;
            __syncthreads();
            t += kResSets;
            if constexpr (j < NP) self(self, std::integral_constant<int, j + 1>{});
        };
        three_steps(three_steps, std::integral_constant<int, 0>{});
        atomicMin(&s_least[row], least);
    }
    __syncthreads();
    if (wave == 0 && lane < nrows) {
        m2 = s_m2[lane];
        // (a deviation too small for the two-step quotient, or anything that is not finite: divide)
        const bool ok = fabsf(mu) <= 3.0e38f && s_least[lane] >= 2u * __float_as_uint(kRkMinDev) - 1u;
        if (!ok) {
            const float2 st = ln_walk_row(p.x + (row0 + lane) * p.ld, nullptr, cols);
            mu = st.x;
            m2 = st.y;
        }
        s_row[lane] = ln_row_stats(p, mu, m2, rstep);
    }
    __syncthreads();

    // ---- levels, into packed rows over the chunks' LDS, and from there to memory in whole 16-byte pieces ----
    uint8_t *const s_out = reinterpret_cast<uint8_t *>(s_x);
    const int pitch = p.row_bytes16 + 16;                 // (spreads the rows over the banks)
    if (wave >= 4 && row < nrows) {
        const u32 unbias = (u32)(p.qmin & ((1 << SB) - 1)) * 0x01010101u;    // added per byte: level - qmin -> field
        auto store_levels = [&](int q, u32 w) {
            uint8_t *dst = s_out + row * pitch + q * (4 * SB / 8);
            if constexpr (SB == 8) {
                *reinterpret_cast<u32 *>(dst) = ((w & 0x7F7F7F7Fu) + (unbias & 0x7F7F7F7Fu)) ^ ((w ^ unbias) & 0x80808080u);
            } else {
                w = (w + unbias) & 0x0F0F0F0Fu;
                *reinterpret_cast<uint16_t *>(dst) = (uint16_t)__builtin_amdgcn_perm(0u, w | (w >> 4), 0x0C0C0200u);
            }
        };
        const float4 st = s_row[row];
        u32 redo = 0;                                     // pieces with an element inside the guard
        static_for<NP>([&](auto I) {
            constexpr int i = decltype(I)::value;
            const int q = (kResSets * i + set) * G + g;   // this piece's group of four columns
            if (4 * q < cols) {
                const float4 gm = s_gm[q], bt = s_bt[q];
                const float e[4] = {x[i].x, x[i].y, x[i].z, x[i].w}, gi[4] = {gm.x, gm.y, gm.z, gm.w}, bi[4] = {bt.x, bt.y, bt.z, bt.w};
                float tp[4], d[4];
                u32 w = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float a = e[k] - st.x;
                    const float gg = a * gi[k];
                    tp[k] = fmaf(gg, st.y, bi[k]);
                    d[k] = tp[k] - rintf(tp[k]);
                    // (to nearest even, saturates to a byte; 8-bit fields: rounded first, adding the bias would round again)
                    const float lv = SB == 8 ? fminf(rintf(tp[k]) - qminf, top) : __builtin_amdgcn_fmed3f(tp[k], 0.0f, top);
                    w = __builtin_amdgcn_cvt_pk_u8_f32(lv, k, w);
                }
                float fig = fmaxf(fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fabsf(d[2])), fabsf(d[3])) + st.z;
                if constexpr (SB == 8)
                    fig = fmaf(fmaxf(fmaxf(fmaxf(fabsf(tp[0]), fabsf(tp[1])), fabsf(tp[2])), fabsf(tp[3])), 4.0f * kLnGuard, fig);
                if (!(fig <= s_limit[q])) redo |= 1u << i;
                store_levels(q, w);
            }
        });
        while (__builtin_amdgcn_ballot_w64(redo != 0) != 0) {                   // (rare)
            if (redo != 0) {
                const int i = __builtin_ctz(redo);
                redo &= redo - 1;
                const int q = (kResSets * i + set) * G + g;
                store_levels(q, ln_compare(p, row0 + row, 4 * q, st, rstep));
            }
        }
    }
    __syncthreads();
    const int pieces = p.row_bytes16 / 16, live = cols * SB / 8;              // of a row; its bytes without the padding
    for (int r = wave; r < nrows; r += kResWaves)
        for (int i = lane; i < pieces; i += 64) {
            uint4 v = *reinterpret_cast<const uint4 *>(s_out + r * pitch + 16 * i);
            const int over = 16 * (i + 1) - live;         // bytes of padding in this piece: zeros
            if (over > 0) {
                auto word = [&](u32 w, int last) {        // last: bytes of the piece behind this word
                    const int pad = over - last;
                    return pad <= 0 ? w : (pad >= 4 ? 0u : w & (0xFFFFFFFFu >> (8 * pad)));
                };
                v = make_uint4(word(v.x, 12), word(v.y, 8), word(v.z, 4), word(v.w, 0));
            }
            *reinterpret_cast<uint4 *>(p.out + (row0 + r) * p.out_stride + 16 * i) = v;
        }
}

template <int SB, int R, int NP>
hipError_t launch_resident(const LnParams &p, int wg_rows, hipStream_t stream) {
    auto kern = layernorm_resident_kernel<SB, R, NP>;
    const size_t lds = resident_lds<R>(p);
    static std::atomic<uint64_t> allowed{0};              // (one per instantiation)
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), 128 * 1024, allowed);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((p.rows + wg_rows - 1) / wg_rows);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kResWaves * 64), lds, stream, p, wg_rows);
    return hipGetLastError();
}

// ---- per-head LayerNorm quantizer of Q and K, plain quantizer of V (Fig. 1(b), Table I) --------
// One lane owns one (token, head) group of 64 channels: it loads the 256 bytes once, runs Eq. 5
// over them and decides the 64 levels from registers (same guess-and-verify use of the
// comparator as above; the lanes are independent, so each stops stepping on its own), then
// writes the head-major packed row the attention kernel reads.  Groups are independent:
// M * 3H lanes of parallelism, no LDS.
template <int SB>
__global__ __launch_bounds__(256) void qkv_headnorm_kernel(HeadNormParams p) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int groups = 3 * p.H;
    const int64_t M = (int64_t)p.B * p.N;
    if (t >= M * groups) return;
    const int64_t m = t / groups;
    const int gi = (int)(t - m * groups);
    const int which = gi / p.H, h = gi - which * p.H;
    const int b = (int)(m / p.N), n = (int)(m - (int64_t)b * p.N);
    const float *src = p.y + m * p.ld + (int64_t)gi * 64;
    float v[64];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const float4 a = *reinterpret_cast<const float4 *>(src + 4 * q);
        v[4 * q] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
    }
    const float qminf = (float)p.qmin, qmaxf = (float)p.qmax;
    float lv[64];
    if (which == 2) {
#pragma unroll
        for (int i = 0; i < 64; ++i) lv[i] = (float)quantize_level(v[i], p.s_v, qminf, qmaxf);
    } else {
        float mu = 0.0f, m2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 64; ++i) {
            const float d1 = v[i] - mu;
            mu = mu + d1 / (float)(i + 1);
            const float d2 = v[i] - mu;
            const float pr = d1 * d2;
            m2 = m2 + pr;
        }
        const float nf = 64.0f;
        const float ne = nf * p.eps;
        const float V = m2 + ne;
        const float step = which == 0 ? p.s_q : p.s_k;
        const float rs = __builtin_amdgcn_rsqf(V / nf);          // for the guess only
        const float rstep = __builtin_amdgcn_rcpf(step);         // for the guess only
        const bool stats_ok = step >= 0x1p-20f && step <= 0x1p10f && V >= 0x1p-40f && V <= 0x1p30f;
        const int span = p.qmax - p.qmin;
        const float *gp = p.gamma + which * p.D + h * 64, *bp = p.beta + which * p.D + h * 64;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float4 g4 = *reinterpret_cast<const float4 *>(gp + 4 * q);
            const float4 b4 = *reinterpret_cast<const float4 *>(bp + 4 * q);
            const float gm[4] = {g4.x, g4.y, g4.z, g4.w}, bt[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float a = v[4 * q + i] - mu;
                const float g = a * gm[i];
                const float gs = g * fabsf(g);
                const float L = gs * nf;
                auto above = [&](float k) {
                    const float rk = (k - 0.5f) * step;
                    const float cc = rk - bt[i];
                    const float cs = cc * fabsf(cc);
                    const float R = cs * V;
                    return L > R;
                };
                // (the guess stands when it is provably far from every boundary: see the kernel above)
                const float tp = fmaf(g, rs, bt[i]) * rstep;
                const float tt = rintf(tp);
                float c = (tt == tt) ? __builtin_amdgcn_fmed3f(tt, qminf, qmaxf) : qminf;
                const float cgi = fmaf(fabsf(bt[i] * rstep), 3.0f * kLnGuard, 3.0f * kLnGuard);
                const float fig = fmaf(fabsf(tp), 4.0f * kLnGuard, fabsf(tp - tt)) + cgi;
                if (!(stats_ok && fig <= 0.5f)) {
                    for (int it = 0; it <= span; ++it) {
                        const bool low_ok = (c <= qminf) || above(c);
                        const bool high_ok = (c >= qmaxf) || !above(c + 1.0f);
                        if (low_ok && high_ok) break;
                        c = c + (!low_ok ? -1.0f : 1.0f);
                    }
                }
                lv[4 * q + i] = c;
            }
        }
    }
    const int64_t row = (((int64_t)which * p.B + b) * p.H + h) * p.N + n;
    uint8_t *dst = p.out + row * (64 * SB / 8);
    constexpr int PW = 32 / SB;                      // levels per 32-bit word
#pragma unroll
    for (int w4 = 0; w4 < 64 / PW / 4; ++w4) {
        u32 w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u32 acc = 0;
#pragma unroll
            for (int i = 0; i < PW; ++i)
                acc |= ((u32)(int)lv[(4 * w4 + j) * PW + i] & ((1u << SB) - 1u)) << (i * SB);
            w[j] = acc;
        }
        *reinterpret_cast<uint4 *>(dst + 16 * w4) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

}  // namespace

hipError_t qkv_headnorm_launch(const HeadNormParams &p, hipStream_t stream) {
    const int64_t threads = (int64_t)p.B * p.N * 3 * p.H;
    if (threads == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((threads + 255) / 256);
    if (p.sb == 4) hipLaunchKernelGGL(qkv_headnorm_kernel<4>, dim3(blocks), dim3(256), 0, stream, p);
    else if (p.sb == 8) hipLaunchKernelGGL(qkv_headnorm_kernel<8>, dim3(blocks), dim3(256), 0, stream, p);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t layernorm_quantize_launch(const LnParams &p, hipStream_t stream) {
    if (p.rows == 0) return hipSuccess;
    const bool vec = (p.cols % 4 == 0) && (p.ld % 4 == 0) && (((uintptr_t)p.x) % 16 == 0) &&
                     (!p.res || ((uintptr_t)p.res) % 16 == 0) && (!p.sum_out || ((uintptr_t)p.sum_out) % 16 == 0);
    // Rows that stay in registers (see layernorm_resident_kernel), as long as one round of workgroups takes them all: its
    // workgroup fills a CU, so a second round would begin when the first is through, and the kernel above, whose
    // workgroups overlap, is ahead or even there (18,000 x 384 20 us against 23, 25,216 x 768 40 and 41, 50,432 x 132 20 and 29).
    // At least four rows, one per SIMD in the level pass: with one row or sixteen 197 x 768 takes as long or 0.6 us more.
    constexpr int64_t kCUs = 256;
    if (vec && !p.res && !p.sum_out && (p.sb == 4 || p.sb == 8) && p.cols > kXBufs * kLnCols && p.cols <= kResMaxCols &&
        p.rows <= 64 * kCUs) {
        const int wg_rows = (int)max((int64_t)4, (p.rows + kCUs - 1) / kCUs);
        auto launch_pieces = [&](auto SB, auto ROWS) {
            constexpr int sb = decltype(SB)::value, R = decltype(ROWS)::value, unit = R / 8;
            if (p.cols <= kResMaxCols / 3) return launch_resident<sb, R, unit>(p, wg_rows, stream);
            if (p.cols <= 2 * kResMaxCols / 3) return launch_resident<sb, R, 2 * unit>(p, wg_rows, stream);
            return launch_resident<sb, R, 3 * unit>(p, wg_rows, stream);
        };
        auto launch_rows = [&](auto SB) {
            if (wg_rows <= 16) return launch_pieces(SB, std::integral_constant<int, 16>{});
            if (wg_rows <= 32) return launch_pieces(SB, std::integral_constant<int, 32>{});
            return launch_pieces(SB, std::integral_constant<int, 64>{});
        };
        return p.sb == 4 ? launch_rows(std::integral_constant<int, 4>{}) : launch_rows(std::integral_constant<int, 8>{});
    }
    // Rows per workgroup.  The recurrences take the same time for 16 rows as for 64 (a lane is a row); fewer rows
    // leave a wave fewer of them in the level pass and bring more CUs in, as long as every workgroup is resident:
    // three per CU (80 registers, 21 waves), so 12,288 and 24,576 rows are where one more round would begin.
    // Measured (768 columns, us; one lane per row with the division-sized step on one wave -> this kernel):
    // 197 rows 50 -> 19.5, 12,608 rows 59 -> 32, 25,216 rows 64 -> 40, 50,432 rows 76 -> 72, 100,000 rows 154 -> 117.
    const int64_t slots = 3 * 256;
    const int R = p.rows <= 16 * slots ? 16 : (p.rows <= 32 * slots ? 32 : 64);
    // A grid holds at most 2^32 - 1 work-items: more rows than that (613 million) go in several launches.
    constexpr int64_t kMaxBlocks = (int64_t)UINT32_MAX / (kLnWaves * 64);
    if (p.rows > kMaxBlocks * R) {
        for (int64_t row = 0; row < p.rows; row += kMaxBlocks * R) {
            LnParams part = p;
            part.rows = min(p.rows - row, kMaxBlocks * R);
            part.x = p.x + row * p.ld;
            if (p.res) part.res = p.res + row * p.ld;
            if (p.sum_out) part.sum_out = p.sum_out + row * p.ld;
            part.out = p.out + row * p.out_stride;
            const hipError_t e = layernorm_quantize_launch(part, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const unsigned blocks = (unsigned)((p.rows + R - 1) / R);
    auto launch = [&](auto M, auto SB) {
        constexpr int mode = decltype(M)::value, sb = decltype(SB)::value;
        auto launch_rows = [&](auto ROWS) {
            constexpr int R_ = decltype(ROWS)::value;
            if (p.cols <= kXBufs * kLnCols) hipLaunchKernelGGL((layernorm_quantize_kernel<mode, sb, R_, true>), dim3(blocks), dim3(kLnWaves * 64), 0, stream, p);
            else hipLaunchKernelGGL((layernorm_quantize_kernel<mode, sb, R_, false>), dim3(blocks), dim3(kLnWaves * 64), 0, stream, p);
        };
        if (R == 16) launch_rows(std::integral_constant<int, 16>{});
        else if (R == 32) launch_rows(std::integral_constant<int, 32>{});
        else launch_rows(std::integral_constant<int, 64>{});
    };
    auto launch_mode = [&](auto SB) {
        if (!vec) launch(std::integral_constant<int, kLnScalar>{}, SB);
        else if (p.res || p.sum_out) launch(std::integral_constant<int, kLnRes>{}, SB);
        else launch(std::integral_constant<int, kLnVec>{}, SB);
    };
    if (p.sb == 4) launch_mode(std::integral_constant<int, 4>{});
    else if (p.sb == 8) launch_mode(std::integral_constant<int, 8>{});
    else if (p.sb == 2) launch_mode(std::integral_constant<int, 2>{});
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace vitq
