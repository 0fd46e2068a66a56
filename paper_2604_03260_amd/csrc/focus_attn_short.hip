// Attention forward for short 16-bit problems in position order (one class: masked and dense layouts): the structure of the
// fp32 kernel (focus_attn_f32.hip) with 16-bit products.
//
// A work-group owns 32 query rows; its eight wavefronts (four at 256 components) walk the 32-key units of the causal prefix
// round-robin with a running softmax each, operands straight from the caches, and merge once.  The tiled kernel
// (focus_attn_mfma.hip) needs V staged by a launch before it and a second launch for rows that need a softmax reference, and
// walks up to n/64 tiles one after the other in work-groups that are too few to fill the chip: at 512 tokens all of it is latency.
// Here a chain is n/256 units and there is one launch.
//
// What bounds it is the issue of vector instructions (one per about 6 cycles and wavefront, and there are two wavefronts on a
// SIMD) and the round trips to memory: 1.7 us each where the caches are cold.  So a unit's membership words, keys and values are
// asked for together, up to 64 components with the next unit's; row addresses are scalars; the pairs near the diagonal
// come from five position words instead of a dozen instructions per pair; values that are not finite are looked for in the
// loaded words; the partial results meet once, all together; and the arguments fit a few cache lines.  12 heads of 64 x
// 512 tokens, with the bucketing: 19.4 -> 16.2 us; 32/8 heads of 128 x 305 tokens, K = 16 top-3 44.2 -> 32.9.
#include "focus_short.h"

namespace focus {

namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 f16x2;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
template <bool F16> struct Half16;
template <> struct Half16<false> {
    typedef __bf16 T;
    typedef bf16x8 V8;
    typedef bf16x2 V2;
    static __device__ inline float dot2(V2 a, V2 b, float c) { return __builtin_amdgcn_fdot2_f32_bf16(a, b, c, false); }
    static constexpr uint32_t EXP = 0x7f80u, ONE = 0x3f80u;
    static __device__ inline f32x16 mfma(V8 a, V8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Half16<true> {
    typedef _Float16 T;
    typedef f16x8 V8;
    typedef f16x2 V2;
    static __device__ inline float dot2(V2 a, V2 b, float c) { return __builtin_amdgcn_fdot2(a, b, c, false); }
    static constexpr uint32_t EXP = 0x7c00u, ONE = 0x3c00u;
    static __device__ inline f32x16 mfma(V8 a, V8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};
template <typename T> __device__ inline uint32_t bits16(T x)
{
    uint16_t b;
    __builtin_memcpy(&b, &x, 2);
    return b;
}
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// Ones where the two 16-bit values of x are +inf or NaN, zeros elsewhere.
template <bool F16>
__device__ inline uint32_t inf_or_nan_marks(uint32_t x)
{
    typedef typename Half16<F16>::T elem_t;
    uint32_t m = 0u;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint16_t b = (uint16_t)(x >> (16 * e));
        elem_t h;
        __builtin_memcpy(&h, &b, 2);
        m |= !(h < (elem_t)INFINITY) ? Half16<F16>::ONE << (16 * e) : 0u;
    }
    return m;
}

// max of the two half-waves (lane l and lane l^32 hold the same query row)
__device__ inline float both_halves_max(float x)
{
    const unsigned xi = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Wavefronts of a work-group: 256 components take the registers of a SIMD for one each.
constexpr int short_waves(int d) { return d == 256 ? 4 : 8; }


// SOFT: Sec. 2 Eq. 2, every causal pair, the score of a pair outside the window times 1 / (1 + 2^G), G = -lambda * log2(e) * g_i . g_j from
// the bf16 high and low parts of the assignments as in the tiled kernel (focus_attn_mfma.hip), taken apart here; SOFT k-steps of
// 16 groups.
template <int D, bool F16, int SOFT>
__global__ __launch_bounds__(64 * short_waves(D), short_waves(D) / 4) void attn_short_kernel(ShortArgs A, HeadMap hm)
{
    typedef Half16<F16> HT;
    typedef typename HT::T elem_t;
    typedef typename HT::V2 V2;
    typedef typename HT::V8 V8;
    constexpr int NW = short_waves(D);
    constexpr int CPL = short_cpl(D);
    constexpr int RPW = 16 / NW;                  // rows of every block that a wavefront adds up and stores
    constexpr int KS = D / 16;                    // products of one S^T unit
    constexpr int DB = (D + 31) / 32;             // 32-component blocks of O^T
    constexpr int VW = (DB + 1) / 2;              // registers of a key's values in a lane
    __shared__ typename ShortMerge<NW, DB>::Space s_merge;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n32 = lane & 31, hh = lane >> 5;
    const ShortWalk W(A, hm, lane);
    const int n = W.n;
    const bool rvalid = W.rvalid;
    V8 qf[KS];
    {
        const uint16_t* qrow = (const uint16_t*)A.q + (size_t)W.b * A.qs[0] + (size_t)W.h * A.qs[1] + (size_t)max(W.qpos, 0) * A.qs[2] + hh * 8;
#pragma unroll
        for (int c = 0; c < KS; ++c) qf[c] = *(const V8*)(qrow + 16 * c);
    }
    const size_t koff = (size_t)W.b * A.ks[0] + (size_t)W.hk * A.ks[1];
    const char* kbase = (const char*)((const uint16_t*)A.k + koff);
    const char* vbase = (const char*)((const uint16_t*)A.v + koff);
    const unsigned pitch = A.pitch_bytes;
    const float scale = A.scale, cap = A.softcap;
    const float sl2 = cap > 0.f ? LOG2E : scale * LOG2E;     // logits (scores without a cap) to log2 units
    bf16x8 gqh[SOFT + 1], gql[SOFT + 1];          // the row's assignment times the slope
    const float* gbase = SOFT ? A.g + (size_t)W.b * n * A.K : nullptr;
    // components 16 * ks + 8 * hh .. + 7 of the assignment of position pos
    auto load_g = [&](int pos, int ks, float (&x)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = 16 * ks + 8 * hh + e;
            x[e] = c < A.K ? gbase[(size_t)pos * A.K + c] : 0.f;
        }
    };
    auto split_g = [&](const float (&x)[8], float slope, bf16x8& hi, bf16x8& lo) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = x[e] * slope;
            hi[e] = (__bf16)y;
            lo[e] = (__bf16)(y - (float)hi[e]);
        }
    };
    if constexpr (SOFT > 0) {
#pragma unroll
        for (int ks = 0; ks < SOFT; ++ks) {
            float x[8];
            load_g(max(W.qpos, 0), ks, x);
            split_g(x, A.gate_slope, gqh[ks], gql[ks]);
        }
    }
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    int npairs = 0;

    // Values of a half-wave's 16 keys of a unit: with the components of a lane side by side a key's values of 64 components are
    // one 4-byte load, those of 128 one of 8, in the place of two and four of 2 bytes.  A row's address is a scalar and one
    // offset that all rows share; rows past the last position are read as the last one again.
    struct Values { uint32_t w[16][VW]; };        // as they are loaded, a key after the other
    auto load_row = [&](const char* p, unsigned at, uint32_t (&x)[VW]) {
        if constexpr (D == 256) {
            const uint4 y = *(const uint4*)(p + at);
            x[0] = y.x; x[1] = y.y; x[2] = y.z; x[3] = y.w;
        } else if constexpr (D == 128) {
            const uint2 y = *(const uint2*)(p + at);
            x[0] = y.x; x[1] = y.y;
        } else {
            x[0] = *(const uint32_t*)(p + at);
            if constexpr (D > 64) x[1] = 64 + n32 < D ? *(const uint16_t*)(p + (at + 128u - 2u * (unsigned)n32)) : 0u;
        }
    };
    const unsigned at_v = (unsigned)n32 * (2u * CPL), four = hh ? 4u * pitch : 0u;
    auto load_v = [&](int u, Values& x) {
        if (32 * u + 32 <= n) {
#pragma unroll
            for (int r = 0; r < 16; ++r) load_row(vbase + (size_t)(unsigned)(32 * u + 8 * (r / 4) + r % 4) * pitch, four + at_v, x.w[r]);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) load_row(vbase, (unsigned)min(32 * u + 8 * (r / 4) + 4 * hh + r % 4, n - 1) * pitch + at_v, x.w[r]);
        }
    };
    auto pair_v = [&](const Values& x, uint32_t (&vv)[8][DB]) {          // two keys to a register
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint32_t a = x.w[2 * r2][db / 2], c = x.w[2 * r2 + 1][db / 2];
                vv[r2][db] = db % 2 ? __builtin_amdgcn_perm(c, a, 0x07060302u) : __builtin_amdgcn_perm(c, a, 0x05040100u);
            }
    };
    auto any_nonfinite = [&](const Values& x) -> bool {  // an exponent of all ones carries into the sign
        uint32_t bad = 0u;
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int i = 0; i < VW; ++i) bad |= (x.w[r][i] & (HT::EXP * 0x10001u)) + (0x8000u - HT::EXP) * 0x10001u;
        return __any((bad & 0x80008000u) != 0u);
    };

    bool again = false;                           // (uniform) values were taken out of a product
    // The membership words, the keys and the values of a unit in one round trip: a unit whose pairs are all masked is rare, and
    // a walk is a chain of few units.  Up to 64 components there are registers for the next unit's too; asked for as this one's
    // are used up, without a second set of registers, those of 128 components made a pass 2 % longer (32 heads x 305 tokens).
    struct Unit {
        uint4 km[4];
        V8 kf[KS];
        Values v;
        float g[SOFT + 1][8];
    };
    auto load_unit = [&](int u, Unit& U) {
        W.load_masks(u, U.km);
        if constexpr (SOFT > 0) {
#pragma unroll
            for (int ks = 0; ks < SOFT; ++ks) load_g(min(32 * u + n32, n - 1), ks, U.g[ks]);
        }
        const char* kr = kbase + (size_t)(unsigned)(32 * u) * pitch;
        const unsigned at_k = (unsigned)min(n32, n - 1 - 32 * u) * pitch + 16u * (unsigned)hh;
#pragma unroll
        for (int c = 0; c < KS; ++c) U.kf[c] = *(const V8*)(kr + (at_k + 32u * c));
        load_v(u, U.v);
    };
    constexpr bool AHEAD = D == 64 && SOFT < 2;
    Unit next;
    if (AHEAD && W.u0 + wave < W.u1) load_unit(W.u0 + wave, next);
    for (int u = W.u0 + wave; u < W.u1; u += NW) {
        Unit U;
        if constexpr (AHEAD) {
            U = next;
            if (u + NW < W.u1) load_unit(u + NW, next);
        } else {
            load_unit(u, U);
        }
        const unsigned ok = W.pairs(u, U.km);
        if (!__any(ok != 0u)) continue;                                  // nothing here for any of the 32 rows
        const bool all_ok = !__any(rvalid && ok != 0xffffu);
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int c = 0; c < KS; ++c) s = HT::mfma(U.kf[c], qf[c], s);
        if constexpr (SOFT > 0) {
            const int at = W.qpos - 32 * u;       // of the row, from the unit's first key on
            if (__any(at >= W.w)) {               // some pair outside the window
                f32x16 gate;
#pragma unroll
                for (int r = 0; r < 16; ++r) gate[r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < SOFT; ++ks) {
                    bf16x8 hi, lo;
                    split_g(U.g[ks], 1.f, hi, lo);
                    gate = Half16<false>::mfma(hi, gqh[ks], gate);
                    gate = Half16<false>::mfma(hi, gql[ks], gate);
                    gate = Half16<false>::mfma(lo, gqh[ks], gate);
                }
                const unsigned far = W.upto(at - W.w);                   // pairs outside the window
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float x = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(gate[r]));
                    s[r] *= (far >> r) & 1u ? x : 1.f;
                }
            }
        }
        // softmax step in log2 units: p = 2^(s * sl2 - m), one rounding in the exponent (a row's m cancels)
        // cap * tanh(s * scale / cap), the quotient rounded once, in place of a division per score.  (As 1 - 2 / (1 + e^(2z)) the
        // difference cancels where z is small: logits of unit variance at cap 50 off by up to 9e-6, here by 6e-7.)
        if (cap > 0.f) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = cap * tanhf(fmaf(s[r], A.cap_ratio, s[r] * A.cap_rest));
        }
        if (!all_ok) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = (ok >> r) & 1u ? s[r] : -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        const float m_new = fmaxf(m, both_halves_max(mx) * sl2);
        if (__any(m_new > m)) {
            const float alpha = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        }
        const float m_use = (m == -INFINITY) ? 0.f : m;
        // probabilities rounded to the storage type; the row sum adds the rounded ones, the numbers the product uses
        uint32_t pw[8];
        V2 ones;
        ones[0] = ones[1] = (elem_t)1.f;
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2) {
            V2 p2;
            p2[0] = (elem_t)__builtin_amdgcn_exp2f(fmaf(s[2 * r2], sl2, -m_use));                 // masked: 2^-inf = 0
            p2[1] = (elem_t)__builtin_amdgcn_exp2f(fmaf(s[2 * r2 + 1], sl2, -m_use));
            l = HT::dot2(p2, ones, l);
            pw[r2] = __builtin_bit_cast(uint32_t, p2);
        }
        uint32_t vv[8][DB];
        pair_v(U.v, vv);
        // A value that is not finite would reach the rows that do not attend it through 0 * inf: where the unit is not
        // attended as a whole it is taken out here and added below to the rows that do attend its key.
        if (!all_ok && any_nonfinite(U.v)) {
            again = true;
#pragma unroll
            for (int r2 = 0; r2 < 8; ++r2)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const uint32_t x = vv[r2][db];
                    vv[r2][db] = ((x & HT::EXP) == HT::EXP ? 0u : x & 0xffffu) | (((x >> 16) & HT::EXP) == HT::EXP ? 0u : x & 0xffff0000u);
                }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {                                    // 16 keys each
            const u32x4 pt = {pw[4 * t], pw[4 * t + 1], pw[4 * t + 2], pw[4 * t + 3]};
            const V8 pb = __builtin_bit_cast(V8, pt);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const u32x4 vt = {vv[4 * t][db], vv[4 * t + 1][db], vv[4 * t + 2][db], vv[4 * t + 3][db]};
                o[db] = HT::mfma(__builtin_bit_cast(V8, vt), pb, o[db]);
            }
        }
        if (A.row_pairs) npairs += __popc(ok);
    }
    // Infinities and NaN that were taken out, component by component: the matrix cores count, per row and component, the
    // infinities of either sign that the row attends (a NaN counts as both).  A walk of its own, so that the registers
    // it takes are not taken from the one above.
    if (again) {
#pragma unroll 1
        for (int u = W.u0 + wave; u < W.u1; u += NW) {
            uint4 km[4];
            W.load_masks(u, km);
            const unsigned ok = W.pairs(u, km);
            if (!__any(ok != 0u) || !__any(rvalid && ok != 0xffffu)) continue;
            Values x;
            load_v(u, x);
            if (!any_nonfinite(x)) continue;
            uint32_t vv[8][DB];
            pair_v(x, vv);
            uint32_t at[8];                                              // the attended keys, two to a register
#pragma unroll
            for (int r2 = 0; r2 < 8; ++r2)
                at[r2] = ((ok >> (2 * r2)) & 1u ? HT::ONE : 0u) | ((ok >> (2 * r2 + 1)) & 1u ? HT::ONE << 16 : 0u);
#pragma unroll 1
            for (int neg = 0; neg < 2; ++neg) {
                const uint32_t flip = neg ? 0x80008000u : 0u;
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    f32x16 cnt;
#pragma unroll
                    for (int r = 0; r < 16; ++r) cnt[r] = 0.f;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        u32x4 mk, ak;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            mk[e] = inf_or_nan_marks<F16>(vv[4 * t + e][db] ^ flip);
                            ak[e] = at[4 * t + e];
                        }
                        cnt = HT::mfma(__builtin_bit_cast(V8, mk), __builtin_bit_cast(V8, ak), cnt);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[db][r] = cnt[r] > 0.f ? o[db][r] + (neg ? -INFINITY : INFINITY) : o[db][r];
                }
            }
        }
    }
    l += __shfl_xor(l, 32, 64);
    npairs += __shfl_xor(npairs, 32, 64);

    const ShortMerge<NW, DB> M(s_merge, o, m, l, npairs, wave, lane, min(NW, W.u1 - W.u0), A.row_pairs != nullptr);
    if (!rvalid) return;
    l = M.l;
    // an empty row (launch restricted to one pair set): out = 0, lse = -inf
    const float inv = (l > 0.f) ? 1.f / l : (l == 0.f) ? 0.f : l;
    uint16_t* orow = (uint16_t*)A.out + (size_t)W.b * A.os[0] + (size_t)W.h * A.os[1] + (size_t)W.qpos * A.os[2];
    const int i0 = M.first_row(wave, hh);
    auto pair = [&](float lo, float hi) -> uint32_t { return bits16((elem_t)(lo * inv)) | (bits16((elem_t)(hi * inv)) << 16); };
    uint32_t word[RPW * CPL / 2];                 // components CPL * i0 ..: two or more pairs, the blocks of a row in turn
#pragma unroll
    for (int e = 0; e < RPW; ++e)
#pragma unroll
        for (int db = 0; db < CPL; db += 2) word[(e * CPL + db) / 2] = pair(M.acc[db][e], M.acc[db + 1][e]);
    uint2* o0 = (uint2*)(orow + CPL * i0);
#pragma unroll
    for (int i = 0; i < RPW * CPL / 4; ++i) o0[i] = make_uint2(word[2 * i], word[2 * i + 1]);
    if constexpr (D > 64 && D < 128) {
        static_assert(D % 32 == 0 || D % 32 == 16, "pairs of the third block are whole");
        if (64 + i0 < D) *(uint32_t*)(orow + 64 + i0) = pair(M.acc[2][0], M.acc[2][1]);
    }
    if (wave == 0 && hh == 0) {
        const size_t row = (size_t)(W.b * A.Hq + W.h) * n + W.qpos;
        if (A.lse) A.lse[row] = fmaf(M.top, LN2, logf(l));
        if (A.row_pairs) A.row_pairs[row] = M.npairs;
    }
}

}  // namespace

// Where one launch of short chains beats the staged tiles: while its work-groups are at most one to four per compute unit
// (those of a causal launch differ in length, the later ones fill the gaps), fewer the longer the walk, whose units load more
// bytes per key.  The softcap does not decide: the bucketing leaves out what only the tiles need, and may have been given parameters
// without it.  It costs a score more here (tanh) than in the tiles (a polynomial), so the lines lie where the one with a cap
// of 50 is, if that is the lower one.  Bucketing and attention, MHA, K = 4 top-2, window 128, tiled / this kernel, then with the cap (us):
//   causal   64: 512 x 1024 groups 33.1 / 31.8, 35.8 / 36.2;  1024 x 768 37.5 / 34.8, 42.8 / 40.2;  4096 x 768 79.5 / 71.6, 101 / 93
//            80: 512 x 1024 36.9 / 33.4, 39.6 / 37.9;  4096 x 768 87.6 / 86.7, 110 / 109
//            96: 512 x 1024 39.3 / 33.8, 42.0 / 38.5;  4096 x 768 90.9 / 83.5, 111 / 104
//            128: 256 x 1024 37.4 / 32.3, 38.8 / 35.4;  512 x 768 42.4 / 37.2;  1024 x 768 51.3 / 51.2, 56.4 / 52.4;  4096 x 640 104 / 102, 126 / 104
//            256: 256 x 896 56.1 / 51.5, 56.7 / 56.4, 1024 57.3 / 55.2, 58.5 / 60.4;  512 x 560 61.2 / 56.1, 63.1 / 61.0, 640 60.0 / 57.7, 62.0 / 63.6
//                 1024 x 544 75.7 / 70.2, 79.6 / 79.1;  4096 x 512 168 / 147, 183 / 176, 640 168 / 188, 185 / 225
//   otherwise 64: 256 x 768 26.6 / 22.9, 27.8 / 25.5, 1024 28.1 / 28.1, 29.5 / 31.2;  512 x 512 29.5 / 23.7, 32.0 / 27.2, 768 31.1 / 30.7, 33.8 / 35.8
//                 1024 x 512 35.7 / 34.7, 40.8 / 40.0;  2048 x 512 48.9 / 49.4, 59.6 / 61.5;  4096 x 512 75.6 / 79.6, 97.3 / 105
//                 dense (no memberships to test): 4096 x 512 83.3 / 69.1, 102 / 95
//            80: 256 x 896 30.8 / 30.0, 32.2 / 33.1;  512 x 640 34.0 / 33.0, 36.3 / 37.4
//            96: 4096 x 384 90.8 / 96.4, 110 / 120;  256 x 1024 34.6 / 31.1, 36.1 / 34.2;  512 x 768 37.0 / 34.1, 39.7 / 38.3, 47 heads (752) 39.2 / 41.5;  1024 x 512 40.7 / 38.8, 45.6 / 44.3
//            128: 256 x 768 37.1 / 32.7, 38.2 / 35.5;  512 x 512 39.6 / 35.6, 42.2 / 37.0;  4096 x 256 101 / 74
//            256: 256 x 512 52.1 / 38.9, 53.1 / 42.3, 640 52.4 / 51.0, 53.6 / 55.2;  512 x 256 54.6 / 38.0, 56.6 / 41.7, 384 57.1 / 57.0, 59.2 / 63.7
bool short_attention(const Layout& L)
{
    const long long groups = (long long)L.B * L.Hq * ((L.n + 31) / 32);
    const bool fits = L.dtype != 0 && L.NC == 1 && (L.masked || L.dense) && !L.soft && !L.local_only && !L.merge_prev && L.BQ == 128 &&
                      (uint64_t)L.ks[2] * 2 < (1u << 24) && (uint64_t)L.n * (uint64_t)L.ks[2] * 2 < 0xffffffffull;
    int most;
    if (L.causal)
        most = L.d == 256 ? (L.n <= 256 ? 896 : 560) : L.n <= (L.d == 128 ? 256 : 512) ? 1024 : (L.d == 128 && L.n > 1024) ? 640 : 768;
    else if (L.n <= 256)
        most = L.d == 96 ? 1024 : L.d == 256 ? 512 : 768;
    else if (L.n <= 512)
        most = L.d == 256 ? 256 : 512;
    else
        most = (L.d >= 128 || (L.masked && L.n > 1024)) ? 256 : 512;
    return fits && groups <= most && L.n <= 4096;
}

hipError_t launch_attn_short(const Layout& L, const HeadMap& hm, const void* q, const void* k, const void* v, char* ws,
                             void* out, float* lse, int32_t* row_pairs, hipStream_t st)
{
    const ShortArgs A = short_args(L, hm, q, k, v, ws, out, lse, row_pairs);
    const dim3 threads(64 * short_waves(L.d));
    const dim3 blocks = short_grid(A);
#define FOCUS_SHORT(D_)                                                                                                   \
    case D_:                                                                                                              \
        if (L.dtype == 2) hipLaunchKernelGGL((attn_short_kernel<D_, true, 0>), blocks, threads, 0, st, A, hm);             \
        else hipLaunchKernelGGL((attn_short_kernel<D_, false, 0>), blocks, threads, 0, st, A, hm);                         \
        break;
    switch (L.d) {
        FOCUS_SHORT(64) FOCUS_SHORT(80) FOCUS_SHORT(96) FOCUS_SHORT(128) FOCUS_SHORT(256)
        default: return hipErrorInvalidValue;
    }
#undef FOCUS_SHORT
    return hipGetLastError();
}

// The soft gate in the place of four launches (positions, assignments, V, tiles).  What a unit costs grows with the groups, which every
// wavefront takes apart for itself.  Pass, tiled / this kernel (us), 40 .. 4096 tokens, by work-groups of 32 rows, one KV head:
//   K = 4   64: 512 x 752 27.7 / 21.1, 300 x 1000 22.3 / 23.1, 512 x 992 1.03 times, 1000 x 992 1.13, 4096 x 896 1.52;  80, 96: 40 x 1000 0.93 times, 512 x 992 1.07
//           128: 300 x 760 1.05 times, 512 x 752 1.09, 4096 x 640 1.53
//   K = 8   64: 40 x 760 1.04 times, 512 x 752 1.12;  80: 1.15, 1.26;  96: 1.10, 1.24;   128: 300 x 760 25.4 / 27.1, 512 x 752 31.3 / 32.5, 1000 x 736 1.03 times
//   K = 16  64: 300 x 760 22.5 / 24.5, 512 x 752 27.4 / 29.3, 1000 x 736 1.01 times;  80: 300 x 760 1.03;  96: 40 x 760 0.98, 512 x 752 1.02
//           128: 300 x 500 1.15 times, 760 25.5 / 30.8, 2048 x 704 74.2 / 77.0
//   K = 32  64: 300 x 500 1.10 times;  80: 1.17;  96: 1.12;   128: 300 x 250 1.46 times, 500 28.5 / 29.8, 512 x 496 1.05, 1000 x 480 1.13
bool short_soft_attention(const Layout& L)
{
    const long long groups = (long long)L.B * L.Hq * ((L.n + 31) / 32);
    int most;
    if (L.K > 16) most = L.d == 128 && L.n <= 512 ? 384 : 512;
    else if (L.K <= 4) most = L.d < 128 && L.n >= 512 ? 1024 : 768;
    else if (L.K <= 8) most = L.d == 128 && L.n < 1000 ? 512 : 768;
    else most = L.d == 128 || (L.d == 64 && L.n < 1000) ? 512 : 768;
    return L.dtype != 0 && L.soft && L.d <= 128 && L.n <= 4096 && groups <= most &&
           (uint64_t)L.ks[2] * 2 < (1u << 24) && (uint64_t)L.n * (uint64_t)L.ks[2] * 2 < 0xffffffffull;
}

hipError_t launch_attn_short_soft(const Layout& L, const HeadMap& hm, const float* g, const void* q, const void* k, const void* v, char* ws,
                                  void* out, float* lse, hipStream_t st)
{
    ShortArgs A = short_args(L, hm, q, k, v, ws, out, lse, nullptr);
    A.g = g;
    A.dense = 1;
    const dim3 threads(64 * short_waves(L.d)), blocks = short_grid(A);
#define FOCUS_SHORT_SOFT(D_)                                                                                              \
    case D_:                                                                                                              \
        if (L.dtype == 2) {                                                                                               \
            if (L.K <= 16) hipLaunchKernelGGL((attn_short_kernel<D_, true, 1>), blocks, threads, 0, st, A, hm);           \
            else hipLaunchKernelGGL((attn_short_kernel<D_, true, 2>), blocks, threads, 0, st, A, hm);                     \
        } else {                                                                                                          \
            if (L.K <= 16) hipLaunchKernelGGL((attn_short_kernel<D_, false, 1>), blocks, threads, 0, st, A, hm);          \
            else hipLaunchKernelGGL((attn_short_kernel<D_, false, 2>), blocks, threads, 0, st, A, hm);                    \
        }                                                                                                                 \
        break;
    switch (L.d) {
        FOCUS_SHORT_SOFT(64) FOCUS_SHORT_SOFT(80) FOCUS_SHORT_SOFT(96) FOCUS_SHORT_SOFT(128)
        default: return hipErrorInvalidValue;
    }
#undef FOCUS_SHORT_SOFT
    return hipGetLastError();
}

}  // namespace focus
