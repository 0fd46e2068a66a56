// Attention forward for short 16-bit problems in position order (one class: masked and dense layouts), up to 128
// components: the structure of the fp32 kernel (focus_attn_f32.hip) with 16-bit products.
//
// A work-group owns 32 query rows; its eight wavefronts walk the 32-key units of the causal prefix round-robin with a
// running softmax each, operands straight from the caches, and merge once.  The tiled kernel (focus_attn_mfma.hip) needs
// V staged by a launch before it and a second launch for rows that need a softmax reference, and walks up to n/64 tiles
// one after the other in work-groups that are too few to fill the chip: at 512 tokens all of it is latency.
// Here a chain is n/256 units and there is one launch.  V is read row-major with 2-byte loads, which is why the tiled
// kernel wins as soon as throughput counts (see short_attention below).  With 128 components 15 to 17 of the registers of a
// unit's operands spill (64 to 72 bytes of scratch a lane).
#include "focus_internal.h"
#include "focus_tileplan.h"

namespace focus {

namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
template <bool F16> struct Half16;
template <> struct Half16<false> {
    typedef __bf16 T;
    typedef bf16x8 V8;
    static constexpr uint32_t EXP = 0x7f80u, ONE = 0x3f80u;
    static __device__ inline f32x16 mfma(V8 a, V8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Half16<true> {
    typedef _Float16 T;
    typedef f16x8 V8;
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

template <int D, bool F16>
__global__ __launch_bounds__(512, 2) void attn_short_kernel(Layout L, HeadMap hm, int default_map, const uint16_t* __restrict__ q,
                                                            const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                            const char* __restrict__ ws, uint16_t* __restrict__ out,
                                                            float* __restrict__ lse, int32_t* __restrict__ row_pairs)
{
    typedef Half16<F16> HT;
    typedef typename HT::T elem_t;
    typedef typename HT::V8 V8;
    constexpr int NW = 8;
    constexpr int KS = D / 16;                    // products of one S^T unit
    constexpr int DB = (D + 31) / 32;             // 32-component blocks of O^T
    __shared__ TilePlanT<1> P;
    __shared__ float s_o[NW / 2][DB * 16][64];         // partial results on their way between the wavefronts
    __shared__ float s_m[NW / 2][64], s_l[NW / 2][64];
    __shared__ int s_np[NW / 2][64];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n32 = lane & 31, hh = lane >> 5;
    const int BH = L.B * L.Hq;
    const int quarter = 3 - (int)(blockIdx.x / BH) % 4, job = (int)(blockIdx.x / BH) / 4;
    const int x = blockIdx.x % BH;
    int b, h;
    if (default_map) {                            // the query heads of a KV head share blockIdx % 8: one XCD, one L2
        const int BHk = L.B * L.Hkv, G = L.Hq / L.Hkv;
        b = (x % BHk) / L.Hkv;
        h = (x % BHk % L.Hkv) * G + x / BHk;
    } else {
        b = x / L.Hq;
        h = x % L.Hq;
    }
    const int bhq = b * L.Hq + h;
    const int bhk = b * L.Hkv + hm.kv[h];
    if (!plan_linear_tile(L, job, P)) return;
    if (quarter * 32 >= P.nvalid) return;

    const int rloc = quarter * 32 + n32;
    const bool rvalid = rloc < P.nvalid;
    const int qpos = rvalid ? P.row0 + rloc : -1;
    const uint32_t mq_row = rvalid ? ((const uint32_t*)(ws + L.off_mq))[(size_t)bhq * L.n + qpos] : 0u;
    const uint32_t* kmsk = (const uint32_t*)(ws + L.off_kmsk) + (size_t)bhk * L.NKP;     // masked only
    const size_t koff = (size_t)b * L.ks[0] + (size_t)hm.kv[h] * L.ks[1];
    // rows by a 24-bit multiply and a 32-bit offset (the launch checks that they fit)
    const char* kbase = (const char*)(k + koff + hh * 8);
    const char* vbase = (const char*)(v + koff + n32);
    const unsigned pitch_bytes = (unsigned)L.ks[2] * 2u;
    const int w = L.window;
    const float scale = L.scale, cap = L.softcap;
    const float sl2 = cap > 0.f ? LOG2E : scale * LOG2E;     // logits (scores without a cap) to log2 units

    V8 qf[KS];
    {
        const uint16_t* qrow = q + (size_t)b * L.qs[0] + (size_t)h * L.qs[1] + (size_t)max(qpos, 0) * L.qs[2] + hh * 8;
#pragma unroll
        for (int c = 0; c < KS; ++c) qf[c] = *(const V8*)(qrow + 16 * c);
    }
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    int npairs = 0;

    // which pairs of unit u count, bit r = score r: key slot0 + 8*(r/4) + 4*hh + r%4.  Without branches per pair: a key is
    // causal from distance first on, inside the window where (distance + woff) < wlim, and the set of pairs decides
    // whether shared pairs count (by_share) and window pairs that share count as such (loc_any); dense: every pair shares.
    const int set = L.masked ? L.pair_set : 0;
    const bool dense = !L.masked, by_share = set != 2, by_window = set != 1, loc_any = set == 0;
    const int first = L.causal ? 0 : -0x7fffffff, woff = L.causal ? 0 : w - 1;
    const unsigned wlim = L.causal ? (unsigned)w : 2u * (unsigned)w - 1u;
    auto pairs_of = [&](int u, int& slot0) -> unsigned {
        const int tile = P.t0[0] + (u >> 1);
        slot0 = tile * KT + (u & 1) * 32;
        unsigned ok = 0xffffu;
        if (!(tile >= P.ibeg[0] && tile < P.iend[0])) {
            ok = 0u;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                uint4 km4 = make_uint4(0u, 0u, 0u, 0u);
                if (!dense) km4 = *(const uint4*)(kmsk + slot0 + 8 * r4 + 4 * hh);
                const uint32_t km[4] = {km4.x, km4.y, km4.z, km4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int kj = slot0 + 8 * r4 + 4 * hh + e, dlt = qpos - kj;
                    const bool share = dense | ((mq_row & km[e]) != 0u);
                    const bool loc = (unsigned)(dlt + woff) < wlim;
                    const bool in = (by_share & share & (dlt >= first)) | (by_window & loc & (loc_any | !share));
                    ok |= ((kj < L.n) & in) ? 1u << (4 * r4 + e) : 0u;
                }
            }
        }
        return rvalid ? ok : 0u;
    };
    // values of a half-wave's 16 keys of a unit, component 32*db + l%32, two keys to a register
    auto load_v = [&](int slot0, uint32_t (&vv)[8][DB]) {
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2) {
            const int k0 = slot0 + 8 * (r2 / 2) + 4 * hh + 2 * (r2 % 2);
            const char* p0 = vbase + __umul24((unsigned)min(k0, L.n - 1), pitch_bytes);
            const char* p1 = vbase + __umul24((unsigned)min(k0 + 1, L.n - 1), pitch_bytes);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const bool there = D % 32 == 0 || db * 32 + n32 < D;
                const uint32_t lo = there ? *(const uint16_t*)(p0 + 64 * db) : 0u, hi = there ? *(const uint16_t*)(p1 + 64 * db) : 0u;
                vv[r2][db] = lo | (hi << 16);
            }
        }
    };
    auto any_nonfinite = [&](const uint32_t (&vv)[8][DB]) -> bool {
        bool bad = false;
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                bad = bad | ((vv[r2][db] & HT::EXP) == HT::EXP) | (((vv[r2][db] >> 16) & HT::EXP) == HT::EXP);
        return __any(bad);
    };

    bool again = false;                           // (uniform) values were taken out of a product
    for (int u = wave; u < 2 * P.total; u += NW) {
        int slot0;
        const unsigned ok = pairs_of(u, slot0);
        if (!__any(ok != 0u)) continue;                                  // nothing here for any of the 32 rows
        const bool all_ok = !__any(rvalid && ok != 0xffffu);

        // keys, and the values with them: those arrive while the scores are computed
        V8 kf[KS];
        {
            const char* kr = kbase + __umul24((unsigned)min(slot0 + n32, L.n - 1), pitch_bytes);
#pragma unroll
            for (int c = 0; c < KS; ++c) kf[c] = *(const V8*)(kr + 32 * c);
        }
        uint32_t vv[8][DB];
        load_v(slot0, vv);
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int c = 0; c < KS; ++c) s = HT::mfma(kf[c], qf[c], s);
        // softmax step in log2 units: p = 2^(s * sl2 - m), one rounding in the exponent (a row's m cancels)
        if (cap > 0.f) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = cap * tanhf(s[r] * scale / cap);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = (ok >> r) & 1u ? s[r] : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
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
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2) {
            const elem_t p0 = (elem_t)__builtin_amdgcn_exp2f(fmaf(s[2 * r2], sl2, -m_use));       // masked: 2^-inf = 0
            const elem_t p1 = (elem_t)__builtin_amdgcn_exp2f(fmaf(s[2 * r2 + 1], sl2, -m_use));
            l += (float)p0 + (float)p1;
            pw[r2] = bits16(p0) | (bits16(p1) << 16);
        }
        // A value that is not finite would reach the rows that do not attend it through 0 * inf: where the unit is not
        // attended as a whole it is taken out here and added below to the rows that do attend its key.
        if (!all_ok && any_nonfinite(vv)) {
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
        npairs += __popc(ok);
    }
    // Infinities and NaN that were taken out, component by component: the matrix cores count, per row and component, the
    // infinities of either sign that the row attends (a NaN counts as both).  A walk of its own, so that the registers
    // it takes are not taken from the one above.
    if (again) {
#pragma unroll 1
        for (int u = wave; u < 2 * P.total; u += NW) {
            int slot0;
            const unsigned ok = pairs_of(u, slot0);
            if (!__any(ok != 0u) || !__any(rvalid && ok != 0xffffu)) continue;
            uint32_t vv[8][DB];
            load_v(slot0, vv);
            if (!any_nonfinite(vv)) continue;
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

    // App. D's merge of the wavefronts' partial softmaxes: the upper half into the lower half until one is left
    auto put = [&](int buf) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) s_o[buf][db * 16 + r][lane] = o[db][r];
        s_m[buf][lane] = m; s_l[buf][lane] = l; s_np[buf][lane] = npairs;
    };
    auto take = [&](int buf) {
        const float m2 = s_m[buf][lane], l2 = s_l[buf][lane];
        const float m_new = fmaxf(m, m2);
        const float a1 = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - m_new), a2 = (m2 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m2 - m_new);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] = o[db][r] * a1 + s_o[buf][db * 16 + r][lane] * a2;
        l = l * a1 + l2 * a2;
        m = m_new;
        npairs += s_np[buf][lane];
    };
#pragma unroll
    for (int half = NW / 2; half >= 1; half >>= 1) {
        if (wave >= half && wave < 2 * half) put(wave - half);
        __syncthreads();
        if (wave < half) take(wave);
        __syncthreads();
    }
    if (wave != 0) return;
    if (!rvalid) return;
    // an empty row (launch restricted to one pair set): out = 0, lse = -inf
    const float inv = (l > 0.f) ? 1.f / l : (l == 0.f) ? 0.f : l;
    uint16_t* orow = out + (size_t)b * L.os[0] + (size_t)h * L.os[1] + (size_t)qpos * L.os[2];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int c = db * 32 + 8 * r4 + 4 * hh;
            if (D % 32 != 0 && c >= D) continue;
            uint2 val;
            val.x = bits16((elem_t)(o[db][4 * r4] * inv)) | (bits16((elem_t)(o[db][4 * r4 + 1] * inv)) << 16);
            val.y = bits16((elem_t)(o[db][4 * r4 + 2] * inv)) | (bits16((elem_t)(o[db][4 * r4 + 3] * inv)) << 16);
            *(uint2*)(orow + c) = val;
        }
    if (hh == 0) {
        if (lse) lse[(size_t)bhq * L.n + qpos] = fmaf(m, LN2, logf(l));
        if (row_pairs) row_pairs[(size_t)bhq * L.n + qpos] = npairs;
    }
}

}  // namespace

// Where one launch of short chains beats the staged tiles: while every work-group of 32 rows has a compute unit of its own.
// Causal launches may have some more (their work-groups differ in length and the first ones end early; 64 components leave
// room for two on a unit), non-causal ones no more: their 257th waits for a whole walk.  Past 64 components the walk itself
// is slower per key on the masked layout, so that it may not be long; 96 of them fill the 32-component blocks that 80 leave empty.
// Attention alone, tiled / this kernel (us), masked layout, K = 4 top-2, measured over 128 .. 8192 tokens and 48 .. 1024 groups:
//   64:  512 tokens, 192 groups 20.3 / 12.6;  1024, 384 27.8 / 22.3;  4096, 256 70.2 / 57.8;  non-causal 1024, 256 26.9 / 20.0, 288 27.5 / 35.3
//   80:  2048, 256 47.5 / 45.9;  4096, 256 80.8 / 82.7;      96: 1024, 320 33.1 / 23.0
//   128: 256, 256 21.0 / 15.8;  1024, 256 34.3 / 33.4;  2048, 256 53.9 / 56.6, dense 47.7 / 41.9;  non-causal 512, 256 25.4 / 22.7, 288 26.4 / 39.5
bool short_attention(const Layout& L)
{
    const long long groups = (long long)L.B * L.Hq * ((L.n + 31) / 32);
    const bool fits = L.dtype != 0 && L.NC == 1 && (L.masked || L.dense) && !L.soft && !L.local_only && !L.merge_prev && L.BQ == 128 &&
                      L.d <= 128 && (uint64_t)L.ks[2] * 2 < (1u << 24) && (uint64_t)L.n * (uint64_t)L.ks[2] * 2 < 0xffffffffull;
    const int most = L.causal ? (L.d <= 64 ? 384 : (L.d == 128 && L.n <= 256) ? 256 : 320) : (L.d <= 64 && L.n <= 256) ? 384 : 256;
    const int longest = (L.dense || L.d == 64 || L.d == 96) ? 4096 : L.d == 80 ? 2048 : 1024;
    return fits && groups <= most && L.n <= longest;
}

hipError_t launch_attn_short(const Layout& L, const HeadMap& hm, const void* q, const void* k, const void* v, char* ws,
                             void* out, float* lse, int32_t* row_pairs, hipStream_t st)
{
    int default_map = (L.Hq % L.Hkv == 0) ? 1 : 0;
    for (int h = 0; default_map && h < L.Hq; ++h) default_map = hm.kv[h] == h / (L.Hq / L.Hkv);
    const unsigned blocks = (unsigned)((size_t)L.NT * 4 * L.B * L.Hq);        // four quarters of every 128-row tile
#define FOCUS_SHORT(D_)                                                                                                   \
    case D_:                                                                                                              \
        if (L.dtype == 2)                                                                                                 \
            hipLaunchKernelGGL((attn_short_kernel<D_, true>), dim3(blocks), dim3(512), 0, st, L, hm, default_map,         \
                               (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const char*)ws, (uint16_t*)out, lse, row_pairs); \
        else                                                                                                              \
            hipLaunchKernelGGL((attn_short_kernel<D_, false>), dim3(blocks), dim3(512), 0, st, L, hm, default_map,        \
                               (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const char*)ws, (uint16_t*)out, lse, row_pairs); \
        break;
    switch (L.d) {
        FOCUS_SHORT(64) FOCUS_SHORT(80) FOCUS_SHORT(96) FOCUS_SHORT(128)
        default: return hipErrorInvalidValue;
    }
#undef FOCUS_SHORT
    return hipGetLastError();
}

}  // namespace focus
