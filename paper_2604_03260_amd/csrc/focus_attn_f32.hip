// Attention forward for fp32 inputs on the fp32 matrix cores (v_mfma_f32_32x32x2_f32): App. D Eq. 3 with top-k sets,
// exact softmax (Sec. 1), products and sums in fp32 like the vector kernel it stands in for.
//
// One product of 32 x 32 x 2 takes 64 cycles of a SIMD and one register per operand, so this kernel is bound by the
// matrix cores as long as their operands arrive: every lane loads its own fragments straight from the caches, no LDS,
// no barriers.  A work-group owns 32 query rows (a quarter of a plan tile); its wavefronts walk the 32-key units
// of the tile's key sequence round-robin, each with its own running softmax, and meet once at the end.  Splitting the
// keys instead of the rows makes the longest chain an eighth as long: at 12 heads x 1024 tokens the 96 tiles of 128
// rows would leave most of the 256 compute units idle behind a walk of 32 units.
//   S^T = K Q^T      A = key rows (lane: key l%32, components of its half-wave), B = query rows in registers.  The order
//                    of the inner index is free: half-wave h takes components [h*d/2, (h+1)*d/2), contiguous loads.
//   O^T += V^T P^T   the accumulator lane of S^T (row l%32) holds keys 8*(r/4) + 4*h + r%4, which is the B operand of
//                    step r; A = V[that key][component], 32 consecutive components per half-wave.
// Two kernels: attn_f32_linear_kernel for most problems in position order, attn_f32_kernel for class tiles, for rows too far apart and
// where it is the faster one (by_tiles).  The latter, measured when it served both (d = 64, K = 4 top-2, attention launch), against the vector kernel: 12 heads x 1024 tokens
// 671 -> 41 us; 40 heads x 4096 tokens 967 us, 89 of the 152 TFLOP/s a library product of 8192 x 8192 matrices reaches: the rest is
// vector work (masks, 16 exponentials and 24 row addresses per unit) that two wavefronts per SIMD cover in part.
#include "focus_short.h"
#include "focus_tileplan.h"

namespace focus {

namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// max of the two half-waves (lane l and lane l^32 hold the same query row)
__device__ inline float both_halves_max(float x)
{
    const unsigned xi = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// LINEAR: one class in position order.  WIDE: some row of k or v lies 4 GiB or more past its head's first, or rows are 16 MiB or more apart: 64-bit products
// for every row address, a fifth of the vector work of a unit.  Otherwise one 24-bit multiply and a 32-bit offset.
template <int D, int NW, bool WIDE, bool LINEAR>
__global__ __launch_bounds__(64 * NW, D <= 128 ? 2 : 1) void attn_f32_kernel(Layout L, HeadMap hm, int default_map,
                                                                        const float* __restrict__ q, const float* __restrict__ k,
                                                                        const float* __restrict__ v, const char* __restrict__ ws,
                                                                        float* __restrict__ out, float* __restrict__ lse,
                                                                        int32_t* __restrict__ row_pairs)
{
    constexpr int H = D / 2;                      // components per half-wave = products of one S^T unit
    constexpr int DB = (D + 31) / 32;             // 32-component blocks of O^T
    constexpr int VG = D <= 96 ? 16 : 4;          // keys whose V rows are in flight (the registers hold no more of longer rows)
    static_assert(D % 16 == 0 && H % 4 == 0, "whole 16-byte loads per half-wave");
    __shared__ TilePlan P;
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
    if (!plan_query_tile(L, ws, bhq, bhk, job, P)) return;
    if (quarter * 32 >= P.nvalid) return;

    const int rloc = quarter * 32 + n32;
    const bool rvalid = rloc < P.nvalid;
    const int qpos = !rvalid ? -1 : L.NC == 1 ? P.row0 + rloc : ((const int*)(ws + L.off_qperm))[(size_t)bhq * L.NQP + P.row0 + rloc];
    const uint32_t mq_row = rvalid ? ((const uint32_t*)(ws + L.off_mq))[(size_t)bhq * L.n + qpos] : 0u;
    const int* kpos = (const int*)(ws + L.off_kpos) + (size_t)bhk * L.NKP;
    const uint32_t* kmsk = (const uint32_t*)(ws + L.off_kmsk) + (size_t)bhk * L.NKP;     // coarse classes and masked only
    const size_t koff = (size_t)b * L.ks[0] + (size_t)hm.kv[h] * L.ks[1];
    const size_t pitch = (size_t)L.ks[2];
    const float* kbase = k + koff + hh * H;
    const float* vbase = v + koff + n32;
    const int w = L.window;
    const float scale = L.scale, cap = L.softcap;
    const float sl2 = cap > 0.f ? LOG2E : scale * LOG2E;     // logits (scores without a cap) to log2 units
    const unsigned pitch_bytes = (unsigned)pitch * 4u;
    auto row_at = [&](const float* base, int pos) -> const float* {
        if constexpr (WIDE) return base + (size_t)pos * pitch;
        else return (const float*)((const char*)base + __umul24((unsigned)pos, pitch_bytes));
    };

    float4 qf[H / 4];
    {
        const float* qrow = q + (size_t)b * L.qs[0] + (size_t)h * L.qs[1] + (size_t)max(qpos, 0) * L.qs[2] + hh * H;
#pragma unroll
        for (int c = 0; c < H / 4; ++c) qf[c] = *(const float4*)(qrow + 4 * c);
    }
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    int npairs = 0;

    // far_end: keys below it lie outside every row's window and are causal for all of them (one class, position order)
    const int first_pos = P.row0 + quarter * 32;
    const int far_end = (L.masked && L.causal && L.pair_set == 0) ? first_pos - w + 1 : 0;
    // (Fetching the next unit's masks before this one's products and its key rows right after them takes 65 registers
    // more in this kernel, and was slower at every size while it walked rows in position order too: 45 -> 48 us at 12 heads x
    // 1024 tokens, 325 -> 338 at 4096.  attn_f32_linear_kernel has the registers at 64 components, and does it.)
    int cur = 0;
    struct Unit {
        int slot0, krow;
        bool inter, interior;
        uint4 km[4];                              // membership masks of the 16 keys (coarse classes and masked)
        int4 kp[LINEAR ? 1 : 4];                  // their positions; LINEAR: slot = position
    };
    auto fetch = [&](Unit& U, int u) {
        const int it = u >> 1;
        while (it >= P.cum[cur + 1]) ++cur;
        const int tile = __builtin_amdgcn_readfirstlane(P.t0[cur] + (it - P.cum[cur]));
        U.inter = LINEAR || P.inter[cur] != 0;
        U.interior = tile >= P.ibeg[cur] && tile < P.iend[cur];
        U.slot0 = tile * KT + (u & 1) * 32;
        U.krow = LINEAR ? U.slot0 + n32 : kpos[U.slot0 + n32];
        if (L.coarse && U.inter) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) U.km[r4] = *(const uint4*)(kmsk + U.slot0 + 8 * r4 + 4 * hh);
        }
        if constexpr (!LINEAR) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) U.kp[r4] = *(const int4*)(kpos + U.slot0 + 8 * r4 + 4 * hh);
        }
    };
    auto key_pos = [&](const Unit& U, int r) -> int {
        if constexpr (LINEAR) return U.slot0 + 8 * (r / 4) + 4 * hh + r % 4;
        const int4 p4 = U.kp[LINEAR ? 0 : r / 4];
        return r % 4 == 0 ? p4.x : r % 4 == 1 ? p4.y : r % 4 == 2 ? p4.z : p4.w;
    };
    auto pairs_of = [&](const Unit& U) -> unsigned {              // which pairs of the unit count, bit r = score r
        unsigned ok = 0xffffu;
        if (U.slot0 + 32 <= far_end) {
            ok = 0u;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                ok |= ((mq_row & U.km[r4].x) ? 1u << (4 * r4) : 0u) | ((mq_row & U.km[r4].y) ? 2u << (4 * r4) : 0u) |
                      ((mq_row & U.km[r4].z) ? 4u << (4 * r4) : 0u) | ((mq_row & U.km[r4].w) ? 8u << (4 * r4) : 0u);
        } else if (!U.interior) {
            ok = 0u;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kj = key_pos(U, r), dlt = qpos - kj;           // pads sit at INT_MAX or past the last position
                const uint32_t km = r % 4 == 0 ? U.km[r / 4].x : r % 4 == 1 ? U.km[r / 4].y : r % 4 == 2 ? U.km[r / 4].z : U.km[r / 4].w;
                const bool share = (L.coarse && U.inter) ? (mq_row & km) != 0u : U.inter;
                const bool loc = L.causal ? (dlt >= 0 && dlt < w) : (dlt < w && -dlt < w);
                const bool cz = L.causal ? dlt >= 0 : true;
                bool in = cz && (share || loc);
                // coarse classes that share a super-group hold pairs of both sets of a restricted launch
                if (L.coarse && U.inter && L.pair_set != 0) in = (L.pair_set == 1) ? (cz && share) : (loc && !share);
                ok |= (kj < L.n && in) ? 1u << r : 0u;
            }
        }
        return rvalid ? ok : 0u;
    };
    auto load_v = [&](const Unit& U, int r0, float (&vv)[VG][DB]) {
#pragma unroll
        for (int r = 0; r < VG; ++r) {
            const float* vr = row_at(vbase, min(key_pos(U, r0 + r), L.n - 1));
#pragma unroll
            for (int db = 0; db < DB; ++db) vv[r][db] = (D % 32 == 0 || db * 32 + n32 < D) ? vr[db * 32] : 0.f;
        }
    };
    auto any_nonfinite = [&](const float (&vv)[VG][DB]) -> bool {
        bool bad = false;
#pragma unroll
        for (int r = 0; r < VG; ++r)
#pragma unroll
            for (int db = 0; db < DB; ++db) bad = bad | !__builtin_isfinite(vv[r][db]);
        return __any(bad);
    };
    bool again = false;                           // (uniform) values were taken out of a product
    for (int u = wave; u < 2 * P.total; u += NW) {
        Unit U;
        fetch(U, u);
        const unsigned ok = pairs_of(U);
        if (!__any(ok != 0u)) continue;                                  // nothing here for any of the 32 rows
        const bool all_ok = !__any(rvalid && ok != 0xffffu);
        float vv[VG][DB];
        // keys, and the values with them: those arrive while the scores are computed
        float4 kf[H / 4];
        {
            const float* kr = row_at(kbase, min(U.krow, L.n - 1));
#pragma unroll
            for (int c = 0; c < H / 4; ++c) kf[c] = *(const float4*)(kr + 4 * c);
        }
        if constexpr (VG == 16) load_v(U, 0, vv);
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int c = 0; c < H / 4; ++c) {
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c].x, qf[c].x, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c].y, qf[c].y, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c].z, qf[c].z, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c].w, qf[c].w, s, 0, 0, 0);
        }
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
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], sl2, -m_use));      // masked: 2^-inf = 0
            l += s[r];
        }
#pragma unroll
        for (int r0 = 0; r0 < 16; r0 += VG) {
            if constexpr (VG < 16) load_v(U, r0, vv);
            // A value that is not finite would reach the rows that do not attend it through 0 * inf: where the unit is
            // not attended as a whole it is taken out here and added below to the rows that do attend its key.
            if (!all_ok && any_nonfinite(vv)) {
                again = true;
#pragma unroll
                for (int r = 0; r < VG; ++r)
#pragma unroll
                    for (int db = 0; db < DB; ++db) vv[r][db] = __builtin_isfinite(vv[r][db]) ? vv[r][db] : 0.f;
            }
#pragma unroll
            for (int r = 0; r < VG; ++r)
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[r][db], s[r0 + r], o[db], 0, 0, 0);
        }
        npairs += __popc(ok);
    }
    // Infinities and NaN that were taken out, component by component: the matrix cores count, per row and component, the
    // infinities of either sign that the row attends (a NaN counts as both).  A walk of its own, so that the registers
    // it takes are not taken from the one above.
    if (again) {
        cur = 0;
#pragma unroll 1
        for (int u = wave; u < 2 * P.total; u += NW) {
            Unit U;
            fetch(U, u);
            const unsigned ok = pairs_of(U);
            if (!__any(ok != 0u) || !__any(rvalid && ok != 0xffffu)) continue;
#pragma unroll
            for (int r0 = 0; r0 < 16; r0 += VG) {
                float vv[VG][DB];
                load_v(U, r0, vv);
                if (!any_nonfinite(vv)) continue;
#pragma unroll 1
                for (int neg = 0; neg < 2; ++neg) {
                    const unsigned flip = neg ? 0x80000000u : 0u;
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        f32x16 cnt;
#pragma unroll
                        for (int r = 0; r < 16; ++r) cnt[r] = 0.f;
#pragma unroll
                        for (int r = 0; r < VG; ++r)
                            cnt = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(__float_as_uint(vv[r][db]) ^ flip) < INFINITY ? 0.f : 1.f,
                                                                       (ok >> (r0 + r)) & 1u ? 1.f : 0.f, cnt, 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < 16; ++r) o[db][r] = cnt[r] > 0.f ? o[db][r] + (neg ? -INFINITY : INFINITY) : o[db][r];
                    }
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
    float* orow = out + (size_t)b * L.os[0] + (size_t)h * L.os[1] + (size_t)qpos * L.os[2];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int c = db * 32 + 8 * r4 + 4 * hh;
            if (D % 32 != 0 && c >= D) continue;
            *(float4*)(orow + c) = make_float4(o[db][4 * r4] * inv, o[db][4 * r4 + 1] * inv, o[db][4 * r4 + 2] * inv, o[db][4 * r4 + 3] * inv);
        }
    if (hh == 0) {
        if (lse) lse[(size_t)bhq * L.n + qpos] = fmaf(m, LN2, logf(l));
        if (row_pairs) row_pairs[(size_t)bhq * L.n + qpos] = npairs;
    }
}

// Rows in position order (one class), a head's rows within 4 GiB: the same walk with the work around the products cut down, as in
// focus_attn_short.hip: scalar row addresses, pairs near the diagonal from position words, a key's values in one load or two
// (DB 4-byte loads before), keys and membership words of the next unit asked for when the scores have used this one's, its values
// after the last product, one merge.  12 heads of 64 x 1024 tokens, with the bucketing: 44.7 -> 40.7 us; 8 x 15/5 of 80 x 627
// 163 -> 128; 32 of 128 x 2028 462 -> 431; 4 x 40/8 of 64 x 2048 1047 -> 955.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D <= 128 ? 2 : 1) void attn_f32_linear_kernel(ShortArgs A, HeadMap hm)
{
    constexpr int H = D / 2;                      // components per half-wave = products of one S^T unit
    constexpr int DB = (D + 31) / 32;             // 32-component blocks of O^T
    constexpr int CPL = short_cpl(D);
    constexpr int RPW = 16 / NW;
    constexpr int VG = D <= 96 ? 16 : 4;          // keys whose V rows are in flight (the registers hold no more of longer rows)
    constexpr bool K_AHEAD = D == 64, V_AHEAD = D <= 96;     // ... nor the next unit's rows of all of them
    __shared__ typename ShortMerge<NW, DB>::Space s_merge;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n32 = lane & 31, hh = lane >> 5;
    const ShortWalk W(A, hm, lane);
    const int n = W.n;
    const bool rvalid = W.rvalid;
    float4 qf[H / 4];
    {
        const float* qrow = (const float*)A.q + (size_t)W.b * A.qs[0] + (size_t)W.h * A.qs[1] + (size_t)max(W.qpos, 0) * A.qs[2] + hh * H;
#pragma unroll
        for (int c = 0; c < H / 4; ++c) qf[c] = *(const float4*)(qrow + 4 * c);
    }
    const size_t koff = (size_t)W.b * A.ks[0] + (size_t)W.hk * A.ks[1];
    const char* kbase = (const char*)((const float*)A.k + koff);
    const char* vbase = (const char*)((const float*)A.v + koff);
    const unsigned pitch = A.pitch_bytes;
    const float scale = A.scale, cap = A.softcap;
    const float sl2 = cap > 0.f ? LOG2E : scale * LOG2E;     // logits (scores without a cap) to log2 units
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    int npairs = 0;

    struct Keys { uint4 km[4]; float4 kf[H / 4]; };
    auto load_keys = [&](int u, Keys& K) {
        if constexpr (D < 256) W.load_masks(u, K.km);
        const char* kr = kbase + (size_t)(unsigned)(32 * u) * pitch;
        const unsigned at = (unsigned)min(n32, n - 1 - 32 * u) * pitch + (unsigned)(hh * H) * 4u;
#pragma unroll
        for (int c = 0; c < H / 4; ++c) K.kf[c] = *(const float4*)(kr + (at + 16u * c));
    };
    // a half-wave's keys r0 .. r0 + VG - 1 of a unit, the lane's components of every block
    auto load_row = [&](const char* p, unsigned at, float (&x)[DB]) {
        __builtin_memcpy(&x[0], __builtin_assume_aligned(p + at, CPL * 4 < 16 ? CPL * 4 : 16), CPL * 4);
        if constexpr (D > 64 && D < 128) x[2] = 64 + n32 < D ? *(const float*)(p + (at + 256u - 4u * (unsigned)n32)) : 0.f;
    };
    const unsigned at_v = (unsigned)n32 * (4u * CPL), four = hh ? 4u * pitch : 0u;
    auto load_v = [&](int u, int r0, float (&vv)[VG][DB]) {
        if (32 * u + 32 <= n) {
#pragma unroll
            for (int r = 0; r < VG; ++r) load_row(vbase + (size_t)(unsigned)(32 * u + 8 * ((r0 + r) / 4) + r % 4) * pitch, four + at_v, vv[r]);
        } else {
#pragma unroll
            for (int r = 0; r < VG; ++r) load_row(vbase, (unsigned)min(32 * u + 8 * ((r0 + r) / 4) + 4 * hh + r % 4, n - 1) * pitch + at_v, vv[r]);
        }
    };
    auto any_nonfinite = [&](const float (&vv)[VG][DB]) -> bool {
        uint32_t top = 0u;
#pragma unroll
        for (int r = 0; r < VG; ++r)
#pragma unroll
            for (int db = 0; db < DB; ++db) top = max(top, __float_as_uint(vv[r][db]) & 0x7fffffffu);
        return __any(top >= 0x7f800000u);
    };
    bool again = false;                           // (uniform) values were taken out of a product
    Keys K;
    float vv[VG][DB];
    if (W.u0 + wave < W.u1) {
        if constexpr (K_AHEAD) load_keys(W.u0 + wave, K);
        if constexpr (V_AHEAD) load_v(W.u0 + wave, 0, vv);
    }
    for (int u = W.u0 + wave; u < W.u1; u += NW) {
        const bool more = u + NW < W.u1;
        if constexpr (D == 256) W.load_masks(u, K.km);                   // (its registers hold the words or the rows)
        else if constexpr (!K_AHEAD) load_keys(u, K);
        const unsigned ok = W.pairs(u, K.km);
        if constexpr (D == 256) {
            if (!__any(ok != 0u)) continue;
            load_keys(u, K);
        }
        const bool some = __any(ok != 0u);                               // else nothing here for any of the 32 rows
        const bool all_ok = !__any(rvalid && ok != 0xffffu);
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        if (some) {
#pragma unroll
            for (int c = 0; c < H / 4; ++c) {
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(K.kf[c].x, qf[c].x, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(K.kf[c].y, qf[c].y, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(K.kf[c].z, qf[c].z, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(K.kf[c].w, qf[c].w, s, 0, 0, 0);
            }
        }
        if (K_AHEAD && more) load_keys(u + NW, K);
        if (some) {
            // softmax step in log2 units: p = 2^(s * sl2 - m), one rounding in the exponent (a row's m cancels)
            if (cap > 0.f) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = cap * tanhf(s[r] * scale / cap);
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
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], sl2, -m_use));      // masked: 2^-inf = 0
                l += s[r];
            }
#pragma unroll
            for (int r0 = 0; r0 < 16; r0 += VG) {
                if constexpr (VG < 16) load_v(u, r0, vv);
                // A value that is not finite would reach the rows that do not attend it through 0 * inf: where the unit is
                // not attended as a whole it is taken out here and added below to the rows that do attend its key.
                if (!all_ok && any_nonfinite(vv)) {
                    again = true;
#pragma unroll
                    for (int r = 0; r < VG; ++r)
#pragma unroll
                        for (int db = 0; db < DB; ++db) vv[r][db] = __builtin_isfinite(vv[r][db]) ? vv[r][db] : 0.f;
                }
#pragma unroll
                for (int r = 0; r < VG; ++r)
#pragma unroll
                    for (int db = 0; db < DB; ++db)
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[r][db], s[r0 + r], o[db], 0, 0, 0);
            }
            if (A.row_pairs) npairs += __popc(ok);
        }
        if constexpr (V_AHEAD) if (more) load_v(u + NW, 0, vv);
    }
    // Infinities and NaN that were taken out (see the kernel above)
    if (again) {
#pragma unroll 1
        for (int u = W.u0 + wave; u < W.u1; u += NW) {
            uint4 km[4];
            W.load_masks(u, km);
            const unsigned ok = W.pairs(u, km);
            if (!__any(ok != 0u) || !__any(rvalid && ok != 0xffffu)) continue;
#pragma unroll
            for (int r0 = 0; r0 < 16; r0 += VG) {
                load_v(u, r0, vv);
                if (!any_nonfinite(vv)) continue;
#pragma unroll 1
                for (int neg = 0; neg < 2; ++neg) {
                    const unsigned flip = neg ? 0x80000000u : 0u;
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        f32x16 cnt;
#pragma unroll
                        for (int r = 0; r < 16; ++r) cnt[r] = 0.f;
#pragma unroll
                        for (int r = 0; r < VG; ++r)
                            cnt = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(__float_as_uint(vv[r][db]) ^ flip) < INFINITY ? 0.f : 1.f,
                                                                       (ok >> (r0 + r)) & 1u ? 1.f : 0.f, cnt, 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < 16; ++r) o[db][r] = cnt[r] > 0.f ? o[db][r] + (neg ? -INFINITY : INFINITY) : o[db][r];
                    }
                }
            }
        }
    }
    l += __shfl_xor(l, 32, 64);
    npairs += __shfl_xor(npairs, 32, 64);
    const ShortMerge<NW, DB> M(s_merge, o, m, l, npairs, wave, lane, min(NW, W.u1 - W.u0), A.row_pairs != nullptr);
    if (!rvalid) return;
    // an empty row (launch restricted to one pair set): out = 0, lse = -inf
    const float inv = (M.l > 0.f) ? 1.f / M.l : (M.l == 0.f) ? 0.f : M.l;
    float* orow = (float*)A.out + (size_t)W.b * A.os[0] + (size_t)W.h * A.os[1] + (size_t)W.qpos * A.os[2];
    const int i0 = M.first_row(wave, hh);
    float x[RPW * CPL];                           // components CPL * i0 ..: the blocks of a row in turn
#pragma unroll
    for (int e = 0; e < RPW; ++e)
#pragma unroll
        for (int db = 0; db < CPL; ++db) x[e * CPL + db] = M.acc[db][e] * inv;
    float4* o0 = (float4*)(orow + CPL * i0);
#pragma unroll
    for (int i = 0; i < RPW * CPL / 4; ++i) o0[i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
    if constexpr (D > 64 && D < 128) {
        if (64 + i0 < D) {
#pragma unroll
            for (int e = 0; e < RPW; e += 2) *(float2*)(orow + 64 + i0 + e) = make_float2(M.acc[2][e] * inv, M.acc[2][e + 1] * inv);
        }
    }
    if (wave == 0 && hh == 0) {
        const size_t row = (size_t)(W.b * A.Hq + W.h) * n + W.qpos;
        if (A.lse) A.lse[row] = fmaf(M.top, LN2, logf(M.l));
        if (A.row_pairs) A.row_pairs[row] = M.npairs;
    }
}

}  // namespace

// Rows in position order that attn_f32_kernel walks faster than attn_f32_linear_kernel: with 256 components the latter has no registers
// to ask for a unit's keys and values together, with 96 the loads of a value come in two sizes, and with 64 the former fits three work-groups
// of four wavefronts on a compute unit where there are no memberships.  Bucketing and attention, MHA, linear / by tiles (us), work-groups of 32 rows:
//   256: causal 1024 tokens x 384 groups 126 / 122, dense 138 / 132, x 800 241 / 246;  2048 x 768 375 / 350;  otherwise 1024 x 384 231 / 218, dense
//        239 / 220;  masked 700 x 400 187 / 183, x 88 92.5 / 97.4, dense 512 x 800 259 / 248, causal x 192 89.7 / 88.4, x 800 160 / 173
//   96:  causal 2048 x 768 150 / 138, dense 143 / 138 (x 640), 1024 x 1024 equal, x 1600 linear by 11 %;  otherwise dense 2048 x 768 231 / 226, masked 1.26 times linear
//   64:  otherwise dense 1024 x 768 111 / 99, 2048 x 768 186 / 162, x 640 155 / 161, x 896 192 / 203
bool by_tiles(const Layout& L)
{
    const long long groups = (long long)L.B * L.Hq * ((L.n + 31) / 32);
    if (L.d == 256) return L.n > 1024 || (L.n >= (!L.masked ? 512 : L.causal || groups <= 256 ? 768 : 640) && !(L.causal && groups > 384));
    if (L.d == 96) return L.n >= 1024 && groups <= 1024 && (L.causal ? groups > 512 : !L.masked);
    return L.d == 64 && !L.causal && !L.masked && L.n >= 1024 && groups > 704 && groups <= 768;
}

hipError_t launch_attn_f32(const Layout& L, const HeadMap& hm, const void* q, const void* k, const void* v, char* ws,
                           void* out, float* lse, int32_t* row_pairs, hipStream_t st)
{
    int default_map = (L.Hq % L.Hkv == 0) ? 1 : 0;
    for (int h = 0; default_map && h < L.Hq; ++h) default_map = hm.kv[h] == h / (L.Hq / L.Hkv);
    const size_t blocks = (size_t)L.NT * 4 * L.B * L.Hq;      // four quarters of every 128-row tile
    if (L.dtype != 0 || L.soft || L.BQ != 128 || blocks > 0x7fffffffull) return hipErrorInvalidValue;
    const bool wide = (uint64_t)L.ks[2] * 4 >= (1u << 24) || (uint64_t)L.n * (uint64_t)L.ks[2] * 4 >= 0xffffffffull;
    // Eight wavefronts share a work-group's units while there are at most two work-groups per compute unit: the chain
    // of every wavefront is then half as long (12 heads x 1024 tokens, d = 64: 45 -> 40 us); beyond that four, which
    // meet in one merge less (12 heads x 2048 tokens: 110 -> 96 us).  128 components are faster with eight at every
    // size (8 heads x 4096: 470 -> 400 us), 256 fill the registers of one wavefront per SIMD.
    const bool eight = L.d == 128 || (L.d < 128 && blocks <= 512);
    const ShortArgs A = short_args(L, hm, q, k, v, ws, out, lse, row_pairs);
    const bool linear = L.NC == 1 && !wide && !L.local_only && A.groups <= 65535;
#define FOCUS_F32N(D_, N_, W_, L_) hipLaunchKernelGGL((attn_f32_kernel<D_, N_, W_, L_>), dim3((unsigned)blocks), dim3(64 * N_), 0, st, L, hm, default_map, \
                                                  (const float*)q, (const float*)k, (const float*)v, (const char*)ws, (float*)out, lse, row_pairs)
#define FOCUS_F32W(D_, N_)                                                                                                \
    {                                                                                                                     \
        if (linear) hipLaunchKernelGGL((attn_f32_linear_kernel<D_, N_>), short_grid(A), dim3(64 * N_), 0, st, A, hm);    \
        else if (wide) FOCUS_F32N(D_, N_, true, false);                                                                   \
        else FOCUS_F32N(D_, N_, false, false);                                                                            \
    }
#define FOCUS_F32(D_) case D_: if (eight) FOCUS_F32W(D_, 8) else FOCUS_F32W(D_, 4) break;
    if (linear && by_tiles(L)) {
        if (L.d == 64) FOCUS_F32N(64, 4, false, true);
        else if (L.d == 96 && eight) FOCUS_F32N(96, 8, false, true);
        else if (L.d == 96) FOCUS_F32N(96, 4, false, true);
        else FOCUS_F32N(256, 4, false, true);
        return hipGetLastError();
    }
    switch (L.d) {
        FOCUS_F32(64) FOCUS_F32(80) FOCUS_F32(96)
        case 128: FOCUS_F32W(128, 8) break;
        case 256: FOCUS_F32W(256, 4) break;
        default: return hipErrorInvalidValue;
    }
#undef FOCUS_F32N
#undef FOCUS_F32
#undef FOCUS_F32W
    return hipGetLastError();
}

}  // namespace focus
