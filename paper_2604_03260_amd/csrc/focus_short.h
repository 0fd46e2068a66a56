// What the kernels for rows in position order with operands straight from the caches share (focus_attn_short.hip, focus_attn_f32.hip):
// their arguments, which 32-key units a work-group of 32 rows walks, which pairs of a unit count, and the merge.
#pragma once
#include "focus_internal.h"

namespace focus {

// What such a kernel needs of a Layout.  A launch begins with reading its arguments: a few cache lines in the place of the whole struct.
struct ShortArgs {
    const void *q, *k, *v;
    const uint32_t *mq, *kmsk;                    // membership masks: [B,Hq,n]; [B,Hkv,NKP] (masked only)
    void* out;
    float* lse;
    int32_t* row_pairs;
    long long qs[3], ks[2], os[3];                // strides in elements (batch, head, position)
    unsigned pitch_bytes;                         // of k and v, position; a head's rows lie within 4 GiB (the launch checks)
    int B, Hq, Hkv, n, NKP, window, causal, dense, pair_set, default_map;
    float scale, softcap;
    float cap_ratio, cap_rest;                    // scale / softcap and what its rounding left off
    int groups;                                   // of 32 rows
    const float* g;                               // soft gate: assignments [B,n,K] and -lambda * log2(e)
    float gate_slope;
    int K;
};

inline ShortArgs short_args(const Layout& L, const HeadMap& hm, const void* q, const void* k, const void* v, const char* ws, void* out,
                            float* lse, int32_t* row_pairs)
{
    ShortArgs A;
    A.q = q; A.k = k; A.v = v;
    A.mq = (const uint32_t*)(ws + L.off_mq); A.kmsk = (const uint32_t*)(ws + L.off_kmsk);
    A.out = out; A.lse = lse; A.row_pairs = row_pairs;
    for (int i = 0; i < 3; ++i) { A.qs[i] = L.qs[i]; A.os[i] = L.os[i]; }
    A.ks[0] = L.ks[0]; A.ks[1] = L.ks[1];
    A.pitch_bytes = (unsigned)L.ks[2] * (unsigned)L.elem;
    A.B = L.B; A.Hq = L.Hq; A.Hkv = L.Hkv; A.n = L.n; A.NKP = L.NKP; A.window = L.window; A.causal = L.causal;
    A.dense = L.masked ? 0 : 1; A.pair_set = L.pair_set;
    A.default_map = (L.Hq % L.Hkv == 0) ? 1 : 0;
    for (int h = 0; A.default_map && h < L.Hq; ++h) A.default_map = hm.kv[h] == h / (L.Hq / L.Hkv);
    A.scale = L.scale; A.softcap = L.softcap;
    const double ratio = L.softcap > 0.f ? (double)L.scale / (double)L.softcap : 0.0;
    A.cap_ratio = (float)ratio; A.cap_rest = (float)(ratio - (double)A.cap_ratio);
    A.groups = (L.n + 31) / 32;
    A.g = nullptr; A.gate_slope = L.gate_slope; A.K = L.K;
    return A;
}
// Grid: (batch and KV head, query head of it, groups of rows) with the default head map: the query heads of a KV head share an
// XCD, one L2, as long as there are a multiple of 8 of them; else (batch and query head, 1, groups).
inline dim3 short_grid(const ShortArgs& A)
{
    return A.default_map ? dim3(A.B * A.Hkv, A.Hq / A.Hkv, A.groups) : dim3(A.B * A.Hq, 1, A.groups);
}

// Row i of block db of O^T is component CPL * i + db: a lane's CPL components of a key lie side by side.  The third block of 80 and
// 96 components stands by itself, at 64 + i.
constexpr int short_cpl(int d) { return d < 128 ? 2 : d / 32; }

// A work-group's 32 rows (lane: row l%32) and the units of 32 keys that it walks.
struct ShortWalk {
    int b, h, hk, n, w, row0, qpos, hh;
    bool rvalid, causal, dense;
    int set;
    int u0, u1;                                   // units that hold a pair at all
    int in_beg, in_end;                           // without a test per pair: keys real, causal for every row and, where the window
                                                  // decides, inside every row's window
    int far_end;                                  // below it: outside every row's window and causal for all of them, membership decides alone
    uint32_t mq_row;
    const uint32_t* kmsk;

    __device__ inline ShortWalk(const ShortArgs& A, const HeadMap& hm, int lane)
    {
        const int heads = A.default_map ? A.Hkv : A.Hq;
        b = A.B == 1 ? 0 : (int)blockIdx.x / heads;
        const int x = (int)blockIdx.x - b * heads;
        h = A.default_map ? x * (int)gridDim.y + (int)blockIdx.y : x;
        hk = A.default_map ? x : hm.kv[h];
        n = A.n; w = A.window; hh = lane >> 5;
        row0 = (A.groups - 1 - (int)blockIdx.z) * 32;                    // longest causal prefix first
        const int last = min(row0 + 31, n - 1);
        rvalid = row0 + (lane & 31) < n;
        qpos = rvalid ? row0 + (lane & 31) : -1;
        dense = A.dense != 0;
        mq_row = rvalid && !dense ? A.mq[(size_t)(b * A.Hq + h) * n + qpos] : 0u;
        kmsk = A.kmsk + (size_t)(b * A.Hkv + hk) * A.NKP;
        causal = A.causal != 0;
        set = dense ? 0 : A.pair_set;
        const int x_hi = causal ? last + 1 : n;
        const bool local = set == 2;
        u0 = local ? max(0, row0 - w + 1) / 32 : 0;
        u1 = (dense && A.pair_set == 2) ? 0 : (min(x_hi, local ? last + w : x_hi) + 31) / 32;
        const int safe = causal ? row0 + 1 : dense ? n : min(n, row0 + w);
        in_beg = dense ? 0 : (max(last - w + 1, 0) + 31) / 32;
        in_end = set != 0 ? 0 : safe / 32;
        far_end = (causal && set == 0 && !dense) ? max(0, row0 - w + 1) / 32 : 0;
    }
    // scores of a unit at or below key offset x, bit r = score r: key 8*(r/4) + 4*hh + r%4
    __device__ inline unsigned upto(int x) const
    {
        const int c = x + 1 - 4 * hh;
        unsigned word = 0u;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) word |= ((1u << min(max(c - 8 * r4, 0), 4)) - 1u) << (4 * r4);
        return word;
    }
    __device__ inline void load_masks(int u, uint4 (&km)[4]) const
    {
        if (dense) return;
        const char* p = (const char*)(kmsk + 32 * u);
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) km[r4] = *(const uint4*)(p + 16u * (unsigned)hh + 32 * r4);
    }
    // which pairs of unit u count, bit r = score r
    __device__ inline unsigned pairs(int u, const uint4 (&km)[4]) const
    {
        if (u >= in_beg && u < in_end) return rvalid ? 0xffffu : 0u;
        unsigned ok = 0xffffu;
        if (!dense) {
            ok = 0u;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                ok |= ((mq_row & km[r4].x) ? 1u << (4 * r4) : 0u) | ((mq_row & km[r4].y) ? 2u << (4 * r4) : 0u) |
                      ((mq_row & km[r4].z) ? 4u << (4 * r4) : 0u) | ((mq_row & km[r4].w) ? 8u << (4 * r4) : 0u);
        }
        if (u >= far_end) {                       // positions decide too
            const int at = qpos - 32 * u;
            const unsigned cz = causal ? upto(at) : 0xffffu;
            const unsigned loc = (causal ? cz : upto(at + w - 1)) & ~upto(at - w);
            ok = set == 0 ? (loc | (ok & cz)) : set == 1 ? (ok & cz) : (loc & ~ok);
            if (32 * u + 32 > n) ok &= upto(n - 1 - 32 * u);
        }
        return rvalid ? ok : 0u;
    }
};

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float short_f32x16;
// App. D's merge of the wavefronts' partial softmaxes in one step: they all lie in LDS, and every wavefront adds up 16 / NW of the 16
// rows that a lane holds of every block.  (The upper half into the lower half until one is left: three steps and six
// barriers, 1.9 us of 12.4 at 512 tokens.)
template <int NW, int DB>
struct ShortMerge {
    static constexpr int RPW = 16 / NW;
    struct Space {
        float4 o[NW][DB * 4][64];
        float m[NW][32], l[NW][32];
        int np[NW][32];
    };
    float acc[DB][RPW], top, l;
    int npairs;
    // m, l, np: of the lane's row, the same in both half-waves; active: the first wavefronts of them had a unit
    __device__ inline ShortMerge(Space& S, const short_f32x16 (&o)[DB], float m, float l_wave, int np, int wave, int lane, int active, bool count)
    {
        const int n32 = lane & 31;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                S.o[wave][db * 4 + r4][lane] = make_float4(o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]);
        if (lane < 32) { S.m[wave][n32] = m; S.l[wave][n32] = l_wave; S.np[wave][n32] = np; }
        __syncthreads();
        float a[NW];
        top = -INFINITY;
        l = 0.f;
        npairs = 0;
#pragma unroll
        for (int w2 = 0; w2 < NW; ++w2) {
            a[w2] = w2 < active ? S.m[w2][n32] : -INFINITY;
            top = fmaxf(top, a[w2]);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e = 0; e < RPW; ++e) acc[db][e] = 0.f;
        const int r0 = wave * RPW;                // registers r0 .. r0 + RPW - 1 of every block
#pragma unroll
        for (int w2 = 0; w2 < NW; ++w2) {
            if (w2 >= active) break;              // (uniform)
            a[w2] = (a[w2] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(a[w2] - top);
            l = fmaf(S.l[w2][n32], a[w2], l);
            if (count) npairs += S.np[w2][n32];
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                float y[RPW];
                __builtin_memcpy(y, (const float*)&S.o[w2][db * 4 + r0 / 4][lane] + r0 % 4, sizeof(y));
#pragma unroll
                for (int e = 0; e < RPW; ++e) acc[db][e] = fmaf(y[e], a[w2], acc[db][e]);
            }
        }
    }
    // the first of the wavefront's RPW rows of every block
    static __device__ inline int first_row(int wave, int hh) { return 8 * (wave * RPW / 4) + 4 * hh + wave * RPW % 4; }
};

}  // namespace focus
