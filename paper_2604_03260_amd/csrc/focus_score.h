// Membership of 64 rows by one wavefront: fp64 scores against K centroids on v_mfma_f64_16x16x4, which adds its four
// products to the accumulator one by one in index order with one rounding each (see focus_route.hip), so the scores are
// the sequential sums of Sec. 2 Eq. 1 bit for bit; top-k by rank counting, ties to the smaller group.
//
// The 64 rows are four tiles of 16 that share the B operand (centroids, staged once per work-group as fp32 [d][WP]); rows
// are staged 128 bytes at a time, coalesced, in the wavefront's own LDS, components 4*i + p of a row side by side for
// each p.  A product runs on 16 columns, so up to 16 groups cost the same.
#pragma once
#include "focus_internal.h"
#include <type_traits>

namespace focus {

typedef double score_f64x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t score_u32x4;
constexpr int SCORE_A_ROW = 128 + 16;             // LDS pitch of a staged row: four interleaved parts of 32 bytes, padded
constexpr int SCORE_LDS = 64 * SCORE_A_ROW;       // staging bytes per wavefront

// LDS pitch (floats) of a component's centroid values: KM groups, zero past K; the rows a step reads on different banks
__host__ __device__ constexpr int score_wp(int km) { return km <= 16 ? 16 : 48; }

// all threads: centroids [K][d] fp32 -> s_c [d][WP]
template <int KM>
__device__ inline void score_stage_centroids(const float* __restrict__ c, float* s_c, int K, int d)
{
    constexpr int WP = score_wp(KM);
    for (int e = threadIdx.x; e < d * WP; e += blockDim.x) {
        const int t = e / WP, g = e % WP;
        s_c[e] = g < K ? c[(size_t)g * d + t] : 0.f;
    }
}

// gbase: first row, pitch: bytes between rows, rows: 1 .. 64 of them; abuf: SCORE_LDS bytes of the wavefront's own.
// Returns the mask of row `lane` (0 past the rows).  KM = K rounded up to 4, 8, 16 or 32.
template <typename T, int KM>
__device__ inline uint32_t score_rows_topk(const char* __restrict__ gbase, size_t pitch, int rows, int d, const float* s_c,
                                           char* abuf, int K, int topk)
{
    constexpr int RC = 128 / (int)sizeof(T);      // components per staged chunk
    constexpr int CB = KM <= 16 ? 1 : 2;          // blocks of 16 columns
    constexpr int WP = score_wp(KM);
    constexpr int SP = KM + 1;                    // doubles per row when the scores meet in LDS
    constexpr int TG = (16 * 4 * SP * 8 <= SCORE_LDS) ? 4 : 2;        // tiles whose scores fit the staging space
    static_assert(16 * TG * SP * 8 <= SCORE_LDS, "scores stay inside the staging space");
    const int lane = threadIdx.x & 63;
    const int row_bytes = d * (int)sizeof(T);
    const int nchunk = (d + RC - 1) / RC;
    score_u32x4 stg[8];
    auto load_chunk = [&](int ch) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = i * 8 + lane / 8, byte = ch * 128 + lane % 8 * 16;
            const score_u32x4 z = {0u, 0u, 0u, 0u};
            stg[i] = (row < rows && byte < row_bytes) ? *(const score_u32x4*)(gbase + (size_t)row * pitch + byte) : z;
        }
    };
    score_f64x4 acc[4][CB];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[t][cb] = score_f64x4{0.0, 0.0, 0.0, 0.0};
    load_chunk(0);
    for (int ch = 0; ch < nchunk; ++ch) {
        // a wavefront's LDS accesses run in order: no barrier, only the compiler must keep the order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t* dst = (uint32_t*)(abuf + (i * 8 + lane / 8) * SCORE_A_ROW) + lane % 8;
            const score_u32x4 v = stg[i];
            if constexpr (sizeof(T) == 4) {
                dst[0] = v[0]; dst[8] = v[1]; dst[16] = v[2]; dst[24] = v[3];
            } else {
                dst[0] = (v[0] & 0xffffu) | (v[2] << 16);
                dst[8] = (v[0] >> 16) | (v[2] & 0xffff0000u);
                dst[16] = (v[1] & 0xffffu) | (v[3] << 16);
                dst[24] = (v[1] >> 16) | (v[3] & 0xffff0000u);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (ch + 1 < nchunk) load_chunk(ch + 1);
        score_u32x4 ar[4][2];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const score_u32x4* p = (const score_u32x4*)(abuf + (t * 16 + (lane & 15)) * SCORE_A_ROW + (lane >> 4) * 32);
            ar[t][0] = p[0];
            ar[t][1] = p[1];
        }
        const float* wr = s_c + (ch * RC + (lane >> 4)) * WP + (lane & 15);
        const int steps = min(RC, d - ch * RC) / 4;
        auto step = [&](int i) {
            double bv[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) bv[cb] = (double)wr[i * 4 * WP + cb * 16];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                double a;
                if constexpr (sizeof(T) == 4) {
                    a = (double)__uint_as_float(ar[t][(i / 4) % 2][i % 4]);
                } else {
                    const uint32_t w2 = ar[t][(i / 8) % 2][(i / 2) % 4];
                    if constexpr (std::is_same<T, f16_bits>::value)
                        a = (double)f16_bits_to_f32((uint16_t)(i % 2 ? w2 >> 16 : w2 & 0xffffu));
                    else
                        a = (double)__uint_as_float(i % 2 ? w2 & 0xffff0000u : w2 << 16);
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[t][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv[cb], acc[t][cb], 0, 0, 0);
            }
        };
        if (steps == RC / 4) {
#pragma unroll
            for (int i = 0; i < RC / 4; ++i) step(i);
        } else {                                  // the last chunk of 80 or 96 components
#pragma unroll
            for (int i = 0; i < RC / 4; ++i)
                if (i < steps) step(i);
        }
    }
    // accumulator register r of lane l: row 4*r + l/16 of the tile, group l%16
    double* s_s = (double*)abuf;
    uint32_t mask = 0;
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += TG) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (cb * 16 + (lane & 15) < KM)
                        s_s[(t * 16 + 4 * r + (lane >> 4)) * SP + cb * 16 + (lane & 15)] = acc[t0 + t][cb][r];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane / (TG * 16) == t0 / TG && lane < rows) {
            // The best group topk times, ties to the smaller index (strictly greater replaces).  Any NaN among the scores
            // gives the first topk groups.  (Rank counting compares all pairs: 32 groups took 150 us at any length.)
            double sc[KM];
#pragma unroll
            for (int g = 0; g < KM; ++g) sc[g] = s_s[(lane - t0 * 16) * SP + g];
            bool nan = false;
#pragma unroll
            for (int g = 0; g < KM; ++g) nan = nan || (g < K && sc[g] != sc[g]);
            uint32_t m = 0;
            for (int t = 0; t < topk; ++t) {
                double best = 0.0;
                uint32_t bit = 0;
#pragma unroll
                for (int g = 0; g < KM; ++g) {
                    const bool take = g < K && !((m >> g) & 1u) && (bit == 0u || sc[g] > best);
                    best = take ? sc[g] : best;
                    bit = take ? 1u << g : bit;
                }
                m |= bit;
            }
            if (nan) m = (topk == 32) ? 0xffffffffu : ((1u << topk) - 1u);
            mask = m;
        }
    }
    return mask;
}

}  // namespace focus
