// Membership of 64 rows by one wavefront: fp64 scores against K centroids on the fp64 matrix cores, whose instructions add
// their four products to the accumulator one by one in index order with one rounding each (v_mfma_f64_4x4x4_4b: 256000
// random results equal the scalar fma chain bit for bit; 16x16x4: see focus_route.hip), so the scores are the sequential
// sums of Sec. 2 Eq. 1 bit for bit; then the topk best, ties to the smaller group.
//
// The 64 rows are four tiles of 16 that share the B operand (centroids, staged once per work-group [d][WP]); rows
// are staged a chunk at a time, coalesced, in the wavefront's own LDS, components 4*i + p of a row side by side for
// each p.  The A operand of both instructions is component 4*i + l/16 of row l%16.  16x16x4 runs on 16 columns, 64 cycles
// whatever K is; 4x4x4_4b is four blocks of 4 rows x 4 columns in 16 cycles, so up to 8 groups take one or two of those
// per tile and step.  Vector instructions do not run beside fp64 products (each adds 5 to 8 cycles to a step of 64), so
// the centroids are widened when they are staged where they are few.  State prefill of
// a generation, scores and lists: 8 x 131072 keys of 128, K = 8 154 -> 116 us; 8 x 32768, K = 4 45 -> 31; 96 x 4096 of 64, K = 4
// 35 -> 25.
#pragma once
#include "focus_internal.h"
#include <type_traits>

namespace focus {

typedef double score_f64x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t score_u32x4;

// up to 8 groups: products of 4 columns, centroids as doubles; more: products of 16 columns, centroids as floats
__host__ __device__ constexpr bool score_small(int km) { return km <= 8; }
// bytes of a row staged at a time: as many work-groups as fit count (bucketing with 128 -> 64: 40 heads of 128 x 32768, K = 16
// 360 -> 323 us; 20000 x 48 heads of 96, K = 4 130 -> 120), above 16 groups the space in which their scores meet does (493 / 677);
// 32-bit rows have half as many components in it (96 heads of 64 x 1024, K = 16: 23.4 / 21.9 with 128)
template <typename T> __host__ __device__ constexpr int score_chunk(int km) { return km <= 16 && sizeof(T) == 2 ? 64 : 128; }
// Chunks of a row asked for together.  Two are a whole cache line, which is otherwise fetched from L2 once for either half of it
// (a work-group's rows are far more than the vector cache holds); where the registers allow them.  Bucketing, one / two: K = 4
// top-2, 32 + 8 heads of 128 x 262144 882 / 866 us, 64 + 8 x 131072 715 / 697, 8 x 12 + 12 of 64 x 4096 39.8 / 37.1; state prefill of
// 8 x 131072 keys of 128 105 / 91.  K = 8 then has a wavefront less: 64 + 8 x 131072 876 / 896.
template <typename T> __host__ __device__ constexpr int score_depth(int km) { return km <= 4 && sizeof(T) == 2 ? 2 : 1; }
// Wavefronts per SIMD the bucketing's scoring asks for, 0: the compiler's choice.  Left to it, 16-bit rows ran at one less than
// the registers allow (its products' accumulators in a part of the register file of their own), and above 16 groups it went one
// register past two, with nothing left to run while a wavefront waits for its rows.  Whole bucketing, its choice / asked for (us):
// 16 + 4 heads of 64 x 131072, K = 8 top-2 209 / 202, K = 16 top-3 276 / 248; 40 + 8 of 128 x 32768, K = 16 282 / 258;
// 16 + 4 of 128 x 131072, K = 24 top-2 1018 / 675; 32 + 8 of 64 x 16384, K = 24 196 / 131; K = 20 top-1 in fp32 296 / 196
template <typename T> __host__ __device__ constexpr int score_waves(int km)
{
    return km == 32 ? 2 : sizeof(T) == 4 ? 0 : km == 16 ? 4 : km == 8 ? 5 : 4;
}
// LDS pitch of a staged row: four interleaved parts, padded; staging bytes per wavefront
__host__ __device__ constexpr int score_a_row(int chunk) { return chunk + 16; }
__host__ __device__ constexpr int score_lds(int chunk) { return 64 * score_a_row(chunk); }
// LDS pitch (elements) of a component's centroid values: KM groups, zero past K; the rows a step reads on different banks
__host__ __device__ constexpr int score_wp(int km) { return score_small(km) ? km : km <= 16 ? 16 : 48; }
// bytes of the staged centroids
__host__ __device__ constexpr size_t score_cent_bytes(int km, int d) { return (size_t)d * score_wp(km) * (score_small(km) ? 8 : 4); }
template <int KM> using score_cent_t = std::conditional_t<score_small(KM), double, float>;

// all threads: centroids [K][d] fp32 -> s_c [d][WP]
template <int KM>
__device__ inline void score_stage_centroids(const float* __restrict__ c, score_cent_t<KM>* s_c, int K, int d)
{
    constexpr int WP = score_wp(KM);
    // a few loads in flight per thread (one at a time, the staging is a chain of up to 48 round trips: whole bucketing of
    // 32 + 8 heads of 128 x 16384, K = 32 top-2 198 -> 192 us; two up to 16 groups: four made the
    // state prefill of a generation 1 to 2 % longer)
    constexpr int BT = KM <= 16 ? 2 : 4;
    for (int e0 = threadIdx.x; e0 < d * WP; e0 += BT * blockDim.x) {
        float v[BT];
#pragma unroll
        for (int i = 0; i < BT; ++i) {
            const int e = e0 + i * blockDim.x, t = e / WP, g = e % WP;
            v[i] = e < d * WP && g < K ? c[(size_t)g * d + t] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < BT; ++i) {
            const int e = e0 + i * blockDim.x;
            if (e < d * WP) s_c[e] = (score_cent_t<KM>)v[i];
        }
    }
}

// acc + the sum of the squares of the eight 16-bit values of a piece (bf16 or IEEE half bit patterns), products in fp32
__device__ inline float piece_norm2(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, bool f16, float acc)
{
    const uint32_t w[4] = {w0, w1, w2, w3};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = f16 ? f16_bits_to_f32((uint16_t)(w[e] & 0xffffu)) : __uint_as_float(w[e] << 16);
        const float b = f16 ? f16_bits_to_f32((uint16_t)(w[e] >> 16)) : __uint_as_float(w[e] & 0xffff0000u);
        acc = fmaf(a, a, acc);
        acc = fmaf(b, b, acc);
    }
    return acc;
}

// gbase: first row, pitch: bytes between rows, rows: at most 64 of them; abuf: score_lds(CHUNK) bytes of the wavefront's own.
// staged: called once by all wavefronts of the work-group, after their first loads are on their way: stages the centroids
// and waits for them.  want_norm (16-bit types): n2max takes the bit pattern of the largest squared norm of the rows (a
// non-negative float orders like its bit pattern, a NaN or infinite norm ends up above every finite one), else it is left as
// it is.  Returns the mask of row `lane` (0 past the rows).  KM = K rounded up to 4, 8, 16 or 32.
template <typename T, int KM, int CHUNK, typename F>
__device__ inline uint32_t score_rows_topk(const char* __restrict__ gbase, size_t pitch, int rows, int d, const score_cent_t<KM>* s_c,
                                           char* abuf, int K, int topk, F&& staged, bool want_norm, unsigned& n2max)
{
    constexpr int A_ROW = score_a_row(CHUNK);
    constexpr int RC = CHUNK / (int)sizeof(T);    // components per staged chunk
    constexpr int NP = CHUNK / 16;                // 16-byte pieces of a row's chunk = loads per lane = dwords of a part
    constexpr bool SMALL = score_small(KM);
    constexpr int CB = SMALL ? KM / 4 : KM <= 16 ? 1 : 2;         // blocks of 4 or of 16 columns
    constexpr int LC = SMALL ? 3 : 15;            // lane bits that say which column of a block
    constexpr int WP = score_wp(KM);
    constexpr int SP = KM + 1;                    // doubles per row when the scores meet in LDS
    constexpr int TG = (16 * 4 * SP * 8 <= score_lds(CHUNK)) ? 4 : (16 * 2 * SP * 8 <= score_lds(CHUNK)) ? 2 : 1;    // tiles whose scores fit the staging space
    static_assert(16 * TG * SP * 8 <= score_lds(CHUNK), "scores stay inside the staging space");
    const int lane = threadIdx.x & 63;
    const int row_bytes = d * (int)sizeof(T);
    const int nchunk = (d + RC - 1) / RC;
    constexpr int DEPTH = score_depth<T>(KM);
    score_u32x4 stage[DEPTH][NP];
    auto load_chunks = [&](int ch) {              // chunks ch .. ch + DEPTH - 1
#pragma unroll
        for (int i = 0; i < NP; ++i)
#pragma unroll
            for (int p = 0; p < DEPTH; ++p) {
                const int row = i * (64 / NP) + lane / NP, byte = (ch + p) * CHUNK + lane % NP * 16;
                const score_u32x4 z = {0u, 0u, 0u, 0u};
                stage[p][i] = (row < rows && byte < row_bytes) ? *(const score_u32x4*)(gbase + (size_t)row * pitch + byte) : z;
            }
    };
    typedef std::conditional_t<SMALL, double, score_f64x4> acc_t;
    acc_t acc[4][CB];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[t][cb] = acc_t{};
    load_chunks(0);
    staged();
    if (rows <= 0) return 0;
    float n2[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) n2[i] = 0.f;
    for (int ch0 = 0; ch0 < nchunk; ch0 += DEPTH) {
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) {
            const int ch = ch0 + p;
            if (p > 0 && ch >= nchunk) break;
            const score_u32x4 (&stg)[NP] = stage[p];
            // a wavefront's LDS accesses run in order: no barrier, only the compiler must keep the order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                uint32_t* dst = (uint32_t*)(abuf + (i * (64 / NP) + lane / NP) * A_ROW) + lane % NP;
                const score_u32x4 v = stg[i];
                if constexpr (sizeof(T) == 4) {
                    dst[0] = v[0]; dst[NP] = v[1]; dst[2 * NP] = v[2]; dst[3 * NP] = v[3];
                } else {
                    dst[0] = (v[0] & 0xffffu) | (v[2] << 16);
                    dst[NP] = (v[0] >> 16) | (v[2] & 0xffff0000u);
                    dst[2 * NP] = (v[1] & 0xffffu) | (v[3] << 16);
                    dst[3 * NP] = (v[1] >> 16) | (v[3] & 0xffff0000u);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if constexpr (sizeof(T) == 2) {
                if (want_norm) {
#pragma unroll
                    for (int i = 0; i < NP; ++i)
                        n2[i] = piece_norm2(stg[i][0], stg[i][1], stg[i][2], stg[i][3], std::is_same<T, f16_bits>::value, n2[i]);
                }
            }
            if (p == DEPTH - 1 && ch + 1 < nchunk) load_chunks(ch + 1);
            constexpr int AR = NP / 4;                // 16-byte reads of a part
            score_u32x4 ar[4][AR];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const score_u32x4* src = (const score_u32x4*)(abuf + (t * 16 + (lane & 15)) * A_ROW + (lane >> 4) * (4 * NP));
#pragma unroll
                for (int i = 0; i < AR; ++i) ar[t][i] = src[i];
            }
            const score_cent_t<KM>* wr = s_c + (ch * RC + (lane >> 4)) * WP + (lane & LC);
            const int steps = min(RC, d - ch * RC) / 4;
            auto step = [&](int i) {
                double bv[CB];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) bv[cb] = (double)wr[i * 4 * WP + cb * (LC + 1)];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    double a;
                    if constexpr (sizeof(T) == 4) {
                        a = (double)__uint_as_float(ar[t][(i / 4) % AR][i % 4]);
                    } else {
                        const uint32_t w2 = ar[t][(i / 8) % AR][(i / 2) % 4];
                        if constexpr (std::is_same<T, f16_bits>::value)
                            a = (double)f16_bits_to_f32((uint16_t)(i % 2 ? w2 >> 16 : w2 & 0xffffu));
                        else
                            a = (double)__uint_as_float(i % 2 ? w2 & 0xffff0000u : w2 << 16);
                    }
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        if constexpr (SMALL) acc[t][cb] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, bv[cb], acc[t][cb], 0, 0, 0);
                        else acc[t][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv[cb], acc[t][cb], 0, 0, 0);
                    }
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
    }
    if constexpr (sizeof(T) == 2) {
        if (want_norm) {
            unsigned top = 0u;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
#pragma unroll
                for (int off = 1; off < NP; off <<= 1) n2[i] += __shfl_xor(n2[i], off, 64);
                const unsigned bits = __float_as_uint(n2[i]) & 0x7fffffffu;      // a NaN may carry a sign bit
                top = bits > top ? bits : top;
            }
#pragma unroll
            for (int off = NP; off <= 32; off <<= 1) {
                const unsigned o = (unsigned)__shfl_xor((int)top, off, 64);
                top = o > top ? o : top;
            }
            n2max = top;
        }
    }
    // accumulator of lane l: row 4*(l%16/4) + l/16 of the tile, group l%4 of the block; register r of the 16-column
    // product: row 4*r + l/16, group l%16
    double* s_s = (double*)abuf;
    uint32_t mask = 0;
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += TG) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                if constexpr (SMALL) {
                    s_s[(t * 16 + (lane & 12) + (lane >> 4)) * SP + cb * 4 + (lane & 3)] = acc[t0 + t][cb];
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (cb * 16 + (lane & 15) < KM)
                            s_s[(t * 16 + 4 * r + (lane >> 4)) * SP + cb * 16 + (lane & 15)] = acc[t0 + t][cb][r];
                }
            }
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

template <typename T, int KM, int CHUNK, typename F>
__device__ inline uint32_t score_rows_topk(const char* __restrict__ gbase, size_t pitch, int rows, int d, const score_cent_t<KM>* s_c,
                                           char* abuf, int K, int topk, F&& staged)
{
    unsigned unused = 0u;
    return score_rows_topk<T, KM, CHUNK>(gbase, pitch, rows, d, s_c, abuf, K, topk, staged, false, unused);
}

}  // namespace focus
