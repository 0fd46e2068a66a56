// focus_route: the per-layer router (Sec. 2 Eq. 1 and the Sinkhorn recipe under it).
//
//   z_i = W_g^T h_i,  S[i,g] = z_i . C[g],  then either g_i = S[i,:] / tau (no normalisation)
//   or Q = exp(S / tau) followed by N rounds of {columns / their sum over the sequence's tokens,
//   rows / their sum over the groups}; the top-k entries of a row become the token's membership.
//
// Everything is fp64.  The projection is the plain inner product of Eq. 1: its products are exact
// (fp32 x bf16/fp16/fp32 fits in fp64) and are added one by one in index order t = 0 .. d_model-1 (one
// fused multiply-add per term, which rounds once, like an exact product followed by an add), so z, S
// and, without Sinkhorn, the membership are reproducible bit for bit.
//
// Kernels:
//   route_project     a wavefront = 16 tokens x all router outputs on the fp64 matrix cores, or, of few tokens, four of the
//                     outputs (see the kernel); writes S, the work-group's largest score, and the masks directly when no
//                     Sinkhorn is asked;
//   sinkhorn_rounds   Sinkhorn in one launch wherever its rows fit the registers of few enough work-groups (sink_groups); the
//                     same sums as
//   sinkhorn_pass     a launch per round: Sinkhorn as diagonal scaling: Q = diag(u) E diag(v) with E = exp((S - max)/tau).
//                     A round is  v_g = 1 / sum_i u_i E[i,g],  u_i = 1 / sum_g E[i,g] v_g,  so one pass
//                     over E per round: every work-group first folds the previous pass's per-block
//                     column partial sums (fixed order, no atomics: deterministic), then updates its
//                     rows and leaves its own partial sums for the next pass.  The last pass writes
//                     the masks (ties to the smaller group index) and, if asked, the soft assignment.
#include "focus_internal.h"
#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <type_traits>

namespace focus {

// Scratch of focus_route_noalloc: device memory of the library's own image, one copy per GPU, held until the
// process ends.  Host code never uses this name as an address: route_static_scratch() asks the runtime for the
// array's device address once per device and hands that pointer to the kernels like any workspace.
static __device__ __align__(256) unsigned char scratch[ROUTE_STATIC_SCRATCH_BYTES];

hipError_t route_static_scratch(char** ptr)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static char* per_device[MAX_DEVICES] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));      // the copy of the array on the current device
        if (e != hipSuccess) return e;
        if (!p || ((uintptr_t)p & 255) != 0) return hipErrorInvalidSymbol;
        per_device[dev] = (char*)p;
    }
    *ptr = per_device[dev];
    return hipSuccess;
}

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ inline double wave_max(double x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x = fmax(x, __shfl_xor(x, off, 64));
    return x;
}

__device__ inline double wave_sum(double x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x = __dadd_rn(x, __shfl_xor(x, off, 64));
    return x;
}

// Sums of KP columns over a wavefront at once: every step halves the columns a lane carries until one is left (of lane
// bits 5, 4, ..), 7 exchanges for 4 columns instead of 24.  Returns the sum of column wave_column<KP>(lane).
template <int KP>
__device__ inline int wave_column(int lane)
{
    int c = 0;
    for (int w = KP / 2, off = 32; w >= 1; w >>= 1, off >>= 1) c += (lane & off) ? w : 0;
    return c;
}
template <int KP>
__device__ inline double wave_sum_columns(const double (&x)[KP], int lane)
{
    static_assert(KP >= 2 && KP <= 32 && (KP & (KP - 1)) == 0, "a power of two");
    double y[KP];
#pragma unroll
    for (int g = 0; g < KP; ++g) y[g] = x[g];
    int off = 32;
#pragma unroll
    for (int w = KP / 2; w >= 1; w >>= 1, off >>= 1) {
        const bool up = (lane & off) != 0;
#pragma unroll
        for (int g = 0; g < w; ++g) {
            const double send = up ? y[g] : y[g + w];
            y[g] = __dadd_rn(up ? y[g + w] : y[g], __shfl_xor(send, off, 64));
        }
    }
#pragma unroll
    for (; off >= 1; off >>= 1) y[0] = __dadd_rn(y[0], __shfl_xor(y[0], off, 64));
    return y[0];
}

// top-k of the first K of KP register values: the best value topk times, ties to the smaller index (strictly greater
// replaces).  A NaN among the scores gives the first topk groups.  (Comparing all pairs, unrolled, spilled 1700 registers
// at 32 groups.)
template <int KP>
__device__ inline uint32_t topk_mask(const double (&s)[KP], int K, int topk)
{
    bool nan = false;
#pragma unroll
    for (int g = 0; g < KP; ++g) nan = nan || (g < K && s[g] != s[g]);
    uint32_t m = 0;
    for (int t = 0; t < topk; ++t) {
        double best = 0.0;
        uint32_t bit = 0;
#pragma unroll
        for (int g = 0; g < KP; ++g) {
            const bool take = g < K && !((m >> g) & 1u) && (bit == 0u || s[g] > best);
            best = take ? s[g] : best;
            bit = take ? 1u << g : bit;
        }
        m |= bit;
    }
    if (nan) m = (topk == 32) ? 0xffffffffu : ((1u << topk) - 1u);
    return m;
}

// ---------------------------------------------------------------- how the Sinkhorn rounds are launched
// Groups padded to a power of two, as the kernels hold them.
constexpr int sink_kp(int K) { return K <= 4 ? 4 : K <= 8 ? 8 : K <= 16 ? 16 : 32; }
// Rows per thread of an instantiation for `tokens` tokens of a work-group (0: more than pays, or than the registers hold, 64 doubles a
// thread.  Of up to 4 groups 14, below the 16 that they would hold: 200000 tokens, a launch per round / one 127 / 123 us, 262144 136.5 / 139).
constexpr int sink_rows(int kp, int tokens)
{
    const int rows = (tokens + 255) / 256, most = kp == 4 ? 14 : 64 / kp;
    return rows > most ? 0 : rows <= 2 ? 2 : rows <= 4 ? 4 : rows <= 8 ? 8 : 16;
}
// Work-groups of an instantiation that a compute unit holds (its launch bounds): 16 and 32 padded groups with 64 doubles a thread take all
// registers of a SIMD.
constexpr int sink_resident(int kp, int rows) { return kp >= 16 && kp * rows >= 64 ? 1 : 2; }
// All rounds in one launch: work-groups per sequence, or 0 where the rows do not fit the registers or there are too many sequences.
// Work-groups that exchange their sums should be resident together; one that is left waiting computes the others' sums itself
// (sinkhorn_rounds_kernel), which is right but slow.  So a launch takes at most a quarter of the work-groups that the device holds: four
// launches at once, one on each hardware queue, still fit.
// One work-group as long as its rows take less time than an exchange (K = 4, d_model 768: 2000 tokens 40 us in one, 4000 37 in several),
// else one for every 512 tokens, the most that fit two rows a thread, as far as the slots do.  Routing with ten rounds, a launch per
// round / one (us; up to 8192 tokens the projection in work-groups of 16 tokens comes with the latter): 2 x 500 tokens, K = 8, d_model
// 3840 106 / 62;  2000, K = 4, 768 51 / 38;  4493, K = 8, 4096 115 / 93;  16000, K = 16, 768 84 / 77 (in 31 work-groups of 517 tokens and
// four rows 86);  32768, K = 4, 4096 142 / 133;  4 x 9000, K = 16, 768 108 / 98;  200000, K = 4, 256 109 / 108.
inline int sink_groups(const RouteLayout& R, int compute_units)
{
    const int kp = sink_kp(R.K);
    if ((long long)R.n * kp <= 6144) return 1;
    for (int per_unit = 2; per_unit >= 1; --per_unit) {
        const int g = std::min({(R.nsink + 1) / 2, 16 * R.nsink / R.K, 64, compute_units / 4 * per_unit / R.B});
        const int rows = g >= 2 ? sink_rows(kp, (R.n + g - 1) / g) : 0;
        if (rows > 0 && sink_resident(kp, rows) >= per_unit) return g;
    }
    return sink_rows(kp, R.n) > 0 ? 1 : 0;
}
// Column sums on their way between the work-groups: [3][work-groups][K] per sequence, in the place of the partial sums of the
// launches.  A slot is EMPTY until its sum is there.
constexpr unsigned long long SINK_EMPTY = ~0ull;
constexpr int SINK_LOOKS = 4096;                  // for a sum that is not there yet, about a microsecond each
__device__ inline unsigned long long* sink_slots(const RouteLayout& R, char* ws, int b)
{
    return (unsigned long long*)(ws + R.off_colpart) + (size_t)b * (3 * R.nround * R.K);     // at most 48 of the 64 * nsink words
}

// ---------------------------------------------------------------- projection + scores
// z = W_g^T h on the fp64 matrix cores.  v_mfma_f64_16x16x4 adds its four products to the accumulator one by one in
// index order, each with one rounding (a fused multiply-add; checked on 512000 results against the scalar chain, and
// by the bit-exact router tests), so one instruction is four steps of the same sum as before for 16 tokens x 16 outputs.
// The vector form of this kernel (a lane per token, W_g through scalar loads) reached 17 % of the fp64 rate at 32768
// tokens, held by the issue of fp64 instructions (one per 16 cycles and wavefront) and by the scalar loads; a matrix
// instruction keeps the fp64 units busy for 64 cycles by itself.  32768 x 4096 bf16, d_g = 16: 306 -> 104 us
// (41 TFLOP/s; products alone reach 60 to 73 on this chip, and every widening of a value adds to them); 1024 tokens 275 -> 73 us,
// 131072 tokens 521 -> 353 us, d_g = 64 x 2048: 306 -> 177 us.
//
// A work-group is NW wavefronts of 16 tokens.  Hidden rows and W_g (fp32) pass through LDS in chunks of 128 bytes per
// row, two buffers, one barrier per chunk, the next four chunks' loads in flight meanwhile.  The A operand of step i is
// component 4*i + l/16 of token l%16: rows are stored with the components of one l/16 side by side, so a lane reads
// its whole chunk with two 16-byte loads.  Accumulator register r of lane l is token 4*r + l/16, output l%16.
//
// d_g = 4 and 8 run on v_mfma_f64_4x4x4_4b (focus_score.h), one or two of 16 cycles per step in the place of one of 64: 20000 x 8192
// f16, d_g = 8: 224 -> 157 us; 32768 x 1200 bf16, d_g = 4: 36 -> 22.  Four of them per step would be no faster at d_g = 16: a step is
// then as long, and widens three more values of W_g (112 -> 135 us; vector instructions do not run beside fp64 products).
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int A_ROW = 128 + 16;              // LDS pitch of a staged row: 4 interleaved parts of 32 bytes, padded
__host__ __device__ constexpr bool route_small(int dg) { return dg <= 8; }
// LDS pitch of a row of W_g (elements): the four rows of a step on different banks
__host__ __device__ constexpr int route_wp(int dg) { return dg <= 16 ? dg : dg + 16; }
// ... which is widened when it is staged where the space allows it, not by every wavefront at every step
template <int DG> using route_w_t = std::conditional_t<DG <= 16, double, float>;

// Wavefronts per SIMD asked for; 0: the compiler's choice.  The operands of four steps took the wide projections past the registers
// of the wavefronts that one step at a time had left (4096 -> 64, bf16, 32768 tokens: 345 us one by one, 413 with four steps in
// one wavefront, 333 in two; 1024 -> 64, 131072: 368 / 474 / 363; 1024 -> 32 in fp32, 131072: 193 / 205 in three, 192 in four).
template <typename T> constexpr int route_waves(int dg) { return dg == 64 ? 2 : (dg == 32 && sizeof(T) == 4) ? 4 : 0; }

// SPLIT (d_g = 16): few tokens leave the chip idle behind a chain of one 64-cycle product per four components.  A work-group then is 16
// tokens, its four wavefronts take four outputs each, one product of 16 cycles a step; all wavefronts read the same rows.
// Routing, whole / split (us), ten rounds, K = 4, bf16: d_model 4096: 500 tokens 83 / 60, 2000 99 / 75, 8000 98 / 84, 12000 104 / 101, 16000 103 / 116;
// 768: 500 30 / 25, 8000 44 / 42, 12000 50 / 50; fp32, 4096: 500 98 / 71, 8000 113 / 97, 12000 118 / 112, 16000 120 / 132.  Without rounds and
// above 16 groups, whose masks take K * K steps a token here, only up to 4096 tokens: K = 32, d_model 768: 2000 85 / 82, 8000 85 / 94.
// CLEAR: the slots of the Sinkhorn sums are emptied here.  A template, since the branch alone cost projections without rounds 1 to 2.5 % (500 tokens,
// K = 32, d_g = 8 80.3 -> 82.3 us; 130 x 600 fp32, K = 8 75.6 -> 82.5).
template <typename T, int DG, int NW, bool SPLIT, bool CLEAR>
__global__ __launch_bounds__(64 * NW, route_waves<T>(DG)) void route_project_kernel(RouteLayout R, const T* __restrict__ hidden,
                                                                 const float* __restrict__ wg,
                                                                 const float* __restrict__ cent,
                                                                 char* __restrict__ ws,
                                                                 uint32_t* __restrict__ masks,
                                                                 double* __restrict__ soft)
{
    static_assert(!SPLIT || (DG == 16 && NW == 4), "four outputs for each of four wavefronts");
    constexpr int NTHR = 64 * NW, TB = SPLIT ? 16 : 16 * NW;
    constexpr int RC = 128 / (int)sizeof(T);             // components per chunk
    constexpr bool SMALL = route_small(DG) || SPLIT;
    constexpr int LC = SMALL ? 3 : 15, CB = SPLIT ? 1 : (DG + LC) / (LC + 1);    // column of a block, blocks of 4 or of 16 outputs
    constexpr int NP = SPLIT ? 1 : 2;                    // 16-byte pieces of the rows per thread and chunk (SPLIT: of the first 128 threads)
    constexpr int WP = route_wp(DG);
    typedef route_w_t<DG> w_t;
    typedef std::conditional_t<SMALL, double, f64x4> acc_t;
    constexpr int PF = 4;                                // chunks in flight: one takes 0.85 us of products, a load 1 to 2
    constexpr int WPT = (RC * DG + NTHR - 1) / NTHR;     // floats of W_g per thread and chunk
    // dynamic LDS: two buffers of hidden rows and of W_g during the projection, then z [TB][DG+1] and S [TB][K|1]
    extern __shared__ __align__(16) char s_dyn[];
    __shared__ double s_wmax[NW];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.y;
    const int tok0 = blockIdx.x * TB;
    const int n = R.n, dm = R.dm, K = R.K;
    const int rows = min(TB, n - tok0);
    const int row0 = SPLIT ? 0 : wave * 16, col0 = SPLIT ? wave * 4 : 0;         // of this wavefront
    const int row_bytes = dm * (int)sizeof(T);
    const char* gbase = (const char*)hidden + ((size_t)b * n + tok0) * row_bytes;
    const int nchunk = (dm + RC - 1) / RC;
    char* s_a = s_dyn;
    w_t* s_w = (w_t*)(s_dyn + 2 * TB * A_ROW);

    u32x4 sta[PF][NP];
    float swa[PF][WPT];
    auto load_chunk = [&](int ch, u32x4 (&st)[NP], float (&sw)[WPT]) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {                   // this wavefront's 16 rows (SPLIT: the work-group's), 8 pieces of 16 bytes each
            const int pid = SPLIT ? tid : i * 64 + lane, row = row0 + pid / 8, byte = ch * 128 + pid % 8 * 16;
            const u32x4 z = {0u, 0u, 0u, 0u};
            st[i] = (row < rows && byte < row_bytes) ? *(const u32x4*)(gbase + (size_t)row * row_bytes + byte) : z;
        }
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const int e = i * NTHR + tid;
            sw[i] = (e < RC * DG && ch * RC + e / DG < dm) ? wg[(size_t)ch * RC * DG + e] : 0.f;
        }
    };
    acc_t acc[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = acc_t{};

#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (p < nchunk) load_chunk(p, sta[p], swa[p]);
    for (int ch0 = 0; ch0 < nchunk; ch0 += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
        const int ch = ch0 + p;
        if (ch >= nchunk) break;                         // uniform over the work-group
        u32x4 (&st)[NP] = sta[p];
        float (&sw)[WPT] = swa[p];
        char* abuf = s_a + (ch & 1) * (TB * A_ROW);
        w_t* wbuf = s_w + (ch & 1) * (RC * WP);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int pid = SPLIT ? tid : i * 64 + lane;
            if (SPLIT && tid >= 128) break;              // (uniform over a wavefront)
            uint32_t* dst = (uint32_t*)(abuf + (row0 + pid / 8) * A_ROW) + pid % 8;
            const u32x4 v = st[i];
            if constexpr (sizeof(T) == 4) {              // components 4c .. 4c+3: step c of the four parts
                dst[0] = v[0]; dst[8] = v[1]; dst[16] = v[2]; dst[24] = v[3];
            } else {                                     // components 8c .. 8c+7: steps 2c and 2c + 1
                dst[0] = (v[0] & 0xffffu) | (v[2] << 16);
                dst[8] = (v[0] >> 16) | (v[2] & 0xffff0000u);
                dst[16] = (v[1] & 0xffffu) | (v[3] << 16);
                dst[24] = (v[1] >> 16) | (v[3] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const int e = i * NTHR + tid;
            if (e < RC * DG) wbuf[(e / DG) * WP + e % DG] = (w_t)sw[i];
        }
        __syncthreads();               // also orders these writes after every wave's reads two chunks ago
        if (ch + PF < nchunk) load_chunk(ch + PF, st, sw);
        const u32x4* ar = (const u32x4*)(abuf + (row0 + (lane & 15)) * A_ROW + (lane >> 4) * 32);
        const u32x4 a0 = ar[0], a1 = ar[1];
        const w_t* wr = wbuf + (lane >> 4) * WP + col0 + (lane & LC);
        const int steps = min(RC, dm - ch * RC) / 4;     // dm is a multiple of 8
        auto a_of = [&](int i) -> double {
            double a;
            if constexpr (sizeof(T) == 4) {
                a = (double)__uint_as_float(i < 4 ? a0[i % 4] : a1[i % 4]);
            } else {
                const uint32_t w2 = (i < 8) ? a0[(i / 2) % 4] : a1[(i / 2) % 4];
                if constexpr (std::is_same<T, f16_bits>::value)
                    a = (double)f16_bits_to_f32((uint16_t)(i % 2 ? w2 >> 16 : w2 & 0xffffu));
                else
                    a = (double)__uint_as_float(i % 2 ? w2 & 0xffff0000u : w2 << 16);
            }
            return a;
        };
        auto step = [&](double a, const double (&w)[CB]) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                if constexpr (SMALL) acc[cb] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, w[cb], acc[cb], 0, 0, 0);
                else acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, w[cb], acc[cb], 0, 0, 0);
            }
        };
        // a full chunk without a branch per step, BATCH steps at a time: their operands first, then the products back to back
        // (32768 tokens, d_g = 16: 108 us one by one, 104 with 4, 106 with 8, 105 with 16; 131072: 364 / 353 / 361 / 413, whose
        // registers leave fewer wavefronts)
        constexpr int BATCH = DG < 16 ? 2 : 4;
        static_assert((RC / 4) % BATCH == 0, "whole batches");
        if (steps == RC / 4) {
#pragma unroll
            for (int i0 = 0; i0 < RC / 4; i0 += BATCH) {
                double w[BATCH][CB], av[BATCH];
#pragma unroll
                for (int i = 0; i < BATCH; ++i)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) w[i][cb] = (double)wr[(i0 + i) * 4 * WP + cb * (LC + 1)];
#pragma unroll
                for (int i = 0; i < BATCH; ++i) av[i] = a_of(i0 + i);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < BATCH; ++i) step(av[i], w[i]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < RC / 4; ++i)
                if (i < steps) {
                    double w[CB];
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) w[cb] = (double)wr[i * 4 * WP + cb * (LC + 1)];
                    step(a_of(i), w);
                }
        }
    }
    }

    // z of the tokens -> LDS, then S[i,g] = sum_j z_j C[g][j] in index order (products rounded, then added)
    __syncthreads();                                     // the staging buffers are free
    double* s_z = (double*)s_dyn;
    double* s_s = s_z + TB * (DG + 1);
    const int KS = K | 1;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        if constexpr (SMALL) {
            s_z[(row0 + (lane & 12) + (lane >> 4)) * (DG + 1) + col0 + cb * 4 + (lane & 3)] = acc[cb];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) s_z[(wave * 16 + 4 * r + (lane >> 4)) * (DG + 1) + cb * 16 + (lane & 15)] = acc[cb][r];
        }
    }
    __syncthreads();
    double mymax = -INFINITY;
    const int tok = tid % TB;
    for (int g = tid / TB; g < K; g += NTHR / TB) {
        double s = 0.0;
#pragma unroll 4
        for (int j = 0; j < DG; ++j) s = __dadd_rn(s, __dmul_rn(s_z[tok * (DG + 1) + j], (double)cent[(size_t)g * DG + j]));
        s_s[tok * KS + g] = s;
        if (tok < rows) mymax = fmax(mymax, s);
    }
    mymax = wave_max(mymax);
    if (lane == 0) s_wmax[wave] = mymax;
    __syncthreads();
    if (tid == 0) {
        double m = s_wmax[0];
        for (int w = 1; w < NW; ++w) m = fmax(m, s_wmax[w]);
        ((double*)(ws + R.off_maxpart))[(size_t)b * R.nproj + blockIdx.x] = m;
    }
    if constexpr (CLEAR) {
        unsigned long long* slots = sink_slots(R, ws, b);
        for (int i = blockIdx.x * NTHR + tid; i < 3 * R.nround * K; i += gridDim.x * NTHR) slots[i] = SINK_EMPTY;
    }
    if (tid < rows) {
        const size_t tg = (size_t)b * n + tok0 + tid;
        double* mine = s_s + tid * KS;
        if (R.iters == 0) {
            for (int g = 0; g < K; ++g) mine[g] = mine[g] / R.tau;
            uint32_t m = 0;
            for (int g = 0; g < K; ++g) {
                const double sg = mine[g];
                int beaten = 0;
                for (int o = 0; o < K; ++o) {
                    const double so = mine[o];
                    beaten += (o != g && (so > sg || (so == sg && o < g))) ? 1 : 0;
                }
                if (beaten < R.topk) m |= (1u << g);
            }
            if (__popc(m) != R.topk) m = (R.topk == 32) ? 0xffffffffu : ((1u << R.topk) - 1u);   // NaN scores
            masks[tg] = m;
            if (soft) for (int g = 0; g < K; ++g) soft[tg * K + g] = mine[g];
        } else {
            double* Srow = (double*)(ws + R.off_S) + tg * K;
            for (int g = 0; g < K; ++g) Srow[g] = mine[g];
        }
    }
}

// ---------------------------------------------------------------- Sinkhorn passes
// pass 0: the largest score of the sequence (the shift that keeps exp finite; the first column step divides it out
// again), E = exp((S - max)/tau) in place, column partial sums of E.
// pass t = 1..N: v from the partial sums of pass t-1, u per row, partial sums of u E (or, on pass N, the outputs).
// A pass is latency (1 MB at 32768 tokens, K = 4): the rows are on their way while the sums are folded, and where K fills KP
// (FULL) a row is loaded in 16-byte pieces instead of one guarded double after the other: 212.7 -> 209 us in all for ten rounds of 32768 tokens.
template <int KP, bool FULL>
__global__ __launch_bounds__(256) void sinkhorn_pass_kernel(RouteLayout R, int pass, char* __restrict__ ws,
                                                            uint32_t* __restrict__ masks, double* __restrict__ soft)
{
    __shared__ double s_v[KP];
    __shared__ double s_part[4][KP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int blk = blockIdx.x, b = blockIdx.y;
    const int n = R.n, K = R.K;
    double* E = (double*)(ws + R.off_S) + (size_t)b * n * K;
    const double* prev = (const double*)(ws + R.off_colpart) + ((size_t)((pass + 1) & 1) * R.B + b) * R.nsink * KP;
    double* mine = (double*)(ws + R.off_colpart) + (((size_t)(pass & 1) * R.B + b) * R.nsink + blk) * KP;
    const bool last = pass == R.iters;
    const int t_beg = blk * R.sink_tokens + tid, t_end = min(n, (blk + 1) * R.sink_tokens);
    double r[KP];                                 // a row of E (pass 0: of S)
    auto load_row = [&](int i) {
        const double* src = E + (size_t)i * K;
        if constexpr (FULL) {
            __builtin_memcpy(r, __builtin_assume_aligned(src, KP * 8 < 16 ? KP * 8 : 16), sizeof(r));
        } else {
#pragma unroll
            for (int g = 0; g < KP; ++g) r[g] = g < K ? src[g] : 0.0;
        }
    };
    if (t_beg < t_end) load_row(t_beg);

    if (pass > 0) {
        for (int g = wave; g < K; g += 4) {
            double s = 0.0;
            for (int i = lane; i < R.nsink; i += 64) s = __dadd_rn(s, prev[(size_t)i * KP + g]);
            s = wave_sum(s);
            if (lane == 0) s_v[g] = 1.0 / s;
        }
        __syncthreads();
    }
    // pass 0: the largest score of the sequence from the projection's work-groups, folded by every work-group
    double smax = 0.0;
    if (pass == 0) {
        __shared__ double s_m[4];
        const double* mp = (const double*)(ws + R.off_maxpart) + (size_t)b * R.nproj;
        double m = -INFINITY;
        for (int i = tid; i < R.nproj; i += 256) m = fmax(m, mp[i]);
        m = wave_max(m);
        if (lane == 0) s_m[wave] = m;
        __syncthreads();
        smax = fmax(fmax(s_m[0], s_m[1]), fmax(s_m[2], s_m[3]));
    }
    double v[KP], cs[KP];
#pragma unroll
    for (int g = 0; g < KP; ++g) {
        v[g] = (pass > 0 && g < K) ? s_v[g] : 1.0;
        cs[g] = 0.0;
    }
    for (int i = t_beg; i < t_end; i += 256) {
        double e[KP];
        double* row = E + (size_t)i * K;
        if (i != t_beg) load_row(i);
        if (pass == 0) {
#pragma unroll
            for (int g = 0; g < KP; ++g)
                if (g < K) {
                    e[g] = exp((r[g] - smax) / R.tau);
                    row[g] = e[g];
                    cs[g] = __dadd_rn(cs[g], e[g]);
                }
            continue;
        }
        double rs = 0.0;
#pragma unroll
        for (int g = 0; g < KP; ++g) {
            e[g] = (g < K) ? __dmul_rn(r[g], v[g]) : 0.0;
            rs = __dadd_rn(rs, e[g]);
        }
        const double u = 1.0 / rs;
        if (!last) {
#pragma unroll
            for (int g = 0; g < KP; ++g)
                if (g < K) cs[g] = __dadd_rn(cs[g], __dmul_rn(u, r[g]));
        } else {
            const size_t tok = (size_t)b * n + i;
#pragma unroll
            for (int g = 0; g < KP; ++g) e[g] = __dmul_rn(e[g], u);
            masks[tok] = topk_mask<KP>(e, K, R.topk);
            if (soft) {
#pragma unroll
                for (int g = 0; g < KP; ++g)
                    if (g < K) soft[tok * K + g] = e[g];
            }
        }
    }
    if (last && pass > 0) return;
    {
        const double s = wave_sum_columns<KP>(cs, lane);
        if ((lane & (64 / KP - 1)) == 0) s_part[wave][wave_column<KP>(lane)] = s;
    }
    __syncthreads();
    if (tid < K) mine[tid] = __dadd_rn(__dadd_rn(s_part[0][tid], s_part[1][tid]), __dadd_rn(s_part[2][tid], s_part[3][tid]));
}

// All rounds in one launch: the rows of E stay in registers (R per thread), a round is their scaling, the work-group's column sums and
// one exchange of them.  Work-group w leaves its sums of round p in slot p % 3 and takes those of the others as they come (8 bytes
// a sum, whole: no flag beside it); they are added in the order of the work-groups, so the result does not depend on who came first.
// Once it has everybody's sums of round p, everybody is done with those of round p - 1, and it empties its slot of that round,
// before it leaves its sums of round p + 1: whoever sees those sees the empty slot.
// Nothing makes the work-groups of a launch resident together (a device of fewer units, a stream that is kept to some of them, other
// launches that wait), so none relies on it: one that has looked `looks` times for a sum goes on alone.  It takes the rows of every
// work-group in turn and adds up their sums itself, in the same order, and leaves no more of its own, so that the others do the same a
// round later at the latest; only its own rows are its to write.  Nobody leaves sums of round p + 1 without having seen all of round
// p, so a slot never holds those of a later round than the one that is looked for.  The result is the same bits either way, and
// every wait ends: with the sum, or as the last wait of its work-group.  Alone, a round takes 0.02 ms for 4096 tokens of 4 groups, 0.13
// for 32768, 0.7 for 131072 of 8, 1.0 for 32768 of 32.
template <int KP, int R>
__global__ __launch_bounds__(256, sink_resident(KP, R)) void sinkhorn_rounds_kernel(RouteLayout L, int tokens, int looks, char* __restrict__ ws,
                                                                                    uint32_t* __restrict__ masks, double* __restrict__ soft)
{
    constexpr int EX = 64 * 32;                   // sums of a round at most
    __shared__ double s_part[4][KP], s_v[KP], s_m[4];
    __shared__ double s_ex[EX];
    __shared__ int s_late;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int blk = blockIdx.x, nwg = gridDim.x, b = blockIdx.y;
    const int n = L.n, K = L.K;
    const double* S = (const double*)(ws + L.off_S) + (size_t)b * n * K;
    unsigned long long* slots = sink_slots(L, ws, b);
    double r[R][KP];
    auto load = [&](int of) {                     // the scores of work-group `of`
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int i = min(of * tokens + t * 256 + tid, n - 1);
            if (K == KP) {
                const double* src = S + (size_t)i * KP;
                __builtin_memcpy(r[t], __builtin_assume_aligned(src, 16), sizeof(r[t]));
            } else {
#pragma unroll
                for (int g = 0; g < KP; ++g) r[t][g] = g < K ? S[(size_t)i * K + g] : 0.0;
            }
        }
    };
    auto there = [&](int of, int t) { return of * tokens + t * 256 + tid < min(n, (of + 1) * tokens); };
    load(blk);
    double smax;
    {
        const double* mp = (const double*)(ws + L.off_maxpart) + (size_t)b * L.nproj;
        double m = -INFINITY;
        for (int i = tid; i < L.nproj; i += 256) m = fmax(m, mp[i]);
        m = wave_max(m);
        if (lane == 0) s_m[wave] = m;
        if (tid == 0) s_late = 0;
        __syncthreads();
        smax = fmax(fmax(s_m[0], s_m[1]), fmax(s_m[2], s_m[3]));
    }
    auto expand = [&](int of) {                   // to rows of E
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
            for (int g = 0; g < KP; ++g) r[t][g] = there(of, t) && g < K ? exp((r[t][g] - smax) / L.tau) : 0.0;
    };
    expand(blk);
    double v[KP];
#pragma unroll
    for (int g = 0; g < KP; ++g) v[g] = 1.0;
    bool alone = false;                           // (uniform over the work-group)
    for (int p = 0; p < L.iters; ++p) {
        unsigned long long* at = slots + (size_t)(p % 3) * nwg * K;
        int of = alone ? 0 : blk;
        for (;;) {
            if (alone) {
                load(of);
                expand(of);
            }
            // column sums of the work-group
            double cs[KP];
#pragma unroll
            for (int g = 0; g < KP; ++g) cs[g] = 0.0;
#pragma unroll
            for (int t = 0; t < R; ++t) {
                if (!there(of, t)) continue;
                double u = 1.0;
                if (p > 0) {
                    double rs = 0.0;
#pragma unroll
                    for (int g = 0; g < KP; ++g) rs = __dadd_rn(rs, g < K ? __dmul_rn(r[t][g], v[g]) : 0.0);
                    u = 1.0 / rs;
                }
#pragma unroll
                for (int g = 0; g < KP; ++g)
                    if (g < K) cs[g] = __dadd_rn(cs[g], __dmul_rn(u, r[t][g]));
            }
            const double ws_sum = wave_sum_columns<KP>(cs, lane);
            if ((lane & (64 / KP - 1)) == 0) s_part[wave][wave_column<KP>(lane)] = ws_sum;
            __syncthreads();
            double mine = 0.0;
            if (tid < K) mine = __dadd_rn(__dadd_rn(s_part[0][tid], s_part[1][tid]), __dadd_rn(s_part[2][tid], s_part[3][tid]));
            if (nwg == 1) {
                if (tid < K) s_v[tid] = 1.0 / mine;
                break;
            }
            if (alone) {
                if (tid < K) s_ex[of * K + tid] = mine;
                __syncthreads();                  // (s_part is written again)
                if (++of < nwg) continue;
                break;
            }
            if (tid < K) {
                unsigned long long bits = __builtin_bit_cast(unsigned long long, mine);
                if (bits == SINK_EMPTY) bits = 0x7ff8000000000000ull;    // another NaN
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the slot of two rounds ago is empty
                __hip_atomic_store(at + blk * K + tid, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            for (int i = tid; i < nwg * K; i += 256) {
                unsigned long long x = SINK_EMPTY;
                for (int look = 0; look < looks; ++look) {
                    x = __hip_atomic_load(at + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (x != SINK_EMPTY) break;
                }
                if (x == SINK_EMPTY) {
                    s_late = 1;
                    break;
                }
                s_ex[i] = __builtin_bit_cast(double, x);
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(s_late) == 0) {
                if (p > 0 && tid < K)
                    __hip_atomic_store(slots + (size_t)((p + 2) % 3) * nwg * K + blk * K + tid, SINK_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            alone = true;
            of = 0;
        }
        if (nwg > 1) {
            for (int g = wave; g < K; g += 4) {
                const double sum = wave_sum(lane < nwg ? s_ex[lane * K + g] : 0.0);
                if (lane == 0) s_v[g] = 1.0 / sum;
            }
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < KP; ++g) v[g] = g < K ? s_v[g] : 1.0;
    }
    if (alone) {
        load(blk);
        expand(blk);
    }
#pragma unroll
    for (int t = 0; t < R; ++t) {
        if (!there(blk, t)) continue;
        double e[KP], rs = 0.0;
#pragma unroll
        for (int g = 0; g < KP; ++g) {
            e[g] = g < K ? __dmul_rn(r[t][g], v[g]) : 0.0;
            rs = __dadd_rn(rs, e[g]);
        }
        const double u = 1.0 / rs;
        const size_t tok = (size_t)b * n + blk * tokens + t * 256 + tid;
#pragma unroll
        for (int g = 0; g < KP; ++g) e[g] = __dmul_rn(e[g], u);
        masks[tok] = topk_mask<KP>(e, K, L.topk);
        if (soft) {
#pragma unroll
            for (int g = 0; g < KP; ++g)
                if (g < K) soft[tok * K + g] = e[g];
        }
    }
}

template <typename T>
hipError_t launch_project(const RouteLayout& R, const void* hidden, const float* wg, const float* cent, char* ws,
                          uint32_t* masks, double* soft, bool split, hipStream_t st)
{
    const int tb = split ? 16 : route_tokens_per_group(R.B, R.n, R.dg), nw = tb == 128 ? 8 : 4;
    dim3 grid(R.nproj, R.B);
    const int rc = 128 / (int)sizeof(T);
    const size_t stage = 2 * ((size_t)tb * A_ROW + (size_t)rc * route_wp(R.dg) * (R.dg <= 16 ? 8 : 4));
    const size_t tail = (size_t)tb * (R.dg + 1 + (R.K | 1)) * sizeof(double);
    const size_t lds = stage > tail ? stage : tail;      // at most 53 KB (8 wavefronts, d_g <= 16) or 59 KB (4, d_g = 64, 16-bit rows)
#define FOCUS_PROJ_C(DG, NW, SPLIT, CLEAR)                                                                   \
    hipLaunchKernelGGL((route_project_kernel<T, DG, NW, SPLIT, CLEAR>), grid, dim3(64 * NW), lds, st, R, (const T*)hidden, wg, \
                       cent, ws, masks, soft)
    // (one work-group exchanges nothing, and a short sequence has no space for its slots)
#define FOCUS_PROJ(DG, NW, SPLIT) do { if (R.nround > 1) FOCUS_PROJ_C(DG, NW, SPLIT, true); else FOCUS_PROJ_C(DG, NW, SPLIT, false); } while (0)
    switch (R.dg) {
        case 4: if (nw == 8) FOCUS_PROJ(4, 8, false); else FOCUS_PROJ(4, 4, false); break;
        case 8: if (nw == 8) FOCUS_PROJ(8, 8, false); else FOCUS_PROJ(8, 4, false); break;
        case 16: if (split) FOCUS_PROJ(16, 4, true); else if (nw == 8) FOCUS_PROJ(16, 8, false); else FOCUS_PROJ(16, 4, false); break;
        case 32: FOCUS_PROJ(32, 4, false); break;
        default: FOCUS_PROJ(64, 4, false); break;
    }
#undef FOCUS_PROJ
#undef FOCUS_PROJ_C
    return hipGetLastError();
}

}  // namespace

hipError_t launch_route(const RouteLayout& layout, const void* hidden, const float* wg, const float* cent, char* ws,
                        uint32_t* masks, double* soft, hipStream_t st)
{
    hipError_t e;
    RouteLayout R = layout;
    const char* env = getenv("FOCUS_SINKHORN_LOOKS");        // (tests, measurements; negative: a launch per round)
    const int looks = env ? atoi(env) : SINK_LOOKS;
    if (R.iters > 0 && looks >= 0) {
        int dev = 0, units = 0;
        if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
        if ((e = hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
        R.nround = sink_groups(R, units);
    }
    const bool split = R.dg == 16 && (long long)R.B * R.n <= ((R.iters == 0 && R.K > 16) ? 4096 : 8192) && (R.iters == 0 || R.nround > 0);
    if (split) {       // a largest score for every 16 tokens: behind the sums of the rounds, which take at most 48 of 64 words a sort block
        R.nproj = (R.n + 15) / 16;
        R.off_maxpart = R.off_colpart + (size_t)48 * R.B * R.nsink * 8;
    }
    if (R.dtype == 0) e = launch_project<float>(R, hidden, wg, cent, ws, masks, soft, split, st);
    else if (R.dtype == 2) e = launch_project<f16_bits>(R, hidden, wg, cent, ws, masks, soft, split, st);
    else e = launch_project<uint16_t>(R, hidden, wg, cent, ws, masks, soft, split, st);
    if (e != hipSuccess) return e;
    if (R.iters == 0) return hipSuccess;
    if (R.nround > 0) {
        const int tokens = (R.n + R.nround - 1) / R.nround, rows = sink_rows(sink_kp(R.K), tokens);
        dim3 grid(R.nround, R.B);
#define FOCUS_ROUNDS(KP_, R_) hipLaunchKernelGGL((sinkhorn_rounds_kernel<KP_, R_>), grid, dim3(256), 0, st, R, tokens, looks, ws, masks, soft)
        if (R.K <= 4) { if (rows == 2) FOCUS_ROUNDS(4, 2); else if (rows == 4) FOCUS_ROUNDS(4, 4); else if (rows == 8) FOCUS_ROUNDS(4, 8); else FOCUS_ROUNDS(4, 16); }
        else if (R.K <= 8) { if (rows == 2) FOCUS_ROUNDS(8, 2); else if (rows == 4) FOCUS_ROUNDS(8, 4); else FOCUS_ROUNDS(8, 8); }
        else if (R.K <= 16) { if (rows == 2) FOCUS_ROUNDS(16, 2); else FOCUS_ROUNDS(16, 4); }
        else FOCUS_ROUNDS(32, 2);
#undef FOCUS_ROUNDS
        return hipGetLastError();
    }
    dim3 grid(R.nsink, R.B);
    for (int pass = 0; pass <= R.iters; ++pass) {
#define FOCUS_SINK(KP_)                                                                                                   \
    { if (R.K == KP_) hipLaunchKernelGGL((sinkhorn_pass_kernel<KP_, true>), grid, dim3(256), 0, st, R, pass, ws, masks, soft);    \
      else hipLaunchKernelGGL((sinkhorn_pass_kernel<KP_, false>), grid, dim3(256), 0, st, R, pass, ws, masks, soft); }
        if (R.K <= 4) FOCUS_SINK(4)
        else if (R.K <= 8) FOCUS_SINK(8)
        else if (R.K <= 16) FOCUS_SINK(16)
        else FOCUS_SINK(32)
#undef FOCUS_SINK
    }
    return hipGetLastError();
}

}  // namespace focus
