// focus_assign: centroid scoring, top-k membership, bucketing by group and by
// membership class (Sec. 2 Eq. 1 in per-head dot-product form; Sec. 2
// "Efficiency at inference"; the stable sort by group of App. D done as a
// counting sort).
//
// Three launches per focus_assign call on class layouts, one or two on masked ones (end of this comment), the work item a
// (sort block of SB positions, batch*head) pair:
//   score        streams q (or k) once, scores every token against the K centroids of its KV
//                head in fp64 (products are exact in fp64, added in index order,
//                so the result is reproducible bit for bit), keeps the top-k
//                groups, writes the membership mask, the class id and the
//                per-block histograms of classes and groups;
//   scan_plan    one work-group per (batch, head) row: exclusive scan of the
//                row's histograms over the sort blocks, then class offsets
//                (padded to tile multiples), group list offsets, the class ->
//                group-mask table and the job list of query tiles;
//   scatter      stable ranks inside a block by wavefront ballot + popcount,
//                coalesced 4-byte writes of the class-ordered position arrays
//                and of the per-group index lists, the pads of those arrays, and
//                (key rows, 16-bit types) the class-ordered copy of the key rows
//                with the largest squared key norm of the head.
// Memberships given per token (focus_assign_tokens) take token_classes in place
// of score.  Layouts without classes (masked) leave the scan out where the scatter launch can add up
// the histograms itself, and short rows of theirs are bucketed in one launch, a work-group per row.
#include "focus_internal.h"
#include "focus_score.h"
#include <hip/hip_bf16.h>
#include <algorithm>
#include <type_traits>

namespace focus {

namespace {

// Pascal's triangle up to C(32, .), built at compile time: the class of a token is the colex rank of
// its membership set, a sum of binomials.
struct BinomTable { uint32_t v[33 * 33]; };
constexpr BinomTable make_binom_table()
{
    BinomTable t{};
    for (int a = 0; a <= 32; ++a) {
        for (int b = 0; b <= 32; ++b) {
            uint32_t x = 0;
            if (b == 0 || b == a) x = (b <= a) ? 1u : 0u;
            else if (b < a) x = t.v[(a - 1) * 33 + b - 1] + t.v[(a - 1) * 33 + b];
            t.v[a * 33 + b] = x;
        }
    }
    return t;
}
__device__ __constant__ BinomTable g_binom = make_binom_table();

// The kernels of the bucketing serve the query side, the key side, or both in one launch (which = 1, 0, -1):
// with both, the rows [0, B*Hq) of the launch are query (batch, head) pairs and the B*Hkv after them key pairs.
constexpr int MAX_GRID_ROWS = 65535;
__device__ inline int side_of_row(const Layout& L, int which, unsigned row) { return which < 0 ? (int)(row < (unsigned)(L.B * L.Hq)) : which; }
__device__ inline int row_in_side(const Layout& L, int which, unsigned row)
{
    return (which < 0 && row >= (unsigned)(L.B * L.Hq)) ? (int)row - L.B * L.Hq : (int)row;
}

// class of a membership: the colex rank of the set among all topk-subsets (coarse: of its set of super-groups)
__device__ inline int token_class(const Layout& L, uint32_t mask)
{
    if (L.coarse) return class_of_mask(mask, 0, 1, L.S);
    int cls = 0;
    if (!L.dense) {
        int j = 0;
        for (int g = 0; g < L.K; ++g)
            if ((mask >> g) & 1u) { ++j; cls += (int)g_binom.v[g * 33 + j]; }
    }
    return cls;
}

// ---------------------------------------------------------------- scan over sort blocks + per-row plan
// One (batch, head) row, all NTHREADS threads of a work-group: exclusive scan of every histogram column over
// the sort blocks (in place, total in row nblk), then class offsets (padded to tile multiples), group list
// offsets, the class -> group-mask table (first query row) and the job list of the query tiles.
// The histograms pass through LDS a chunk of sort blocks at a time.  tmp: tmp_ints >= SCAN_PLAN_FIXED_INTS + NC + K ints of LDS.

constexpr int SCAN_THREADS = 1024;                                   // threads of the scan + plan work-group
constexpr int SCAN_PLAN_FIXED_INTS = SCAN_THREADS + 2 * MAX_CLASSES + 40;   // s_part, s_tot, s_nt, s_total
constexpr int SCAN_PLAN_TMP_INTS = 9216;                             // 36 KB of LDS
static_assert(SCAN_PLAN_TMP_INTS >= SCAN_PLAN_FIXED_INTS + MAX_CLASSES + 32, "room for at least one sort block");

template <int NTHREADS>
__device__ inline void scan_and_plan_row(const Layout& L, int is_query, int bh, char* __restrict__ ws, int* tmp, int tmp_ints)
{
    const int tid = threadIdx.x;
    const int NC = L.NC, K = L.K, nblk = L.nblk;
    int* s_part = tmp;                          // [NTHREADS] partial sums of the scan
    int* s_tot = tmp + NTHREADS;                // [NC + K] running column totals
    int* s_nt = s_tot + MAX_CLASSES + 32;       // [NC] query tiles per class
    int* s_total = s_nt + MAX_CLASSES;          // [1]
    int* stage = tmp + SCAN_PLAN_FIXED_INTS;    // histograms of a chunk of sort blocks, [blocks][NC + K]
    int* bc_base = (int*)(ws + (is_query ? L.off_qbc : L.off_kbc)) + (size_t)bh * (nblk + 1) * NC;
    int* bg_base = (int*)(ws + (is_query ? L.off_qbg : L.off_kbg)) + (size_t)bh * (nblk + 1) * K;
    const int ncol = NC + K;
    const int cb = max(1, min(nblk, (tmp_ints - SCAN_PLAN_FIXED_INTS) / ncol));   // sort blocks per chunk
    const int cpp = min(ncol, NTHREADS);        // columns per pass
    const int P = NTHREADS / cpp;               // threads per column: each scans a run of the chunk's blocks
    for (int c = tid; c < ncol; c += NTHREADS) s_tot[c] = 0;
    for (int b0 = 0; b0 < nblk; b0 += cb) {
        const int nb = min(cb, nblk - b0);
        const int ne = nb * ncol;
        __syncthreads();                        // the previous chunk's stage is no longer read; s_tot is set
        // the chunk into LDS, eight independent loads in flight per thread
        for (int e0 = 0; e0 < ne; e0 += 8 * NTHREADS) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = e0 + i * NTHREADS + tid;
                v[i] = 0;
                if (e < ne) {
                    const int b = b0 + e / ncol, c = e % ncol;
                    v[i] = c < NC ? bc_base[(size_t)b * NC + c] : bg_base[(size_t)b * K + (c - NC)];
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = e0 + i * NTHREADS + tid;
                if (e < ne) stage[e] = v[i];
            }
        }
        __syncthreads();
        const int run = (nb + P - 1) / P;
        for (int col0 = 0; col0 < ncol; col0 += cpp) {
            const int cl = tid % cpp, part = tid / cpp, col = col0 + cl;
            const bool active = part < P && col < ncol;
            const int r_lo = min(nb, part * run), r_hi = min(nb, r_lo + run);
            int sum = 0;
            if (active)
                for (int r = r_lo; r < r_hi; ++r) sum += stage[r * ncol + col];
            s_part[tid] = active ? sum : 0;
            __syncthreads();
            int running = 0;
            if (active) {
                running = s_tot[col];
                for (int p2 = 0; p2 < part; ++p2) running += s_part[p2 * cpp + cl];
                int* base = col < NC ? bc_base + col : bg_base + (col - NC);
                const int stride = col < NC ? NC : K;
                for (int r = r_lo; r < r_hi; ++r) {
                    base[(size_t)(b0 + r) * stride] = running;
                    running += stage[r * ncol + col];
                }
            }
            __syncthreads();                    // every reader of s_tot[col] and s_part is done
            if (active && part == P - 1) s_tot[col] = running;
        }
    }
    __syncthreads();
    for (int c = tid; c < ncol; c += NTHREADS) {    // totals in row nblk
        if (c < NC) bc_base[(size_t)nblk * NC + c] = s_tot[c];
        else bg_base[(size_t)nblk * K + (c - NC)] = s_tot[c];
    }

    int* cc = (int*)(ws + (is_query ? L.off_qcc : L.off_kcc)) + (size_t)bh * NC;
    int* co = (int*)(ws + (is_query ? L.off_qco : L.off_kco)) + (size_t)bh * (NC + 1);
    int* gc = (int*)(ws + (is_query ? L.off_qgc : L.off_kgc)) + (size_t)bh * K;
    int* go = (int*)(ws + (is_query ? L.off_qgo : L.off_kgo)) + (size_t)bh * (K + 1);
    const int pad = is_query ? L.BQ : KT;
    for (int c = tid; c < NC; c += NTHREADS) {
        const int v = s_tot[c];
        s_nt[c] = (v + L.BQ - 1) / L.BQ;
        cc[c] = v;
    }
    if (tid < K) gc[tid] = s_tot[NC + tid];
    __syncthreads();
    if (tid == 0) {
        int off = 0, tot = 0;
        for (int c = 0; c < NC; ++c) {
            co[c] = off;
            off += (s_tot[c] + pad - 1) / pad * pad;
            tot += s_nt[c];
        }
        co[NC] = off;
        *s_total = tot;
        int goff = 0;
        for (int g = 0; g < K; ++g) { go[g] = goff; goff += s_tot[NC + g]; }
        go[K] = goff;
    }
    // class -> group mask (written once, by the first query head)
    if (is_query && bh == 0) {
        uint32_t* clsmask = (uint32_t*)(ws + L.off_clsmask);
        for (int c = tid; c < NC; c += NTHREADS) {
            uint32_t m = 0;
            if (L.dense) {
                m = 0xffffffffu;
            } else {
                // exact classes: topk-subsets of the K groups in colex order; coarse classes: sets of
                // 1..topk of the S super-groups, by size, then colex
                uint32_t r = (uint32_t)c;
                int size = L.topk, top = K - 1;
                if (L.coarse) {
                    size = 1;
                    while (r >= binom_u32(L.S, size)) { r -= binom_u32(L.S, size); ++size; }
                    top = L.S - 1;
                }
                int g = top;
                for (int j = size; j >= 1; --j) {
                    while (binom_u32(g, j) > r) --g;      // largest g with C(g,j) <= r
                    m |= (1u << g);
                    r -= binom_u32(g, j);
                    --g;
                }
            }
            clsmask[c] = m;
        }
    }
    __syncthreads();
    if (!is_query) return;
    // Job list = the order in which the work-groups of the attention launch are dispatched.
    //  * Long sequences (256-row tiles, n >= LONG_N: a head's K and V no longer sit in the L2 of its XCD), class-major:
    //    the tiles of class 0 from its last (longest key walk) to its first, then class 1, ...  The work-groups
    //    resident at any moment are then neighbouring tiles of ONE class: they walk the same key classes from the
    //    same first tile at the same pace and share every K/V tile they fetch (at 1M tokens 1 TB is fetched from
    //    memory per launch instead of 20 TB).  The list still ends with short tiles, as the tail of the launch needs.
    //  * Otherwise slot-major: slot s = how many tiles from the end of its class a tile is; every class's last
    //    (longest-prefix) tile first.  K and V mostly stay in L2 at these lengths, and the mix of classes among the
    //    resident work-groups keeps them from asking for the same lines in the same cycles (class-major measured
    //    6 to 10 % slower at 131072 tokens with 8 groups).
    int* jobs = (int*)(ws + L.off_jobs) + (size_t)bh * L.NT;
    const int total = *s_total;
    for (int j = total + tid; j < L.NT; j += NTHREADS) jobs[j] = -1;
    for (int u = tid; u < total; u += NTHREADS) {                 // one thread per tile, tiles counted class by class
        int c = 0, first = 0;
        while (u >= first + s_nt[c]) { first += s_nt[c]; ++c; }
        const int ntc = s_nt[c], t = u - first;
        const int s = ntc - 1 - t;
        int j = first + s;
        if (!L.class_major) {
            j = 0;
            for (int c2 = 0; c2 < NC; ++c2) {
                j += min(s_nt[c2], s);
                if (c2 < c && s_nt[c2] > s) ++j;
            }
        }
        jobs[j] = (int)(((unsigned)c << 24) | (unsigned)t);       // t < 2^17: never the unused marker -1
    }
    __syncthreads();                                              // tmp may be reused by the caller
}

// scan + plan as a launch of its own (memberships given per token): one work-group per row
__global__ __launch_bounds__(SCAN_THREADS) void scan_plan_kernel(Layout L, char* __restrict__ ws)
{
    __shared__ int s_tmp[SCAN_PLAN_TMP_INTS];
    const int is_query = side_of_row(L, -1, blockIdx.x);
    const int bh = row_in_side(L, -1, blockIdx.x);
    scan_and_plan_row<SCAN_THREADS>(L, is_query, bh, ws, s_tmp, SCAN_PLAN_TMP_INTS);
}

// ---------------------------------------------------------------- score + top-k
// Memberships of one sort block on the fp64 matrix cores (focus_score.h), its group histogram and, on layouts with classes
// (CLS), the class of every token and the class histogram.  norms: the largest squared key norm of the block goes into the
// block's own slot (layouts whose keys are read in place by the tiled kernel).
template <typename T, int KM, bool CLS>
__global__ __launch_bounds__(SB, score_waves<T>(KM)) void score_kernel(Layout L, HeadMap hm, const T* __restrict__ xq, const T* __restrict__ xk,
                                                   const float* __restrict__ cents, int which, int norms, char* __restrict__ ws)
{
    __shared__ __align__(16) char s_a[4][score_lds(score_chunk<T>(KM))];
    __shared__ int s_h[4][32];
    __shared__ int s_hist_c[CLS ? MAX_CLASSES : 1];
    extern __shared__ __align__(16) char s_cent[];
    score_cent_t<KM>* s_c = (score_cent_t<KM>*)s_cent;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x, K = L.K, n = L.n;
    const int is_query = side_of_row(L, which, blockIdx.y);
    const int bh = row_in_side(L, which, blockIdx.y);
    const int H = is_query ? L.Hq : L.Hkv, h = bh % H, hk = is_query ? hm.kv[h] : h;
    const long long* xs = is_query ? L.qs : L.ks;
    // (the scatter launch after this one raises these; with norms every block writes its own slot)
    unsigned* kn2 = (unsigned*)(ws + L.off_kn2) + (size_t)bh * KN2_SLOTS;
    if (!is_query && blk == 0 && tid < KN2_SLOTS && (!norms || tid >= L.nblk)) kn2[tid] = 0u;
    const bool want_norms = !CLS && sizeof(T) == 2 && norms && !is_query;
    __shared__ unsigned s_n2[4];
    unsigned n2 = 0u;
    const int j0 = blk * SB + wave * 64, rows = min(64, n - j0);
    const T* x = (is_query ? xq : xk) + (size_t)(bh / H) * xs[0] + (size_t)h * xs[1] + (size_t)j0 * xs[2];
    const uint32_t m = score_rows_topk<T, KM, score_chunk<T>(KM)>((const char*)x, (size_t)xs[2] * sizeof(T), rows, L.d, s_c, s_a[wave], K, L.topk, [&]() {
        score_stage_centroids<KM>(cents + (size_t)hk * K * L.d, s_c, K, L.d);
        if constexpr (CLS)
            for (int e = tid; e < L.NC; e += SB) s_hist_c[e] = 0;
        __syncthreads();
    }, want_norms, n2);
    if (want_norms && lane == 0) s_n2[wave] = n2;
    if (lane < rows) {
        ((uint32_t*)(ws + (is_query ? L.off_mq : L.off_mk)))[(size_t)bh * n + j0 + lane] = m;
        if constexpr (CLS) {
            const int cls = token_class(L, m);
            const size_t cls_stride = is_query ? (size_t)n : (size_t)L.nblk * SB;
            ((uint8_t*)(ws + (is_query ? L.off_qcls : L.off_kcls)))[(size_t)bh * cls_stride + j0 + lane] = (uint8_t)cls;
            atomicAdd(&s_hist_c[cls], 1);
        }
    }
    for (int g = 0; g < K; ++g) {
        const unsigned long long has = __ballot((m >> g) & 1u);
        if (lane == 0) s_h[wave][g] = __popcll(has);
    }
    __syncthreads();
    if (tid < K)
        ((int*)(ws + (is_query ? L.off_qbg : L.off_kbg)))[((size_t)bh * (L.nblk + 1) + blk) * K + tid] =
            s_h[0][tid] + s_h[1][tid] + s_h[2][tid] + s_h[3][tid];
    if (want_norms && tid == 0) kn2[blk] = max(max(s_n2[0], s_n2[1]), max(s_n2[2], s_n2[3]));
    int* bc = (int*)(ws + (is_query ? L.off_qbc : L.off_kbc)) + ((size_t)bh * (L.nblk + 1) + blk) * L.NC;
    if constexpr (CLS)
        for (int c = tid; c < L.NC; c += SB) bc[c] = s_hist_c[c];
    else if (tid == 0)
        bc[0] = min(SB, n - blk * SB);
}

// ---------------------------------------------------------------- short rows in one launch
// The whole bucketing of a (batch, head) row of a masked layout by one work-group, 64 tokens per wavefront: memberships, group
// counts and lists, positions.  For attention kernels that read k in place (no key copy, no bits, no norms).  All of it is
// latency: the launch between scores and lists costs more than spreading a row over several compute units saves
// (12 + 12 heads of 64, K = 4: 512 tokens 18.7 -> 7.9 us with the key copy left out, 10.7 in two launches).
template <typename T, int KM, int NW>
__global__ __launch_bounds__(64 * NW) void bucket_row_kernel(Layout L, HeadMap hm, const T* __restrict__ xq, const T* __restrict__ xk,
                                                             const float* __restrict__ cents, char* __restrict__ ws)
{
    __shared__ __align__(16) char s_a[NW][score_lds(64)];
    __shared__ int s_w[NW][KM];
    extern __shared__ __align__(16) char s_cent[];
    score_cent_t<KM>* s_c = (score_cent_t<KM>*)s_cent;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int is_query = side_of_row(L, -1, blockIdx.x), bh = row_in_side(L, -1, blockIdx.x);
    const int K = L.K, n = L.n;
    const int H = is_query ? L.Hq : L.Hkv, h = bh % H, hk = is_query ? hm.kv[h] : h;
    const long long* xs = is_query ? L.qs : L.ks;
    const int pos = wave * 64 + lane;
    const T* x = (is_query ? xq : xk) + (size_t)(bh / H) * xs[0] + (size_t)h * xs[1] + (size_t)(wave * 64) * xs[2];
    const uint32_t m = score_rows_topk<T, KM, 64>((const char*)x, (size_t)xs[2] * sizeof(T), min(64, n - wave * 64), L.d, s_c, s_a[wave], K,
                                              L.topk, [&]() {
                                                  score_stage_centroids<KM>(cents + (size_t)hk * K * L.d, s_c, K, L.d);
                                                  __syncthreads();
                                              });
    for (int g = 0; g < K; ++g) {
        const unsigned long long has = __ballot((m >> g) & 1u);
        if (lane == 0) s_w[wave][g] = __popcll(has);
    }
    __syncthreads();
    // lane g: entries of group g in all and before this wavefront, then where its list begins
    int total = 0, before = 0;
    if (lane < K) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int c = s_w[w][lane];
            total += c;
            before += w < wave ? c : 0;
        }
    }
    int go = total;                               // inclusive prefix sum over the groups: they lie back to back in the list
    for (int off = 1; off < K; off <<= 1) {
        const int y = __shfl_up(go, off, 64);
        if (lane >= off) go += y;
    }
    go -= total;
    if (wave == 0 && lane < K) {
        ((int*)(ws + (is_query ? L.off_qgc : L.off_kgc)))[(size_t)bh * K + lane] = total;
        int* goff = (int*)(ws + (is_query ? L.off_qgo : L.off_kgo)) + (size_t)bh * (K + 1);
        goff[lane] = go;
        if (lane == K - 1) goff[K] = go + total;
    }
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int* lists = (int*)(ws + (is_query ? L.off_qgl : L.off_kgl)) + (size_t)bh * L.topk * n;
    for (int g = 0; g < K; ++g) {
        const unsigned long long has = __ballot((m >> g) & 1u);
        const int first = __builtin_amdgcn_readlane(go + before, g);
        if ((m >> g) & 1u) lists[first + __popcll(has & lt)] = pos;
    }
    if (pos < n) ((uint32_t*)(ws + (is_query ? L.off_mq : L.off_mk)))[(size_t)bh * n + pos] = m;
    const int plen = is_query ? L.NQP : L.NKP;
    for (int p = tid; p < plen; p += 64 * NW) {       // (the first round holds every token)
        if (is_query) {
            ((int*)(ws + L.off_qperm))[(size_t)bh * L.NQP + p] = p < n ? p : -1;
        } else {
            ((int*)(ws + L.off_kpos))[(size_t)bh * L.NKP + p] = p < n ? p : KPOS_PAD;
            ((uint32_t*)(ws + L.off_kmsk))[(size_t)bh * L.NKP + p] = p < n ? m : 0u;
        }
    }
}

__global__ void fill_i32_kernel(int* __restrict__ p, size_t count, int value)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < count; i += step) p[i] = value;
}

// ---------------------------------------------------------------- scatter
// k: the key rows (16-bit types) for the class-ordered copy the matrix-core attention kernel reads, or NULL.
// The copy also leaves the largest squared key norm of the (batch, KV head) in the workspace (off_kn2: KN2_SLOTS
// partial maxima per head, cleared by the kernel before it): a non-negative float orders like its bit pattern, so one
// atomicMax on the bits per work-group does it, and a NaN or infinite norm ends up above every finite one.
// LINEAR (masked layouts): one class, slot = position.  OWN_SCAN: no scan launch ran; the work-group adds up the group
// histograms of the row's sort blocks itself (a few thousand integers at most), and sort block 0 writes the row's counts.
template <bool LINEAR, bool OWN_SCAN>
__global__ __launch_bounds__(SB) void scatter_kernel(Layout L, int which, const uint16_t* __restrict__ k, int norms_done, char* __restrict__ ws)
{
    static_assert(LINEAR || !OWN_SCAN, "class offsets come from the scan launch");
    __shared__ int s_wc[LINEAR ? 1 : 4][LINEAR ? 1 : MAX_CLASSES];
    __shared__ int s_lo[32], s_tot[32];           // first entry of this block in every group's list; list lengths (OWN_SCAN)
    __shared__ int s_wg[4][32];
    __shared__ int s_dest[SB];
    __shared__ unsigned s_n2[SB / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int blk = blockIdx.x;
    // the key rows (the long ones: they copy their sort block of K) are dispatched first
    const unsigned yrow = gridDim.y - 1u - blockIdx.y;
    const int is_query = side_of_row(L, which, yrow);
    const int bh = row_in_side(L, which, yrow);
    const int n = L.n, NC = L.NC, K = L.K;
    const int pos = blk * SB + tid;
    const bool valid = pos < n;
    const uint32_t* masks = (const uint32_t*)(ws + (is_query ? L.off_mq : L.off_mk));
    const uint8_t* clsarr = (const uint8_t*)(ws + (is_query ? L.off_qcls : L.off_kcls));
    const size_t cls_stride = is_query ? (size_t)n : (size_t)L.nblk * SB;
    const uint32_t mask = valid ? masks[(size_t)bh * n + pos] : 0u;
    const int cls = !valid ? -1 : LINEAR ? 0 : (int)clsarr[(size_t)bh * cls_stride + pos];

    if constexpr (!LINEAR) {
        for (int e = tid; e < 4 * MAX_CLASSES; e += SB) (&s_wc[0][0])[e] = 0;
    }
    const int* bg_row = (const int*)(ws + (is_query ? L.off_qbg : L.off_kbg)) + (size_t)bh * (L.nblk + 1) * K;
    if constexpr (OWN_SCAN) {
        for (int g = wave; g < K; g += 4) {       // a wavefront per group: entries before this block, and in all
            int before = 0, all = 0;
            for (int b2 = lane; b2 < L.nblk; b2 += 64) {
                const int x = bg_row[(size_t)b2 * K + g];
                before += b2 < blk ? x : 0;
                all += x;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                before += __shfl_xor(before, off, 64);
                all += __shfl_xor(all, off, 64);
            }
            if (lane == 0) { s_lo[g] = before; s_tot[g] = all; }
        }
    }
    __syncthreads();

    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // stable rank among the tokens of the same class inside this wavefront
    int rank_c = 0;
    unsigned long long todo = LINEAR ? 0ull : __ballot(valid);
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int c0 = __shfl(cls, leader, 64);
        const unsigned long long same = __ballot(valid && cls == c0);
        if (valid && cls == c0) rank_c = __popcll(same & lt);
        if (lane == leader) s_wc[LINEAR ? 0 : wave][LINEAR ? 0 : c0] = __popcll(same);
        todo &= ~same;
    }
    // per-wavefront totals of every group bit
    const bool put_bits = !is_query && L.masked && k != nullptr;
    for (int g = 0; g < K; ++g) {
        const unsigned long long has = __ballot(valid && ((mask >> g) & 1u));
        if (lane == 0) s_wg[wave][g] = __popcll(has);
        if (put_bits && lane < 4 && (blk * 4 + wave) * KT < L.NKP) {
            // masked layout: slot = position, this wavefront holds one key tile of 64
            ((uint32_t*)(ws + L.off_kbits))[(((size_t)bh * (L.NKP / KT) + blk * 4 + wave) * 4 + lane) * (K + 1) + g] =
                pack_unit_bits((uint32_t)(has >> (32 * (lane >> 1))), lane & 1);
        }
    }
    __syncthreads();
    if (tid < K) {
        if constexpr (OWN_SCAN) {
            int go = 0;                           // groups lie back to back in the list
            for (int g = 0; g < tid; ++g) go += s_tot[g];
            if (blk == 0) {
                ((int*)(ws + (is_query ? L.off_qgc : L.off_kgc)))[(size_t)bh * K + tid] = s_tot[tid];
                ((int*)(ws + (is_query ? L.off_qgo : L.off_kgo)))[(size_t)bh * (K + 1) + tid] = go;
                if (tid == K - 1) ((int*)(ws + (is_query ? L.off_qgo : L.off_kgo)))[(size_t)bh * (K + 1) + K] = go + s_tot[tid];
            }
            s_wg[3][tid] = go + s_lo[tid] + s_wg[0][tid] + s_wg[1][tid] + s_wg[2][tid];
        } else {
            const int* go = (const int*)(ws + (is_query ? L.off_qgo : L.off_kgo)) + (size_t)bh * (K + 1);
            s_wg[3][tid] = go[tid] + bg_row[(size_t)blk * K + tid] + s_wg[0][tid] + s_wg[1][tid] + s_wg[2][tid];
        }
        // s_wg[w]: first list entry of wavefront w
        s_wg[2][tid] = s_wg[3][tid] - s_wg[2][tid];
        s_wg[1][tid] = s_wg[2][tid] - s_wg[1][tid];
        s_wg[0][tid] = s_wg[1][tid] - s_wg[0][tid];
    }
    __syncthreads();

    const int* bc = (const int*)(ws + (is_query ? L.off_qbc : L.off_kbc)) + ((size_t)bh * (L.nblk + 1) + blk) * NC;
    const int* co = (const int*)(ws + (is_query ? L.off_qco : L.off_kco)) + (size_t)bh * (NC + 1);
    int dest = -1;
    if (valid) {
        if constexpr (LINEAR) {
            dest = pos;
        } else {
            int before = 0;
            for (int w = 0; w < wave; ++w) before += s_wc[w][cls];
            dest = co[cls] + bc[cls] + before + rank_c;
        }
        if (is_query) {
            ((int*)(ws + L.off_qperm))[(size_t)bh * L.NQP + dest] = pos;
        } else {
            ((int*)(ws + L.off_kpos))[(size_t)bh * L.NKP + dest] = pos;
            if (L.coarse) ((uint32_t*)(ws + L.off_kmsk))[(size_t)bh * L.NKP + dest] = mask;
        }
    }
    // group lists: position-ascending because ranks follow the position order
    int* lists = (int*)(ws + (is_query ? L.off_qgl : L.off_kgl)) + (size_t)bh * L.topk * n;
    for (int g = 0; g < K; ++g) {
        const bool mine = valid && ((mask >> g) & 1u);
        const unsigned long long has = __ballot(mine);
        if (mine) lists[s_wg[wave][g] + __popcll(has & lt)] = pos;
    }

    // ---- pads of the class-ordered arrays: the work-group of sort block b fills those of the classes b, b + nblk, ...
    // (class NC stands for the unused end of the arrays).  qperm -1, kpos KPOS_PAD, masks and key rows zero.
    const int* cnt = (const int*)(ws + (is_query ? L.off_qcc : L.off_kcc)) + (size_t)bh * NC;
    const int plen = is_query ? L.NQP : L.NKP;
    const bool copy_k = !is_query && k != nullptr && !L.k_direct;       // else at most the norms
    const int CPR = L.d / 8;                         // 16-byte chunks per row of k and of the key copy
    uint4* kc = (uint4*)(ws + L.off_kc) + (size_t)bh * L.NKP * CPR;
    for (int c = LINEAR ? L.nblk - 1 - blk : blk; c <= NC; c += L.nblk) {      // (LINEAR: NC = 1, left to the last sort blocks)
        const int end0 = LINEAR ? min(plen, (n + KT - 1) / KT * KT) : 0;
        const int p0 = LINEAR ? (c == 0 ? n : end0) : c < NC ? co[c] + cnt[c] : co[NC];
        const int p1 = LINEAR ? (c == 0 ? end0 : plen) : c < NC ? co[c + 1] : plen;
        for (int p = p0 + tid; p < p1; p += SB) {
            if (is_query) {
                ((int*)(ws + L.off_qperm))[(size_t)bh * L.NQP + p] = -1;
            } else {
                ((int*)(ws + L.off_kpos))[(size_t)bh * L.NKP + p] = KPOS_PAD;
                if (L.coarse) ((uint32_t*)(ws + L.off_kmsk))[(size_t)bh * L.NKP + p] = 0u;
            }
        }
        if (copy_k && c < NC)                        // (nothing reads the key rows past the last class)
            for (int id = tid; id < (p1 - p0) * CPR; id += SB) kc[(size_t)p0 * CPR + id] = make_uint4(0, 0, 0, 0);
    }

    // ---- key rows: this sort block's rows into their class-ordered places
    if (!copy_k && (is_query || k == nullptr || norms_done)) return;
    s_dest[tid] = dest;
    __syncthreads();
    const int lsh = CPR <= 8 ? 3 : CPR <= 16 ? 4 : 5, lpr = 1 << lsh;    // lanes per row, the last ones idle at d = 80 and 96
    const bool f16 = L.dtype == 2;
    // source rows through the strides of k (multiples of 8 elements = one 16-byte chunk)
    const uint4* src = (const uint4*)k + ((size_t)(bh / L.Hkv) * L.ks[0] + (size_t)(bh % L.Hkv) * L.ks[1] + (size_t)blk * SB * L.ks[2]) / 8;
    const size_t pitch = (size_t)L.ks[2] / 8;
    unsigned n2max = 0u;
    // four pieces in flight per lane (8 heads of 128 x 32768: 41 -> 35 us for the launch)
    for (int id0 = tid; id0 < SB * lpr; id0 += 4 * SB) {
        uint4 val[4];
        int dd[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int id = id0 + i * SB, row = id >> lsh, ch = id & (lpr - 1);
            dd[i] = ch < CPR ? s_dest[row] : -1;
            val[i] = dd[i] >= 0 ? src[(size_t)row * pitch + ch] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (copy_k && dd[i] >= 0) kc[(size_t)dd[i] * CPR + ((id0 + i * SB) & (lpr - 1))] = val[i];
            // the chunks of a row sit in lpr consecutive lanes (a power of two <= 32, rows do not straddle waves)
            float n2 = piece_norm2(val[i].x, val[i].y, val[i].z, val[i].w, f16, 0.f);
            for (int off = 1; off < lpr; off <<= 1) n2 += __shfl_xor(n2, off, 64);
            const unsigned bits = __float_as_uint(n2) & 0x7fffffffu;     // a NaN may carry a sign bit
            n2max = bits > n2max ? bits : n2max;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const unsigned o = (unsigned)__shfl_xor((int)n2max, off, 64);
        n2max = o > n2max ? o : n2max;
    }
    if (lane == 0) s_n2[wave] = n2max;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < SB / 64; ++w) n2max = s_n2[w] > n2max ? s_n2[w] : n2max;
        // KN2_SLOTS slots per head, so that the work-groups of a head do not queue up on one address
        if (n2max != 0u) atomicMax((unsigned*)(ws + L.off_kn2) + (size_t)bh * KN2_SLOTS + (blk % KN2_SLOTS), n2max);
    }
}

// ---------------------------------------------------------------- one class in position order
// What the tiled kernel reads of a layout in which every token is in one class and no membership counts (the soft gate, the
// window pass of a two-pass launch): the keys' positions and their copy, in one launch.  The bucketing with a constant
// membership did the same in three, with lists, histograms and a scan that nobody read (8192 tokens, 8 heads of 128:
// 41 us before, 11 now).  kn2: the largest key norms of the same keys, found by the bucketing before; NULL: not needed.
__global__ __launch_bounds__(SB) void position_layout_kernel(Layout L, const uint4* __restrict__ k, const unsigned* __restrict__ kn2,
                                                             char* __restrict__ ws)
{
    const int tid = threadIdx.x, bh = blockIdx.y, p0 = blockIdx.x * SB, p1 = min(L.NKP, p0 + SB);
    const int CPR = L.d / 8;                          // 16-byte chunks per row
    if (p0 + tid < p1) ((int*)(ws + L.off_kpos))[(size_t)bh * L.NKP + p0 + tid] = p0 + tid < L.n ? p0 + tid : KPOS_PAD;
    if (kn2 && blockIdx.x == 0 && tid < KN2_SLOTS)
        ((unsigned*)(ws + L.off_kn2))[(size_t)bh * KN2_SLOTS + tid] = kn2[(size_t)bh * KN2_SLOTS + tid];
    const uint4* src = k + ((size_t)(bh / L.Hkv) * L.ks[0] + (size_t)(bh % L.Hkv) * L.ks[1]) / 8;
    const size_t pitch = (size_t)L.ks[2] / 8;
    uint4* dst = (uint4*)(ws + L.off_kc) + ((size_t)bh * L.NKP + p0) * CPR;
    if (L.k_direct) return;                           // (the tiled kernel reads the keys in place)
    for (int id = tid; id < (p1 - p0) * CPR; id += SB) {
        const int p = p0 + id / CPR, ch = id % CPR;
        dst[id] = p < L.n ? src[(size_t)p * pitch + ch] : make_uint4(0, 0, 0, 0);
    }
}

// ---------------------------------------------------------------- membership given per token
// The paper's router assigns one membership per token of a layer, shared by all heads and by the
// query and key roles (Sec. 2).  A work-group turns the token masks of a sort block of a batch element into
// class ids and histograms and writes them for its share of the query and KV heads (heads z, z + gridDim.z, ..),
// in the same places the score kernel fills.  A mask that is not a topk-subset of the K groups would index
// outside the class tables: it is replaced by the first topk groups and counted.
__global__ __launch_bounds__(SB) void token_classes_kernel(Layout L, const uint32_t* __restrict__ token_masks,
                                                           char* __restrict__ ws, int32_t* __restrict__ invalid_count)
{
    __shared__ int s_hist_c[MAX_CLASSES];
    __shared__ int s_hist_g[32];
    const int tid = threadIdx.x;
    const int blk = blockIdx.x, b = blockIdx.y;
    const int n = L.n, K = L.K;
    const int pos = blk * SB + tid;
    for (int e = tid; e < MAX_CLASSES; e += SB) s_hist_c[e] = 0;
    if (tid < 32) s_hist_g[tid] = 0;
    if (blk == 0 && blockIdx.z == 0)              // (the scatter launch raises these)
        for (int e = tid; e < L.Hkv * KN2_SLOTS; e += SB) ((unsigned*)(ws + L.off_kn2))[(size_t)b * L.Hkv * KN2_SLOTS + e] = 0u;
    __syncthreads();
    uint32_t mask = 0;
    int cls = 0;
    if (pos < n) {
        // no masks given: every token in the first topk groups (callers that need one class in position order)
        mask = token_masks ? token_masks[(size_t)b * n + pos] : ((L.topk == 32) ? 0xffffffffu : ((1u << L.topk) - 1u));
        const uint32_t allowed = (K == 32) ? 0xffffffffu : ((1u << K) - 1u);
        if ((mask & ~allowed) != 0u || __popc(mask) != L.topk) {
            mask = (L.topk == 32) ? 0xffffffffu : ((1u << L.topk) - 1u);
            if (invalid_count && blockIdx.z == 0) atomicAdd(invalid_count, 1);
        }
        cls = token_class(L, mask);
        atomicAdd(&s_hist_c[cls], 1);
        for (int g = 0; g < K; ++g)
            if ((mask >> g) & 1u) atomicAdd(&s_hist_g[g], 1);
    }
    __syncthreads();
    for (int is_query = 1; is_query >= 0; --is_query) {
        const int H = is_query ? L.Hq : L.Hkv;
        uint32_t* masks = (uint32_t*)(ws + (is_query ? L.off_mq : L.off_mk));
        uint8_t* clsarr = (uint8_t*)(ws + (is_query ? L.off_qcls : L.off_kcls));
        const size_t cls_stride = is_query ? (size_t)n : (size_t)L.nblk * SB;
        for (int h = blockIdx.z; h < H; h += gridDim.z) {
            const size_t bh = (size_t)b * H + h;
            if (pos < n) {
                masks[bh * n + pos] = mask;
                clsarr[bh * cls_stride + pos] = (uint8_t)cls;
            }
            int* bc = (int*)(ws + (is_query ? L.off_qbc : L.off_kbc)) + (bh * (L.nblk + 1) + blk) * L.NC;
            int* bg = (int*)(ws + (is_query ? L.off_qbg : L.off_kbg)) + (bh * (L.nblk + 1) + blk) * K;
            for (int c = tid; c < L.NC; c += SB) bc[c] = s_hist_c[c];
            if (tid < K) bg[tid] = s_hist_g[tid];
        }
    }
}

// scores and memberships of the queries and of the keys, one launch: query rows first, key rows after them
template <typename T, int KM>
hipError_t launch_score(const Layout& L, const HeadMap& hm, const void* q, const void* k, const float* centroids, int norms, char* ws, hipStream_t st)
{
    const size_t lds = score_cent_bytes(KM, L.d);                    // with the staging space below 87 KB
    // (more rows than one launch can have: the two sides one after the other)
    const bool both = L.B * (L.Hq + L.Hkv) <= MAX_GRID_ROWS;
    for (int which = both ? -1 : 1; which >= -1; --which) {
        const dim3 grid(L.nblk, which < 0 ? L.B * (L.Hq + L.Hkv) : which ? L.B * L.Hq : L.B * L.Hkv);
        if (L.masked) hipLaunchKernelGGL((score_kernel<T, KM, false>), grid, dim3(SB), lds, st, L, hm, (const T*)q, (const T*)k, centroids, which, norms, ws);
        else hipLaunchKernelGGL((score_kernel<T, KM, true>), grid, dim3(SB), lds, st, L, hm, (const T*)q, (const T*)k, centroids, which, norms, ws);
        if (which <= 0) break;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_score_k(const Layout& L, const HeadMap& hm, const void* q, const void* k, const float* centroids, int norms, char* ws, hipStream_t st)
{
    if (L.K <= 4) return launch_score<T, 4>(L, hm, q, k, centroids, norms, ws, st);
    if (L.K <= 8) return launch_score<T, 8>(L, hm, q, k, centroids, norms, ws, st);
    if (L.K <= 16) return launch_score<T, 16>(L, hm, q, k, centroids, norms, ws, st);
    return launch_score<T, 32>(L, hm, q, k, centroids, norms, ws, st);
}

// One launch where a row is little enough work for one compute unit (scores are n * d products of 4 or 8 groups; above 8
// groups 16 columns are computed).  Bucketing, one launch / two (us): 12 + 12 heads of 64, K = 4: 512 tokens 7.9 / 10.7, 1024 10.5 / 11.6;
// 8 + 2 of 128: K = 4 512 tokens 10.0 / 12.3, 700 12.1 / 11.9, 1024 14.4 / 12.1; K = 8 512 13.0 / 15.2, 1024 19.2 / 15.1; K = 16 512
// 21.7 / 22.7; 16 + 4 of 256 in fp32, 512, K = 16 34 / 32.
// Many rows, where the chip is full in any case (fp32; a 16-bit layout of the short kernel has few): two launches share a row in
// sort blocks of 256 tokens, and lose where the last one is mostly empty.  Rows of 64, K = 4: 480 x 512 tokens 17.4 / 19.1, 768
// 29.6 / 25.6, 1536 52.0 / 42.7; 3072 x 400 64.3 / 78.2, x 256 42.4 / 43.0; K = 8: 3072 x 512 99.9 / 109, x 256 52.8 / 52.2; K = 16: 1536 x 256
// 47.5 / 48.9, 3072 87.5 / 85.7, x 100 81.0 / 76.5, x 512 130 / 164.
bool short_rows(const Layout& L)
{
    const int rows = L.B * (L.Hq + L.Hkv);
    const int most = L.n > 512 || (L.n > 448 && L.K <= 4) ? 512 : L.n <= 256 && L.K > 8 ? 2048 : 0x7fffffff;
    return L.masked && (L.dtype == 0 || short_attention(L)) && (long long)L.n * L.d <= 65536 && L.n <= (L.K <= 8 ? 1024 : L.K <= 16 ? 512 : 0) &&
           rows <= most;
}

template <typename T, int KM, int NW>
hipError_t launch_bucket_rows(const Layout& L, const HeadMap& hm, const void* q, const void* k, const float* centroids, char* ws, hipStream_t st)
{
    hipLaunchKernelGGL((bucket_row_kernel<T, KM, NW>), dim3(L.B * (L.Hq + L.Hkv)), dim3(64 * NW), score_cent_bytes(KM, L.d), st, L, hm,
                       (const T*)q, (const T*)k, centroids, ws);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_bucket_rows_k(const Layout& L, const HeadMap& hm, const void* q, const void* k, const float* centroids, char* ws, hipStream_t st)
{
#define FOCUS_ROWS(KM_) (L.n <= 512 ? launch_bucket_rows<T, KM_, 8>(L, hm, q, k, centroids, ws, st) : launch_bucket_rows<T, KM_, 16>(L, hm, q, k, centroids, ws, st))
    if (L.K <= 4) return FOCUS_ROWS(4);
    if (L.K <= 8) return FOCUS_ROWS(8);
    return launch_bucket_rows<T, 16, 8>(L, hm, q, k, centroids, ws, st);
#undef FOCUS_ROWS
}

// Masked layouts need no class tables and no job list: where a row's group histograms are few, the scatter launch adds
// them up itself and the scan launch (10 us of latency, one work-group per row) is left out.
bool own_scan(const Layout& L) { return L.masked && (long long)L.nblk * L.K <= 4096; }

// from class ids, block prefixes and the per-row plan to the class-ordered arrays, group lists and key copy
hipError_t launch_scatter(const Layout& L, const void* k, int norms_done, char* ws, hipStream_t st)
{
    // query side and key side in the same launch: rows [0, B*Hq) and the B*Hkv rows after them
    // (more rows than one launch can have: the two sides one after the other)
    const uint16_t* kcopy = L.dtype != 0 && !short_attention(L) ? (const uint16_t*)k : nullptr;   // key copy for the tiled kernel
    const bool both = L.B * (L.Hq + L.Hkv) <= MAX_GRID_ROWS;
    for (int which = both ? -1 : 1; which >= -1; --which) {
        const int rows = which < 0 ? L.B * (L.Hq + L.Hkv) : which ? L.B * L.Hq : L.B * L.Hkv;
        if (own_scan(L)) hipLaunchKernelGGL((scatter_kernel<true, true>), dim3(L.nblk, rows), dim3(SB), 0, st, L, which, kcopy, norms_done, ws);
        else if (L.masked) hipLaunchKernelGGL((scatter_kernel<true, false>), dim3(L.nblk, rows), dim3(SB), 0, st, L, which, kcopy, norms_done, ws);
        else hipLaunchKernelGGL((scatter_kernel<false, false>), dim3(L.nblk, rows), dim3(SB), 0, st, L, which, kcopy, norms_done, ws);
        if (which <= 0) break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_assign(const Layout& L, const HeadMap& hm, const void* q, const void* k,
                         const float* centroids, char* ws, hipStream_t st)
{
    if (short_rows(L))
        return L.dtype == 0 ? launch_bucket_rows_k<float>(L, hm, q, k, centroids, ws, st)
               : L.dtype == 2 ? launch_bucket_rows_k<f16_bits>(L, hm, q, k, centroids, ws, st)
                              : launch_bucket_rows_k<uint16_t>(L, hm, q, k, centroids, ws, st);
    // keys that the tiled kernel reads where they are: their norms come with the scores, a slot for every sort block
    static_assert(KEYS_IN_PLACE / SB <= KN2_SLOTS, "a slot for every sort block of keys read in place");
    const int norms = L.k_direct && !short_attention(L) ? 1 : 0;
    const hipError_t e = L.dtype == 0 ? launch_score_k<float>(L, hm, q, k, centroids, norms, ws, st)
                         : L.dtype == 2 ? launch_score_k<f16_bits>(L, hm, q, k, centroids, norms, ws, st)
                                        : launch_score_k<uint16_t>(L, hm, q, k, centroids, norms, ws, st);
    if (e != hipSuccess) return e;
    if (!own_scan(L)) hipLaunchKernelGGL(scan_plan_kernel, dim3(L.B * (L.Hq + L.Hkv)), dim3(SCAN_THREADS), 0, st, L, ws);
    return launch_scatter(L, k, norms, ws, st);
}

hipError_t launch_position_layout(const Layout& L, const void* k, const unsigned* kn2, char* ws, hipStream_t st)
{
    hipLaunchKernelGGL(position_layout_kernel, dim3((L.NKP + SB - 1) / SB, L.B * L.Hkv), dim3(SB), 0, st, L, (const uint4*)k, kn2, ws);
    return hipGetLastError();
}

hipError_t launch_assign_tokens(const Layout& L, const uint32_t* token_masks, const void* k, char* ws,
                                int32_t* invalid_count, hipStream_t st)
{
    if (invalid_count) hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, st, invalid_count, (size_t)1, 0);
    // the heads of a sort block are split until there are a few work-groups per compute unit (128 blocks x 40 heads: one
    // work-group for all heads wrote for 11 us, eight for 5)
    const int zsplit = (int)std::max<long long>(1, std::min<long long>(std::max(L.Hq, L.Hkv), 1024 / ((long long)L.nblk * L.B)));
    hipLaunchKernelGGL(token_classes_kernel, dim3(L.nblk, L.B, zsplit), dim3(SB), 0, st, L, token_masks, ws, invalid_count);
    if (!own_scan(L)) hipLaunchKernelGGL(scan_plan_kernel, dim3(L.B * (L.Hq + L.Hkv)), dim3(SCAN_THREADS), 0, st, L, ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_scatter(L, k, 0, ws, st);
}

}  // namespace focus
