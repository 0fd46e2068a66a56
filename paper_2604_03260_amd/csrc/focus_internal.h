// Internal layout of the workspace and the launch entry points shared by the
// translation units of libfocus.so.  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace focus {

constexpr int SB = 256;        // positions per sort block (one work-group of the bucketing kernels)
constexpr int BQ_VECTOR = 128; // query rows the fp32 vector kernel handles per pass (and its tile size)
constexpr int LONG_N = 1 << 18; // from this sequence length on the MFMA kernel uses 8-wavefront work-groups (256-row tiles)
constexpr int LONG_N_TWO_PASS = 1 << 17; // ... and from this length on where the attention launch runs as two passes
constexpr int KT = 64;         // keys per attention tile; class segments of the permuted keys are padded to this
constexpr int MAX_CLASSES = 256;
constexpr int MAX_HQ = 256;
constexpr int KEYS_IN_PLACE = 8192;    // longest sequence whose keys the tiled kernel reads in place (Layout::k_direct)
constexpr int KN2_SLOTS = 64;  // partial maxima of the squared key norms per (batch, KV head), one per lane of a wavefront
constexpr int KPOS_PAD = 0x7fffffff;  // position stored in padded key slots: never <= a query position

// Element types as the kernels see them: float, uint16_t for a bfloat16 bit pattern, f16_bits for an IEEE half.
struct f16_bits { uint16_t v; };
// Direct global -> LDS load of one wavefront: lane l fetches the 16 bytes at (sbase + voff) into LDS byte address
// lds_addr + 16*l (global_load_lds_dwordx4; sbase and lds_addr wave-uniform, voff per lane).  Counted by vmcnt
// like any vector memory load: `s_waitcnt vmcnt(0)` before the data is read from LDS.
__device__ inline void lds_dma16(const void* sbase, unsigned voff, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}
// LDS byte address of a __shared__ object (the low half of its generic address)
__device__ inline unsigned lds_addr_of(const void* p) { return (unsigned)(uintptr_t)p; }

__device__ inline float f16_bits_to_f32(uint16_t b)
{
    _Float16 h;
    __builtin_memcpy(&h, &b, 2);
    return (float)h;
}
__device__ inline uint16_t f32_to_f16_bits(float f)
{
    const _Float16 h = (_Float16)f;                     // round to nearest even
    uint16_t b;
    __builtin_memcpy(&b, &h, 2);
    return b;
}

struct HeadMap {               // query head -> KV head, passed by value to kernels
    uint8_t kv[MAX_HQ];
};

// Everything the kernels need to know about shapes and where things live in the
// workspace (byte offsets from its base, all multiples of 256).
struct Layout {
    int B, Hq, Hkv, n, d;
    int K, topk, window;       // window clamped to n
    int causal;                // 1: keys j <= i, local = i-w < j <= i; 0: every j, local = |i-j| < w
    int dtype;                 // 0 fp32, 1 bf16, 2 fp16
    int elem;                  // bytes per element
    int k_direct;              // masked and soft-gate layouts of 16-bit types: the tiled kernel reads the keys in place, through
                               // the strides of k (a wavefront's tile addresses fit 32 bits); no key copy
    int BQ;                    // query rows per attention tile (128; 256 for 16-bit types at n >= LONG_N, d <= 128)
    int NC;                    // number of membership classes (1 in dense mode)
    int dense;                 // every causal pair allowed: one class, no masks beyond causal
    int soft;                  // Sec. 2 Eq. 2: every causal pair, the logit of a pair outside the window scaled by
    float gate_slope;          // sigmoid(lambda * g_i . g_j); gate_slope = -lambda * log2(e).  One class, position order.
    int coarse;                // C(K,topk) exceeds MAX_CLASSES: classes are sets of S super-groups (group g folds
    int S;                     // onto g % S), a superset test; the kernels then test the real masks per pair
    int masked;                // one class in position order, every pair outside the window tested against the two
                               // membership masks (coarse with S = 1): where classes would leave tiles mostly empty,
                               // in short sequences and at any length with many sets (see prefer_masked in focus_api.hip)
    int pair_set;              // which pairs a launch attends: 0 the whole mask, 1 only pairs that share a group
                               // (set A of App. D), 2 only window pairs that share none (set B), 3 pairs that share
                               // a group and lie outside the window (second pass of a two-pass launch)
    int two_pass;              // the whole-mask attention launch of this problem runs as two passes: every pair inside
                               // the window over position-ordered rows and keys (the embedded local layout), then the
                               // pairs outside the window that share a group over class-ordered ones, merged per row
    int class_major;           // job list of the attention launch by class (long sequences) instead of by slot
    int local_only;            // this IS the embedded local layout: one class in position order, window pairs only
    int merge_prev;            // launch flag of the second pass: out / lse / row_pairs hold the first pass's partial
                               // result of every row; merge instead of overwriting (App. D's log-sum-exp merge)
    int nblk;                  // ceil(n / SB)
    int NQP;                   // padded per-head length of the class-ordered query index
    int NKP;                   // padded per-head length of the class-ordered key arrays (multiple of KT)
    int NT;                    // upper bound of query tiles per head
    float scale;
    float softcap;

    long long qs[3], ks[3], os[3];     // strides of q, of k and v, of out in elements (batch, head, position)

    size_t off_mq, off_mk;
    size_t off_qgc, off_kgc;           // group counts
    size_t off_qgl, off_kgl;           // group lists
    size_t off_qgo, off_kgo;           // group list offsets [.,K+1]
    size_t off_qcls, off_kcls;         // class id per position, uint8
    size_t off_qbc, off_kbc;           // per sort block class histogram -> exclusive prefix [.,nblk,NC]
    size_t off_qbg, off_kbg;           // per sort block group histogram -> exclusive prefix [.,nblk,K]
    size_t off_qcc, off_kcc;           // class counts [.,NC]
    size_t off_qco, off_kco;           // padded class offsets [.,NC+1]
    size_t off_clsmask;                // group bit mask of each class [NC]
    size_t unused;                     // 8 bytes without a meaning.  Without them the attention kernel at 262144 tokens took 0.4 to 0.9 %
                                       // longer (three boxes, in turn: 400.2 / 402.2, 408.5 / 411.2, 411.2 / 414.9 ms; 32768 tokens +0.1 %,
                                       // 131072 with a softcap +0.3 %), also with the structure padded back to its size: the offsets below
                                       // are then loaded in other groups, and the kernel's registers fall otherwise.  Results are the same
                                       // bits.  To be measured again when a field is added or leaves.
    size_t off_qperm;                  // [B,Hq,NQP] positions in class order, -1 in pads (the scatter kernel writes both)
    size_t off_kpos;                   // [B,Hkv,NKP] positions in class order, KPOS_PAD in pads
    size_t off_kmsk;                   // [B,Hkv,NKP] membership masks in class order, 0 in pads (coarse classes only)
    size_t off_kbits;                  // [B,Hkv,NKP/KT][2 units of 32 keys][2 half-waves][K + 1] one bit per key (masked,
                                       // 16-bit types; pack_unit_bits): membership by group, then "its V row is not finite" 
    size_t off_jobs;                   // [B,Hq,NT] (class << 24 | tile) heaviest first, -1 unused
    size_t off_gk;                     // [B,NKP,2,16 or 32] bf16: the soft assignment of every key position as bf16 high and
                                       // low parts, groups padded to 16 or 32, chunks swizzled per key (soft gate, 16-bit types)
    size_t off_kn2;                    // [B,Hkv,KN2_SLOTS] bit patterns of partial maxima of the squared key norms of the
                                       // head (16-bit types; cleared with the memberships, raised by the scatter kernel's key
                                       // copy, the attention kernel takes the largest)
    size_t off_local;                  // the embedded local layout's own workspace (two_pass)
    size_t off_lse1;                   // [B,Hq,n] fp32: log-sum-exp of the first pass when the caller passes no lse (two_pass)
    size_t off_nrflag;                 // [B,Hq,NT] per work-group of the attention launch: 1 = the no-reference
                                       // instantiation did the tile, 0 = left to the other one (16-bit types)
    size_t off_kc;                     // [B,Hkv,NKP,d] keys in class order (16-bit types, unless k_direct)
    size_t off_vt;                     // [B,Hkv,NKP/KT,d,KT] values, transposed per key tile (16-bit types)
    size_t total;
};

// The bits of one half-wave of a 32-key unit (x: bit j = key j) in the order its attention lanes hold their scores:
// score r belongs to key 8*(r/4) + 4*half + r%4; score 2p in bit p, score 2p + 1 in bit 16 + p.
__host__ __device__ inline uint32_t pack_unit_bits(uint32_t x, int half)
{
    uint32_t word = 0;
    for (int r = 0; r < 16; ++r) word |= ((x >> (8 * (r / 4) + 4 * half + r % 4)) & 1u) << (r / 2 + (r & 1) * 16);
    return word;
}

// colex rank of the k-subset `m` among all k-subsets (device + host)
__host__ __device__ inline uint32_t binom_u32(int a, int b)
{
    if (b < 0 || b > a) return 0;
    if (b > a - b) b = a - b;
    uint64_t r = 1;
    for (int i = 1; i <= b; ++i) r = r * (uint64_t)(a - b + i) / (uint64_t)i;
    return (uint32_t)r;
}

// Coarse classes: the S-bit set of super-groups a membership mask folds onto
__host__ __device__ inline uint32_t fold_groups(uint32_t mask, int S)
{
    uint32_t r = 0;
    while (mask) {
        const int g = __builtin_ctz(mask);
        r |= 1u << (g % S);
        mask &= mask - 1;
    }
    return r;
}

// Class id of a membership mask.  Exact classes: the colex rank of the topk-subset of the K groups.
// Coarse classes: the folded set has 1..topk members; sets are ordered by size, then colex.
__host__ __device__ inline int class_of_mask(uint32_t mask, int dense, int coarse, int S)
{
    if (dense) return 0;
    uint32_t m = coarse ? fold_groups(mask, S) : mask;
    int j = 0, cls = 0;
    while (m) {
        const int g = __builtin_ctz(m);
        ++j;
        cls += (int)binom_u32(g, j);
        m &= m - 1;
    }
    if (coarse)
        for (int t = 1; t < j; ++t) cls += (int)binom_u32(S, t);
    return cls;
}

// Tokens per work-group of the router's projection: 8 wavefronts of 16 tokens where that still gives every compute unit
// a work-group (they share the staged W_g), 4 otherwise and where d_g > 16 (the scores would not fit 64 KB of LDS).
inline int route_tokens_per_group(int B, int n, int dg) { return (dg <= 16 && (long long)B * ((n + 127) / 128) >= 256) ? 128 : 64; }

// Shapes and workspace offsets of the router (focus_route).
struct RouteLayout {
    int B, n, dm, dg, K, topk;
    int dtype;                 // of the hidden states: 0 fp32, 1 bf16
    int iters;                 // Sinkhorn rounds, 0 = none
    double tau;
    int nproj;                 // work-groups of the projection per sequence = ceil(n / route_tokens_per_group)
    int nsink;                 // work-groups of a Sinkhorn pass per sequence (<= 256)
    int sink_tokens;           // tokens per Sinkhorn work-group
    int nround;                // work-groups per sequence of the launch that does all rounds, 0 = a launch per round (launch_route sets it)
    size_t off_S;              // [B][n][K] fp64: scores, then exp((S - max)/tau) in place
    size_t off_maxpart;        // [B][nproj] fp64
    size_t off_colpart;        // [2][B][nsink][KP] fp64 column partial sums, ping-pong between passes
    size_t total;
};

// Shapes and state offsets of the incremental (one token per step) path.
constexpr int DEC_CHUNK = 512;               // keys of the key sequence a work-group of the vector decode attention resolves at a time
constexpr int DEC_CHUNK_SHORT = 128;         // one round of 32 keys for each wavefront of a work-group: what a share of the matrix-core decode
                                             // attention is launched for at least (decode_shares: what it gets); sizes max_parts
constexpr int DEC_MAX_PARTS = 384;           // partial results per head the merge reads at most
// Shares of a walk of `units` rounds (32 keys each) in a launch of the matrix-core decode attention with `parts` work-groups for
// each of `rows` (batch, KV head, 16 query heads).  The walk may be far shorter than the launch was made for.  With the position
// in device memory (at) the launch is made for the whole caches, its work-groups are paid for anyway, and the walk is spread over
// all of them; so it is up to 128 rows, where the chip is not full.  Otherwise only a walk over lists is shorter, and above 128 rows
// a share of less than a round for each of the four wavefronts costs more work-groups than it saves time; the first eight
// shares do not.  A step (us), spread / four rounds / as here, and with the chunks of 512 entries of before: 256 rows of 64,
// K = 16 top-1, 9000 keys 39.0 / 33.5 / 33.4 / 34.4, 20000 70.1 / 56.2 / 55.8 / 63.6; 300 rows of 80 x 4000, K = 32 top-1 38.4 / 42.7 / 38.5 /
// 63.7.  In device memory, 256 rows, capacity 32768, position 1000, K = 4 top-2: four rounds 79, as here 70.5, before 125.
constexpr int DEC_MANY_ROWS = 128;
__host__ __device__ inline int decode_shares(int units, int parts, int rows, bool at)
{
    if (!at && rows > DEC_MANY_ROWS) {
        constexpr int ROUNDS = DEC_CHUNK_SHORT / 32;
        const int most = units <= 8 * ROUNDS ? 8 : (units + ROUNDS - 1) / ROUNDS;
        parts = most < parts ? most : parts;
    }
    return units < parts ? units : parts;
}
struct DecodeLayout {
    int B, Hq, Hkv, n, d;      // n = capacity of the caches
    int K, topk, window;
    int dtype;
    float scale, softcap;
    int max_chunks;            // chunks of DEC_CHUNK keys the longest key sequence (n entries) has
    int max_parts;             // partial results per head: min(chunks of DEC_CHUNK_SHORT keys, DEC_MAX_PARTS)
    size_t off_mk;             // [B,Hkv,n] uint32 membership of the cached keys
    size_t off_lists;          // [B,Hkv,K,n] int32 positions of every group, ascending
    size_t off_counts;         // [B,Hkv,K] int32 list lengths
    size_t off_wp;             // [B,Hkv,K] int32 list entries below the current step's window
    size_t off_mq;             // [B,Hq] uint32 membership of the current queries
    size_t off_part;           // [B,Hq,max_parts,d+4] fp32 partial (o, max, sum, count) per work-group
    size_t total;
};

// token_masks / token_mask non-NULL: memberships given per token (centroids unused) instead of scored per head
hipError_t launch_decode_prefill(const DecodeLayout& L, int n_ctx, const void* kc, const float* cents,
                                 const uint32_t* token_masks, char* st, hipStream_t s);
hipError_t launch_decode_step(const DecodeLayout& L, const HeadMap& hm, int pos, const int* pos_dev, const void* q_new, const void* k_new,
                              const void* v_new, const float* cents, const uint32_t* token_mask, void* kc, void* vc, char* st,
                              void* out, float* lse, int32_t* row_pairs, hipStream_t s);
hipError_t launch_route(const RouteLayout& R, const void* hidden, const float* wg, const float* cent, char* ws,
                        uint32_t* masks, double* soft, hipStream_t st);
// The router's scratch for callers that may not allocate: a buffer of ROUTE_STATIC_SCRATCH_BYTES that lives in
// the library's device image; *ptr is its address on the CURRENT device (looked up once per device).
constexpr size_t ROUTE_STATIC_SCRATCH_BYTES = (size_t)16 << 20;
hipError_t route_static_scratch(char** ptr);
hipError_t launch_assign_tokens(const Layout& L, const uint32_t* token_masks, const void* k, char* ws,
                                int32_t* invalid_count, hipStream_t st);
// positions and key copy of a layout of one class in position order (16-bit types, tiled kernel only)
hipError_t launch_position_layout(const Layout& L, const void* k, const unsigned* kn2, char* ws, hipStream_t st);
hipError_t launch_assign(const Layout& L, const HeadMap& hm, const void* q, const void* k,
                         const float* centroids, char* ws, hipStream_t st);
hipError_t launch_attn_simple(const Layout& L, const HeadMap& hm, const void* q, const void* k,
                              const void* v, const float* g, char* ws, void* out, float* lse, int32_t* row_pairs,
                              hipStream_t st);
bool short_attention(const Layout& L);
hipError_t launch_attn_short(const Layout& L, const HeadMap& hm, const void* q, const void* k, const void* v, char* ws,
                             void* out, float* lse, int32_t* row_pairs, hipStream_t st);
bool short_soft_attention(const Layout& L);
hipError_t launch_attn_short_soft(const Layout& L, const HeadMap& hm, const float* g, const void* q, const void* k, const void* v, char* ws,
                                  void* out, float* lse, hipStream_t st);
hipError_t launch_attn_f32(const Layout& L, const HeadMap& hm, const void* q, const void* k, const void* v, char* ws,
                           void* out, float* lse, int32_t* row_pairs, hipStream_t st);
hipError_t launch_soft_gather_g(const Layout& L, const float* g, char* ws, hipStream_t st);
hipError_t launch_attn_merge(size_t rows, int d, int dtype, const void* oa, const float* la, const void* ob,
                             const float* lb, void* out, float* lse, hipStream_t st);
hipError_t launch_attn_mfma(const Layout& L, const HeadMap& hm, const void* q, const void* k,
                            const void* v, const float* g, char* ws, void* out, float* lse, int32_t* row_pairs,
                            hipStream_t st);

}  // namespace focus
