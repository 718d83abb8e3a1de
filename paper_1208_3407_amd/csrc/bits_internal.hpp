// Internal declarations of libbits.so (gfx950).  Device helpers used by the
// search, Monte-Carlo, batch and learned-index kernels, and the host-side
// launchers each translation unit exports to the C ABI layer (api.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/bits.h"

#define BITS_CHECK_HIP(expr)                                   \
    do {                                                       \
        hipError_t e_ = (expr);                                \
        if (e_ != hipSuccess) return BITS_E_HIP;               \
    } while (0)

namespace bits {

constexpr int kWave = 64;
constexpr uint32_t kMaxTreeNodes = 1u << BITS_MAX_DEPTH;   // per array, entry 0 unused

// ------------------------------------------------------------------ reductions

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        uint32_t olo = __shfl_xor(lo, o);
        uint32_t ohi = __shfl_xor(hi, o);
        uint32_t nlo = lo + olo;
        hi = hi + ohi + (nlo < lo ? 1u : 0u);
        lo = nlo;
    }
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ int32_t wave_max_i32(int32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
    return v;
}

// ------------------------------------------------------------------ Philox-4x32-10
// Counter-based generator of Salmon et al. (SC'11): ten rounds of two 32x32
// multiplies, word exchange and key xor, the key advancing by two Weyl
// increments after every round.
__device__ __forceinline__ void philox4x32_10(uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3,
                                              uint32_t k0, uint32_t k1) {
    // Each 32 x 32 -> 64 product is one v_mad_u64_u32 and each three-way xor one
    // v_bitop3 (truth table 0x96), four VALU instructions per round.
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u, p1 = (uint64_t)c2 * 0xCD9E8D57u;
        c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
        c1 = (uint32_t)p1;
        c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Start of a query's placement in shuffle s (Sec. 3.2): counter g = s * na + i
// (i the query's input index), key = the seed; the 64-bit draw u = (c1, c0)
// scaled to [0, span) by a high multiply, span > 0 being the number of legal
// starts of the query in its chromosome, which begins at `off`.
__device__ __forceinline__ uint32_t mc_place(uint64_t g, uint32_t k0, uint32_t k1, uint32_t off, uint32_t span) {
    uint32_t c0 = (uint32_t)g, c1 = (uint32_t)(g >> 32), c2 = 0u, c3 = 0u;
    philox4x32_10(c0, c1, c2, c3, k0, k1);
    const uint64_t u = ((uint64_t)c1 << 32) | c0;
    return off + (uint32_t)__umul64hi(u, (uint64_t)span);
}

// ------------------------------------------------------------------ search arguments

struct SearchArgs {
    const uint32_t* bs;          // sorted starts
    const uint32_t* be;          // sorted ends
    const uint32_t* tree;        // [2][tree_stride] Eytzinger splitters
    const bits_rmi_model* rmi;   // [2] learned models or nullptr
    const uint32_t* hs;          // line heads of B_S: hs[j] = bs[32 j], 0xFFFFFFFF past the end
    const uint32_t* he;          // line heads of B_E
    uint32_t* status;            // device status word
    unsigned long long* fallbacks;
    uint32_t n;                  // |B|
    uint32_t tree_stride;        // 2^built_depth
    uint32_t depth;              // levels searched from LDS (<= built depth)
    float mean_len;              // mean_length(), set by the kernels that use it
};

// Entries of one line-head array for n keys: ceil(n / 32) heads plus at
// least 32 entries of 0xFFFFFFFF, rounded up to whole 128-byte lines, so a
// 32-entry window starting at or before head ceil(n / 32) - 1 + 16 stays in bounds.
__host__ __device__ constexpr uint64_t heads_len(uint64_t n) { return ((n + 31) / 32 + 32 + 31) / 32 * 32; }

// Boundary rank of node k of an Eytzinger top tree over n keys (level
// l = floor(log2 k), j = k - 2^l): floor((2j + 1) n / 2^(l + 1)); the node
// holds the key before it, the last of the bucket on its left.
__host__ __device__ constexpr uint64_t tree_rank(uint32_t k, uint64_t n) {
    uint32_t l = 31u - (uint32_t)__builtin_clz(k);
    return ((2 * (uint64_t)(k - (1u << l)) + 1) * n) >> (l + 1);
}

// Number of LDS words a search kernel stages for depth d (both arrays).
__host__ __device__ constexpr uint32_t tree_lds_words(uint32_t d) { return d ? (2u << d) : 0u; }

// LDS scratch of the learned search per chain: (leaf, x) of 64 owners, then
// 6 result words per owner; per wave: 2 * QPL chains.
constexpr uint32_t kLeafScr = 2 * kWave + 6 * kWave;
__host__ __device__ constexpr uint32_t probe_scratch_words(int qpl) { return 2u * (uint32_t)qpl * kLeafScr; }

// Dynamic LDS of a search kernel: the top trees (plain) or the per-wave
// scratch (learned).
__host__ __device__ constexpr size_t search_lds_bytes(bool learned, uint32_t depth, int qpl, uint32_t block) {
    return learned ? (size_t)(block / kWave) * probe_scratch_words(qpl) * 4u : (size_t)tree_lds_words(depth) * 4u;
}

// Forms of the search kernels.  The path without a model (BITS_PATH_TIERED,
// and AUTO on a reference without one) takes kModeDirect up to kDirectKeys
// keys in buckets of at most kDirectBucket and kModeTiered else: a window of keys
// covers the whole bucket of a small reference, but misses as buckets grow, with
// the keys or with fewer levels of the tree (1e7 queries against 3e5 keys at
// depth 13, 12, 11, 10, 0: 188, 294, 313, 475, 2270 us, through the line heads
// 416, 407, 415, 406, 492; 1e6 against 1e5 at depth 13, 11, 10, 0: 29, 30, 38,
// 208 and 29, 30, 30, 29).
// AUTO takes the plain path up to kPlainKeys: the LDS tree then resolves all but
// a step or two (1.5e7 queries against 1e3 keys 81 us, 206 with windows; 8e3
// 155, 223; 1.6e4 205, 236; 6.4e4 455, 271); in query-ordered shuffles, which
// run over one part of the reference at a time and find it in the nearest
// caches, up to kPlainShuffleKeys (1e5 x 100 against 1.7e4, 5e4, 7e4, 1e5 keys
// 152, 164, 194, 265 us, with windows 234, 233, 232, 236; 1e6 x 30 against 7e4
// and 1e5 473 and 698, 584 and 585).  Counting through the models takes
// kModePaired up to kPairedKeys keys, kModeLearned above.
enum : int { kModePlain = 0, kModeLearned = 1, kModeTiered = 2, kModeDirect = 3, kModePaired = 4 };
__host__ __device__ constexpr bool learned_mode(int mode) { return mode == kModeLearned || mode == kModePaired; }
constexpr uint32_t kPlainKeys = 1u << 14;
constexpr uint32_t kPlainShuffleKeys = 1u << 16;
constexpr uint32_t kPairedKeys = 1u << 15;
constexpr uint32_t kDirectKeys = 1u << 19;
constexpr uint32_t kDirectBucket = 128;
__host__ __device__ constexpr bool direct_form(uint32_t n, uint32_t depth) {
    return n <= kDirectKeys && (n >> depth) <= kDirectBucket;
}

// Copy the first 2^d - 1 nodes of both trees into LDS: lds[0..2^d) starts,
// lds[2^d..2^(d+1)) ends, 1-based BFS order (slot 0 unused).
__device__ __forceinline__ void stage_tree(uint32_t* lds, const uint32_t* tree, uint32_t stride, uint32_t d) {
    if (!d) return;
    const uint32_t m = 1u << d;
    if (d < 2) {
        for (uint32_t k = threadIdx.x; k < m; k += blockDim.x) {
            lds[k] = tree[k];
            lds[m + k] = tree[stride + k];
        }
        return;
    }
    // 16 bytes a load (the trees are 256-byte aligned; m and stride are multiples of 4)
    const uint4* T0 = reinterpret_cast<const uint4*>(tree);
    const uint4* T1 = reinterpret_cast<const uint4*>(tree + stride);
    uint4* L = reinterpret_cast<uint4*>(lds);
    for (uint32_t k = threadIdx.x; k < m / 4; k += blockDim.x) {
        const uint4 a = T0[k], b = T1[k];
        L[k] = a;
        L[m / 4 + k] = b;
    }
}

// ------------------------------------------------------------------ learned index

__device__ __forceinline__ uint32_t rmi_route(float a, float b, uint32_t x) {
    float r = floorf(fmaf(a, (float)x, b));
    r = fminf(fmaxf(r, 0.0f), (float)(BITS_RMI_LEAVES - 1));
    return (uint32_t)r;
}

// Leaf prediction, in one fixed arithmetic order shared by the error-window
// measurement (sequential, rmi_pred_offset) and the queries (4 lanes per
// leaf, rmi_quad_partial + two lane-pair additions):
//   h_j = max(fma(w1_j, u, b1_j), 0),  s_q = fma-chain over j = 4q..4q+3 of w2_j h_j,
//   y   = b2 + ((s_0 + s_1) + (s_2 + s_3)).
__device__ __forceinline__ float rmi_quad_partial(const float* w1, const float* b1, const float* w2, float u) {
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) s = fmaf(w2[k], fmaxf(fmaf(w1[k], u, b1[k]), 0.0f), s);
    return s;
}

__device__ __forceinline__ int32_t rmi_offset_from_y(float y, uint32_t cnt) {
    float r = rintf(y * (float)cnt);
    r = fminf(fmaxf(r, 0.0f), (float)cnt);
    return (int32_t)r;
}

__device__ __forceinline__ float rmi_u(uint32_t dx, float kinv) { return (float)dx * kinv; }

// IEEE binary16 <-> fp32 (round to nearest even) for the stored leaf weights.
__device__ __forceinline__ float h2f(uint32_t bits) { return (float)__builtin_bit_cast(_Float16, (uint16_t)bits); }
__device__ __forceinline__ uint32_t f2h(float f) { return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)f); }

// Rank offset predicted inside a leaf for a key x with kmin <= x (dx = x - kmin);
// p holds the stored weights (w1, b1, w2 already rounded to binary16) and b2.
__device__ __forceinline__ int32_t rmi_pred_offset(const float* p, uint32_t cnt, float kinv, uint32_t dx) {
    const float u = rmi_u(dx, kinv);
    const float s0 = rmi_quad_partial(p + 0, p + 16, p + 32, u);
    const float s1 = rmi_quad_partial(p + 4, p + 20, p + 36, u);
    const float s2 = rmi_quad_partial(p + 8, p + 24, p + 40, u);
    const float s3 = rmi_quad_partial(p + 12, p + 28, p + 44, u);
    const float y = p[48] + ((s0 + s1) + (s2 + s3));
    return rmi_offset_from_y(y, cnt);
}

// ------------------------------------------------------------------ host launchers

struct LaunchCfg {
    uint32_t block, qpl, depth, grid, path;
    bool open = false;   // block and qpl were left to the library
};

int device_cu_count();
size_t device_lds_per_block();
int resolve_launch(const bits_ref* ref, const bits_launch* in, LaunchCfg* out);
SearchArgs make_search_args(const bits_ref* ref, const LaunchCfg& cfg);

// search.hip
hipError_t launch_fill_u64(unsigned long long* p, uint64_t n, unsigned long long v, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s);
// counts (nullable), firsts (nullable: #{B_S <= a.end} per query), total (nullable)
hipError_t launch_count(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                        uint64_t na, uint32_t* counts, unsigned long long* total, hipStream_t s,
                        uint32_t* firsts = nullptr);
// Monte-Carlo query table in the caller's workspace: uint32[na] each of
// chromosome offset, legal-start count, length and original index, grouped
// by chromosome; hist and cursor hold BITS_MAX_CHROM words each.
struct McTable {
    uint32_t *off, *span, *len, *idx, *hist, *cursor;
};
// Zeros of the outputs and (tab != nullptr) of the table's histogram and cursors.
hipError_t launch_mc_zero(unsigned long long* totals, uint64_t ns, unsigned long long* observed, const McTable* tab,
                          hipStream_t s);
// Fills the table (after launch_mc_zero).  packed != nullptr: uint2[na] of the
// binned path in place of off and len.  cursor[c] ends as the first table
// position past chromosome c, hist[c] as its number of queries.
hipError_t launch_mc_prepare(const uint32_t* as, const uint32_t* ae, uint64_t na, const uint32_t* chrom_len,
                             uint32_t n_chrom, const McTable& tab, void* packed, uint32_t* status, hipStream_t s);
hipError_t launch_mc(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                     const McTable& tab, uint64_t na, uint64_t seed, uint64_t s0, uint64_t nshuf,
                     unsigned long long* totals, unsigned long long* observed, hipStream_t s);
hipError_t launch_rmi_window(const SearchArgs& sa, uint32_t which, const uint32_t* xs, uint64_t n, uint32_t* lo,
                             uint32_t* hi, hipStream_t s);
hipError_t launch_decide(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                         uint64_t na, uint32_t* found, unsigned long long* witness, hipStream_t s);
hipError_t launch_select_u64(const unsigned long long* v, uint64_t n, uint64_t k0, uint64_t k1,
                             unsigned long long* out0, unsigned long long* out1, hipStream_t s);
// Rounds lie `stride` words apart, a multiple of 32 that is >= nb.
hipError_t launch_place_rounds(const McTable& tab, const uint32_t* b_start, uint64_t nb, uint64_t stride,
                               uint64_t seed, uint64_t s0, uint32_t rounds, bool identity, uint32_t* S, uint32_t* E,
                               hipStream_t s);
hipError_t launch_fill_tails(uint32_t* S, uint32_t* E, uint64_t nb, uint64_t stride, uint32_t rounds, hipStream_t s);
// Sorted rounds, 0xFFFFFFFF between nb and stride; trees and heads: scratch of
// `stride` words per round each.
hipError_t launch_count_rounds(const uint32_t* S, const uint32_t* E, uint64_t nb, uint64_t stride, uint32_t rounds,
                               uint32_t* trees, uint32_t* heads, const uint32_t* as, const uint32_t* ae, uint64_t na,
                               unsigned long long* totals, uint32_t* status, hipStream_t s);
// binned.hip: the Monte-Carlo path binned by genome region.
struct BinLayout {
    uint64_t ncells, nreg_max;
    uint32_t splits;              // search workgroups per region
};
// Cell count and an upper bound on the region count for a genome and |B| = n;
// false if the genome cannot be cut (sizes past 2^32).
bool bin_layout(const uint32_t* chrom_len, uint32_t n_chrom, uint64_t n, BinLayout* L);
struct BinWs {                    // device buffers, carved from the caller's workspace
    uint32_t *rs, *re;            // [ncells]
    uint64_t* nreg;               // [2]: number of regions, whether a chromosome is heavy
    uint32_t* cell_region;        // [ncells]
    void* desc;                   // [nreg_max + 1] region descriptors (16 bytes)
    uint32_t *seg_start, *seg_cnt;    // [batch][nreg_max]
    unsigned long long* partial;      // [nreg_max * splits][batch]
    void* recs;                       // [batch][na] {start, end}
    void* packed;                     // [na] {input index, length or 0}
    uint32_t nreg_max, splits;
};
hipError_t launch_bin_regions(const uint32_t* chrom_len, uint32_t n_chrom, const McTable& tab, uint64_t na, const uint32_t* bs, const uint32_t* be,
                              uint32_t n, const BinWs& w, uint32_t* status, hipStream_t s);
// Shuffles [sb, sb + nb) (absolute indices); totals points at shuffle sb's slot.
hipError_t launch_bin_batch(const uint32_t* chrom_len, uint32_t n_chrom, const McTable& tab, uint64_t na,
                            const uint32_t* bs, const uint32_t* be, uint32_t n, uint64_t seed, uint64_t sb,
                            uint32_t nb, const BinWs& w, unsigned long long* totals, hipStream_t s,
                            hipEvent_t* ev = nullptr);   // ev[4]: before binning, search, reduction, after
hipError_t launch_mc_tail(const unsigned long long* totals, uint64_t nshuf, const unsigned long long* observed,
                          unsigned long long* n_ge, unsigned long long* n_le, hipStream_t s);
hipError_t launch_project(const uint32_t* chrom_len, uint32_t n_chrom, const uint32_t* chrom,
                          const uint32_t* ls, const uint32_t* le, uint64_t n, uint32_t* gs, uint32_t* ge,
                          uint32_t* status, hipStream_t s);

// Batched pairs (search.hip)
struct BatchRef {        // one reference in the batch table
    const uint32_t* bs;
    const uint32_t* be;
    const uint32_t* tree;
    const bits_rmi_model* rmi;       // learned path: the two models (else nullptr)
    const uint32_t* hs;              // learned path: line heads of B_S and B_E
    const uint32_t* he;
    unsigned long long* fallbacks;   // the reference's learned-path fallback counter
    uint32_t n, tree_stride, depth, pad;
};
struct BatchQuery {
    const uint32_t* as;
    const uint32_t* ae;
    uint64_t n;
};
struct BatchItem {       // a tile of one query set against one reference
    uint32_t q, r, begin, count;
};
// cfg.path selects the plain (LDS tree + bisection) or the learned search for every pair;
// the learned path needs every reference learned.
hipError_t launch_batch(const BatchRef* refs, const BatchQuery* qs, const BatchItem* items,
                        const uint32_t* wg_begin, uint32_t n_wg, uint32_t n_ref, uint32_t max_depth,
                        const LaunchCfg& cfg, unsigned long long* pair_totals, uint32_t* status,
                        hipStream_t s);
int batch_blocks_per_cu(const LaunchCfg& cfg, uint32_t max_depth);

// merge.hip: every pair at once from sorted query keys.
constexpr uint64_t kMergeMaxKeys = 1ull << 26;           // query keys over all sets
constexpr uint32_t kMergeMaxSets = 192;                  // their accumulators (512 bytes each) fit the LDS
constexpr uint32_t kMergeMaxRefs = 4096;
constexpr uint64_t kMergeMinEvaluations = 1ull << 22;    // queries x references; fewer never pay for the sort
constexpr uint32_t kMergeCus = 256;
struct MergeLayout {
    uint32_t total, chunks, groups, wgs;
    size_t offs, in, sid, out, sets, splits, part, sort, sort_bytes, bytes;
};
// Workspace of the sorted form for these sets; false where only the search per pair is used.
bool merge_layout(const uint64_t* na, uint32_t n_q, uint32_t n_ref, MergeLayout* L);
// Whether the sorted form is expected to be the faster one against references of nb[j] keys.
bool merge_pays(const MergeLayout& L, const uint64_t* nb, uint32_t n_ref);
// offs (uint32[n_q + 1], the sets' first positions) is already in ws.
int launch_merge(const BatchRef* refs, uint32_t n_ref, const BatchQuery* qs, uint32_t n_q, const MergeLayout& L, void* ws,
                 unsigned long long* totals, uint32_t* status, hipStream_t s);

// sort.hip
// One segment to sort: n keys in -> out, optionally with one uint32 value per
// key moved along (vmode 1: values from vin; 2: the input index 0..n-1).
struct SortSeg {
    const uint32_t* in;
    uint32_t* out;
    uint64_t n;
    uint32_t vmode = 0;
    const uint32_t* vin = nullptr;
    uint32_t* vout = nullptr;
    // gets BITS_FLAG_SORT if a tile's look-back walk gave up (never expected; the
    // sorted output is then invalid); its first `clear` words (at most 256) are zeroed first
    uint32_t* status = nullptr;
    uint32_t clear = 0;
};
// The workspace for the tile these segments want, and the least one launch_sort
// accepts for them (larger tiles).
size_t sort_workspace_bytes(const uint64_t* n, uint32_t nseg, const uint32_t* vmode = nullptr);
size_t sort_workspace_least(const uint64_t* n, uint32_t nseg, const uint32_t* vmode = nullptr);
int launch_sort(const SortSeg* segs, uint32_t nseg, void* ws, size_t ws_bytes, hipStream_t s);
// Trees, line tails and (heads != nullptr) line heads of sorted references.
struct FinishRef {
    uint32_t* k[2];      // sorted starts and ends
    uint32_t* tree;      // [2][2^depth]
    uint32_t* heads;     // [2][heads_len(n)] or nullptr
    uint32_t n, depth;
};
constexpr uint32_t kFinishRefs = 64;   // references per launch (40 bytes of arguments each)
struct FinishChunk {
    FinishRef r[kFinishRefs];
};
hipError_t launch_finish_refs(const FinishRef* refs, uint32_t n_ref, hipStream_t s);

// enum.hip
uint64_t scan_tiles(uint64_t n);
hipError_t launch_gather_u32(const uint32_t* src, const uint32_t* idx, uint64_t n, uint32_t* dst, hipStream_t s);
hipError_t launch_scan_counts(const uint32_t* counts, uint64_t n, uint64_t* offsets, uint64_t* tile_sum,
                              hipStream_t s);
hipError_t launch_enumerate(const uint32_t* starts, const uint32_t* ends, const uint32_t* ids, uint32_t n,
                            const uint32_t* as, const uint32_t* ae, uint64_t na, const uint32_t* counts,
                            const uint32_t* firsts, const uint64_t* offsets, uint32_t* pa, uint32_t* pb,
                            uint64_t max_pairs, uint32_t* status, hipStream_t s);

// rmi.hip
size_t rmi_workspace_bytes();
// Also writes the line heads of both arrays (heads_len(n) words each).
int launch_rmi_build2(const uint32_t* keys0, const uint32_t* keys1, uint64_t n, bits_rmi_model* m0,
                      bits_rmi_model* m1, uint32_t* heads0, uint32_t* heads1, const bits_train& tr, void* ws,
                      hipStream_t s);
hipError_t launch_rmi_leaf_grad(const float* u, const float* t, uint32_t m, const float* params, float* grad,
                                float* loss, hipStream_t s);

}  // namespace bits
