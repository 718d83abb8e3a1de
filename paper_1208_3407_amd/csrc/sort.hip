// On-device LSD radix sort of uint32 keys (the two Sort steps of Algorithm 2)
// and the Eytzinger top-tree build.
//
// Segmented: every segment (e.g. B_S and B_E of one or many references) is
// sorted independently in the same launches, keys only or with one uint32
// value per key carried along (explicit, or the implicit 0..n-1 input order;
// the sort is stable, so equal keys keep their input order).  One read of
// the input counts all four 8-bit digits of every segment; then each pass is
// a single kernel over tiles taken in order from a counter: the tile ranks
// its keys by digit, publishes its digit counts, adds up the counts of the
// tiles before it in its segment by decoupled look-back (the nearest tile
// that has published its inclusive prefix ends the walk), and writes its keys
// out in digit runs.  Every key is read once and written once per pass.  A
// segment's digits that are constant over it are skipped (the tiles of the first
// pass work out the schedule from the segment's four histograms, so the sort
// never waits for the host and needs no launch for it).  Segments that fit
// one tile are sorted by one workgroup in LDS.  Inputs are never written.
#include <string.h>

#include <vector>

#include "bits_internal.hpp"

namespace bits {

namespace {

constexpr int kThreads = 256;                  // histogram, scan and copy kernels
constexpr int kWaves = kThreads / kWave;
constexpr int kSweepThreads = 1024;            // one pass of the sort
constexpr int kSweepWaves = kSweepThreads / kWave;
// A tile is ROUNDS rounds of 1024 keys held in registers, and a shape is taken
// from kWant* tiles on.  Few keys want many small tiles: at 20 rounds a tile
// takes 17 us however idle the chip is (index of 1e5 intervals: 105 us at 20
// rounds, 48 at 4; of 1e6: 107 at 4, 94 at 12).  Many keys want what two
// workgroups on a CU hold in 64 registers and 80 KB of LDS each, so that one
// ranks while the other waits for its loads, its look-back or its stores:
// index of 5e7 intervals 1738 us at 20 rounds (one workgroup a CU), 1551 at
// 10, 1446 at 12, 1520 at 14 (spills).  With values along, two workgroups hold
// 7 rounds (2e6 keys: 166 us at 4 rounds, 150 at 7, 159 at 16; 1e7: 677, 540,
// 543) until the look-back steps of many tiles cost more (2e7: 1121 at 7, 1040
// at 16).
constexpr int kRoundsKeys[3] = {4, 12, 20};
constexpr uint64_t kWantKeys[3] = {0, 110, ~0ull};   // 20 only where the workspace holds no smaller tiles' words
constexpr int kRoundsVals[3] = {4, 7, 16};
constexpr uint64_t kWantVals[3] = {0, 200, 730};
// A segment sorted by one workgroup.  At 16 rounds that takes longer (index of
// 1.6e4 intervals: 47 us) than small tiles on several CUs (2e4: 42 us).
constexpr uint32_t kLoneTile = 8u * kSweepThreads;
// Look-back words, one per (tile, digit): bits 0-31 the count, bits 32-39
// the pass (1 + p; 0 = not yet published in this call), bit 40 set once the
// count is the inclusive prefix over the segment's tiles up to this one
// (else it is the tile's own count).
constexpr uint64_t kLbPrefix = 1ull << 40;
// Polls of a predecessor's word before giving up (the walk cannot deadlock:
// tiles are taken in order, so every tile waited on is held by a running
// workgroup; the bound only turns a fault into BITS_FLAG_SORT, not a hang).
constexpr uint32_t kLbSpinLimit = 1u << 20;
constexpr int kLbBatch = 8;   // predecessor words loaded at once

struct SegDesc {
    const uint32_t* in;
    uint32_t* ping;
    uint32_t* out;
    uint32_t n;
    uint32_t tile0;   // first global tile of the segment
    const uint32_t* vin;   // values: input (nullptr with vmode 2: the input index)
    uint32_t* vping;
    uint32_t* vout;
    uint32_t vmode;   // 0 keys only, 1 values from vin, 2 values = input index
    uint32_t active;  // from the host: status words cleared before the sort; from pass 0 on: bit q
                      // set if pass q moves keys (digit q takes two or more values in the segment)
    uint32_t* status; // gets BITS_FLAG_SORT if a tile gave up its look-back walk (nullable)
};
static_assert(sizeof(SegDesc) == 72, "SegDesc layout");

struct SortPlan {
    uint32_t next_tile[4];   // tile counter of each pass
    uint32_t active;         // bit q: pass q moves the keys of some segment (set by pass 0)
};

constexpr int kDescChunk = 44;   // about 3 KB of kernel arguments
struct DescChunk {
    SegDesc d[kDescChunk];
};

__device__ __forceinline__ uint32_t seg_of_tile(const SegDesc* descs, uint32_t nseg, uint32_t t) {
    uint32_t lo = 0, hi = nseg;      // last s with tile0 <= t
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (descs[mid].tile0 <= t) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ const uint32_t* buf_ro(const SegDesc& d, uint32_t sel) {
    return sel == 0 ? d.in : sel == 1 ? d.ping : d.out;
}
__device__ __forceinline__ uint32_t* buf_rw(const SegDesc& d, uint32_t sel) {
    return sel == 1 ? d.ping : d.out;
}
__device__ __forceinline__ const uint32_t* vbuf_ro(const SegDesc& d, uint32_t sel) {
    return sel == 0 ? d.vin : sel == 1 ? d.vping : d.vout;
}
__device__ __forceinline__ uint32_t* vbuf_rw(const SegDesc& d, uint32_t sel) {
    return sel == 1 ? d.vping : d.vout;
}

// The sort's setup in one launch: a chunk of descriptors from the kernel
// arguments into the workspace, the status words the descriptors ask to
// clear, and with the first chunk the zeros (tile counters, histograms,
// look-back words) as uint4.
__global__ void __launch_bounds__(256) k_sort_init(SegDesc* dst, DescChunk chunk, uint32_t count, uint4* zero,
                                                   uint64_t nzero) {
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < count; i += blockDim.x) dst[i] = chunk.d[i];
        for (uint32_t i = 0; i < count; ++i)
            if (threadIdx.x < chunk.d[i].active) chunk.d[i].status[threadIdx.x] = 0u;
    }
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nzero; k += (uint64_t)gridDim.x * blockDim.x)
        zero[k] = make_uint4(0u, 0u, 0u, 0u);
}

// All four digit histograms of every segment in one read of the input.
// Workgroup b walks a contiguous range of tiles, accumulating in LDS and
// flushing when the segment changes.
__global__ void __launch_bounds__(kThreads) k_hist_all(const SegDesc* __restrict__ descs, uint32_t nseg,
                                                       uint32_t ntiles, uint32_t tile,
                                                       uint32_t* __restrict__ seg_hist) {
    __shared__ uint32_t h[4][256];
    const uint32_t t0 = (uint32_t)((uint64_t)ntiles * blockIdx.x / gridDim.x);
    const uint32_t t1 = (uint32_t)((uint64_t)ntiles * (blockIdx.x + 1) / gridDim.x);
    for (int k = threadIdx.x; k < 1024; k += kThreads) (&h[0][0])[k] = 0;
    __syncthreads();
    uint32_t cur = 0xFFFFFFFFu;
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t s = seg_of_tile(descs, nseg, t);
        if (s != cur) {
            if (cur != 0xFFFFFFFFu) {
                __syncthreads();
                for (int k = threadIdx.x; k < 1024; k += kThreads) {
                    const uint32_t v = (&h[0][0])[k];
                    if (v) atomicAdd(seg_hist + (size_t)cur * 1024 + k, v);
                    (&h[0][0])[k] = 0;
                }
                __syncthreads();
            }
            cur = s;
        }
        const SegDesc d = descs[s];
        const uint32_t begin = (t - d.tile0) * tile;
        const uint32_t cnt = min(tile, d.n - begin);
        const uint32_t* src = d.in + begin;
        // four independent loads per thread in flight, then their counts
        for (uint32_t k0 = threadIdx.x; k0 < cnt; k0 += 4 * kThreads) {
            uint32_t key[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t k = k0 + (uint32_t)u * kThreads;
                key[u] = src[min(k, cnt - 1u)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (k0 + (uint32_t)u * kThreads >= cnt) break;
                atomicAdd(&h[0][key[u] & 255u], 1u);
                atomicAdd(&h[1][(key[u] >> 8) & 255u], 1u);
                atomicAdd(&h[2][(key[u] >> 16) & 255u], 1u);
                atomicAdd(&h[3][key[u] >> 24], 1u);
            }
        }
    }
    __syncthreads();
    if (cur != 0xFFFFFFFFu) {
        for (int k = threadIdx.x; k < 1024; k += kThreads) {
            const uint32_t v = (&h[0][0])[k];
            if (v) atomicAdd(seg_hist + (size_t)cur * 1024 + k, v);
        }
    }
}

// The look-back word of (tile, digit).
__device__ __forceinline__ unsigned long long* lb_word(unsigned long long* lb, uint32_t ntiles, uint32_t tile,
                                                      uint32_t dg) {
    return lb + (size_t)tile * 256 + dg;
}

// Exclusive prefix over the first 256 threads of two values at once (the low
// and the high word of v; neither sum reaches 2^32).  All threads call it.
__device__ __forceinline__ uint64_t excl_scan_256(uint64_t v, uint64_t* tmp) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint64_t x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint64_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (w < 4 && lane == kWave - 1) tmp[w] = x;
    __syncthreads();
    uint64_t pre = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (k < w) pre += tmp[k];
    return pre + x - v;
}

// Rank of each of a wave's keys among the keys of its digit seen so far by
// the wave (register round r holds keys [w ROUNDS + r] 64 .. + 63 of the tile), and in
// wcnt[w] the wave's digit counts.  Within a round, lanes holding the same
// digit are found with 8 ballots (each folded into the lane's peer mask by
// one v_bitop3 per half) and ranked by lane order.
template <int ROUNDS>
__device__ __forceinline__ void rank_keys(const uint32_t (&key)[ROUNDS], uint32_t cnt, uint32_t shift,
                                          uint32_t (*wcnt)[256], uint32_t (&rank)[ROUNDS]) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
        const bool valid = idx < cnt;
        const uint32_t dg = (key[r] >> shift) & 255u;
        const uint64_t pv = __ballot(valid);
        uint32_t plo = (uint32_t)pv, phi = (uint32_t)(pv >> 32);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t sb = 0u - ((dg >> b) & 1u);   // all ones where the bit is set
            const uint64_t m = __ballot(sb != 0u);
            // peers &= bit ? m : ~m, i.e. peers & ~(m ^ sb): one v_bitop3 per half
            plo = __builtin_amdgcn_bitop3_b32(plo, (uint32_t)m, sb, 0x90);
            phi = __builtin_amdgcn_bitop3_b32(phi, (uint32_t)(m >> 32), sb, 0x90);
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
        uint32_t old = 0;
        if (valid) old = wcnt[w][dg];
        rank[r] = old + before;
        if (valid && before == 0) wcnt[w][dg] = old + (uint32_t)(__popc(plo) + __popc(phi));
        __builtin_amdgcn_wave_barrier();
    }
}

// One pass of the sort over one tile (taken from the pass's counter).  Wave
// w ranks keys [w ROUNDS 64, (w + 1) ROUNDS 64) of the tile.  The tile's digit
// counts are published, the exclusive prefix over the segment's earlier tiles
// is gathered by look-back (one thread per digit), and the tile, sorted by
// digit in LDS, is written out in digit runs.  Pass 0 copies a segment whose
// keys are all equal.
// Eight waves per SIMD (two workgroups a CU) up to 12 rounds.
template <bool VALS, int ROUNDS>
__global__ void __launch_bounds__(kSweepThreads, ROUNDS <= 12 ? 8 : 4) k_onesweep(SegDesc* __restrict__ descs, uint32_t nseg,
                                                            SortPlan* plan, int p,
                                                            unsigned long long* __restrict__ lb, uint32_t ntiles,
                                                            const uint32_t* __restrict__ seg_hist) {
    constexpr uint32_t kTile = ROUNDS * kSweepThreads;
    __shared__ uint32_t keys_lds[kTile];
    __shared__ uint32_t vals_lds[VALS ? kTile : 1];
    __shared__ uint32_t wcnt[kSweepWaves][256];
    __shared__ uint32_t dstart[256];
    __shared__ uint32_t goff[256];
    __shared__ uint64_t tmp[4];
    __shared__ uint32_t nzc[kSweepWaves];
    __shared__ uint32_t tile_sh;
    if (p != 0 && !((plan->active >> p) & 1u)) return;
    if (threadIdx.x == 0) tile_sh = atomicAdd(&plan->next_tile[p], 1u);
    for (int k = threadIdx.x; k < kSweepWaves * 256; k += kSweepThreads) (&wcnt[0][0])[k] = 0;
    __syncthreads();
    const uint32_t t = tile_sh;
    const uint32_t s = seg_of_tile(descs, nseg, t);
    const SegDesc d = descs[s];
    const uint32_t begin = (t - d.tile0) * kTile;
    const uint32_t cnt = min(kTile, d.n - begin);
    const uint32_t shift = 8u * p;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t dg = threadIdx.x;
    // The schedule: pass q is active when digit q takes two or more values in the segment;
    // the last active pass writes the output, earlier ones alternate so that the first
    // reads the input.  Pass 0 works it out while its keys arrive, and leaves it in the
    // descriptor for the later ones, which then read the right buffer or nothing (with the
    // keys of every pass loaded on the usual schedule, an index of 3e7 keys of one digit took
    // 1090 us, 880 so, and one of 3e7 starts over the genome 910, 860).
    const uint32_t hp = dg < 256 ? seg_hist[((size_t)s * 4 + p) * 256 + dg] : 0u;
    uint32_t act = d.active;
    if (p != 0 && !((act >> p) & 1u)) return;
    const uint32_t na_ = (uint32_t)__popc(act), r_ = (uint32_t)__popc(act & ((1u << p) - 1u));
    uint32_t to = ((na_ - 1u - r_) & 1u) ? 1u : 2u, from = p == 0 || r_ == 0u ? 0u : 3u - to;
    uint32_t key[ROUNDS], rank[ROUNDS];
    const uint32_t* src = buf_ro(d, from) + begin;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
        key[r] = idx < cnt ? src[idx] : 0u;
    }
    if (p == 0) {
        const uint32_t hv = seg_hist[(size_t)s * 1024 + threadIdx.x];   // digit dg & 255 of pass dg / 256
        const uint64_t nz = __ballot(hv != 0u);
        if (lane == 0) nzc[w] = (uint32_t)__popcll(nz);
        __syncthreads();
        act = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (nzc[4 * q] + nzc[4 * q + 1] + nzc[4 * q + 2] + nzc[4 * q + 3] >= 2u) act |= 1u << q;
        if (threadIdx.x == 0 && t == d.tile0) {
            descs[s].active = act;
            atomicOr(&plan->active, act);
        }
        if (!act) {   // all keys equal: already sorted
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
                if (idx >= cnt) continue;
                d.out[begin + idx] = key[r];
                if (VALS && d.vmode) d.vout[begin + idx] = d.vmode == 2 ? begin + idx : d.vin[begin + idx];
            }
        }
        if (!(act & 1u)) return;
        to = (__popc(act) - 1) & 1 ? 1u : 2u;
    }
    uint32_t* dst = buf_rw(d, to);
    // values: vmode 2 reads the input index on the first active pass
    const bool vals = VALS && d.vmode != 0;
    const bool iota = d.vmode == 2 && from == 0;
    const uint32_t* vsrc = vals && !iota ? vbuf_ro(d, from) + begin : nullptr;
    uint32_t* vdst = vals ? vbuf_rw(d, to) : nullptr;
    rank_keys<ROUNDS>(key, cnt, shift, wcnt, rank);
    __syncthreads();
    // per digit: wave offsets within the tile, the tile's count, published at once
    uint32_t tot = 0;
    const unsigned long long tag = (unsigned long long)(p + 1) << 32;
    if (dg < 256) {
#pragma unroll
        for (int k = 0; k < kSweepWaves; ++k) {
            const uint32_t c = wcnt[k][dg];
            wcnt[k][dg] = tot;
            tot += c;
        }
        __hip_atomic_store(lb_word(lb, ntiles, t, dg), (d.tile0 == t ? kLbPrefix : 0ull) | tag | tot, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    // tile offset of the digit (low word) and its first place in the segment (high word)
    const uint64_t both = excl_scan_256(((uint64_t)hp << 32) | tot, tmp);
    const uint32_t ds = (uint32_t)both;
    if (dg < 256) {
        // wave offsets become tile offsets: each key then needs one LDS read
        dstart[dg] = ds;
#pragma unroll
        for (int k = 0; k < kSweepWaves; ++k) wcnt[k][dg] += ds;
    }
    __syncthreads();
    // the tile sorted by digit in LDS (needs only tile-local offsets)
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)k) * kWave + lane;
        if (idx < cnt) {
            const uint32_t kd = (key[k] >> shift) & 255u;
            const uint32_t at = wcnt[w][kd] + rank[k];
            keys_lds[at] = key[k];
            if constexpr (VALS) {
                if (vals) vals_lds[at] = iota ? begin + idx : vsrc[idx];
            }
        }
    }
    if (dg < 256) {
        // look-back over the segment's earlier tiles, kLbBatch words loaded at
        // once (independent loads), then taken nearest first: a word not yet
        // published is polled until it is; the walk ends at an inclusive prefix
        uint32_t excl = 0;
        if (t != d.tile0) {
            uint32_t tp = t - 1;
            uint32_t spins = 0;
            bool done = false;
            while (!done) {
                unsigned long long v[kLbBatch];
#pragma unroll
                for (int k = 0; k < kLbBatch; ++k) {
                    const uint32_t tk = tp >= d.tile0 + (uint32_t)k ? tp - (uint32_t)k : d.tile0;
                    v[k] = __hip_atomic_load(lb_word(lb, ntiles, tk, dg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int k = 0; k < kLbBatch; ++k) {
                    if (done) break;
                    const uint32_t tk = tp - (uint32_t)k;
                    while ((v[k] & (0xFFull << 32)) != tag) {
                        if (++spins > kLbSpinLimit) {
                            if (d.status) atomicOr(d.status, BITS_FLAG_SORT);
                            v[k] = kLbPrefix | tag;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
                        v[k] = __hip_atomic_load(lb_word(lb, ntiles, tk, dg), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                    }
                    excl += (uint32_t)v[k];
                    done = (v[k] & kLbPrefix) || tk == d.tile0;
                }
                tp -= kLbBatch;
            }
            __hip_atomic_store(lb_word(lb, ntiles, t, dg), kLbPrefix | tag | (excl + tot), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        goff[dg] = (uint32_t)(both >> 32) + excl;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < cnt; k += kSweepThreads) {
        const uint32_t v = keys_lds[k];
        const uint32_t kd = (v >> shift) & 255u;
        const uint32_t at = goff[kd] + (k - dstart[kd]);
        dst[at] = v;
        if constexpr (VALS) {
            if (vals) vdst[at] = vals_lds[k];
        }
    }
}

// A segment of at most ROUNDS * 1024 keys, sorted by one workgroup: the four
// passes go through LDS.  Workgroup b sorts segment b.
template <bool VALS, int ROUNDS>
__global__ void __launch_bounds__(kSweepThreads) k_sort_lone(const SegDesc* __restrict__ descs) {
    constexpr uint32_t kTile = ROUNDS * kSweepThreads;
    __shared__ uint32_t keys_lds[kTile];
    __shared__ uint32_t vals_lds[VALS ? kTile : 1];
    __shared__ uint32_t wcnt[kSweepWaves][256];
    __shared__ uint64_t tmp[4];
    const SegDesc d = descs[blockIdx.x];
    const uint32_t cnt = d.n, dg = threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const bool vals = VALS && d.vmode != 0;
    uint32_t key[ROUNDS], val[VALS ? ROUNDS : 1], rank[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
        key[r] = idx < cnt ? d.in[idx] : 0u;
        if constexpr (VALS) val[r] = d.vmode == 1 && idx < cnt ? d.vin[idx] : idx;
    }
#pragma unroll 1
    for (uint32_t p = 0; p < 4; ++p) {
        const uint32_t shift = 8u * p;
        for (int k = threadIdx.x; k < kSweepWaves * 256; k += kSweepThreads) (&wcnt[0][0])[k] = 0;
        __syncthreads();
        rank_keys<ROUNDS>(key, cnt, shift, wcnt, rank);
        __syncthreads();
        uint32_t tot = 0;
        if (dg < 256) {
#pragma unroll
            for (int k = 0; k < kSweepWaves; ++k) {
                const uint32_t c = wcnt[k][dg];
                wcnt[k][dg] = tot;
                tot += c;
            }
        }
        const uint32_t ds = (uint32_t)excl_scan_256(tot, tmp);
        if (dg < 256) {
#pragma unroll
            for (int k = 0; k < kSweepWaves; ++k) wcnt[k][dg] += ds;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
            if (idx < cnt) {
                const uint32_t at = wcnt[w][(key[r] >> shift) & 255u] + rank[r];
                keys_lds[at] = key[r];
                if constexpr (VALS) vals_lds[at] = val[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
            if (idx < cnt) {
                key[r] = keys_lds[idx];
                if constexpr (VALS) val[r] = vals_lds[idx];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t idx = ((uint32_t)w * ROUNDS + (uint32_t)r) * kWave + lane;
        if (idx < cnt) {
            d.out[idx] = key[r];
            if constexpr (VALS) {
                if (vals) d.vout[idx] = val[r];
            }
        }
    }
}

// The rest of reference indexes over their sorted arrays, one launch for up to
// kFinishRefs references (blockIdx.y): the top trees (node k holds
// keys[tree_rank(k, n) - 1]; the first 2^d - 1 nodes form the depth-d tree for
// every d <= depth), 0xFFFFFFFF after the keys up to the end of the last
// 128-byte line, and unless the learned build writes them the line heads
// (the first key of every line, then 0xFFFFFFFF).
__global__ void __launch_bounds__(256) k_finish_refs(FinishChunk F) {
    const FinishRef R = F.r[blockIdx.y];
    const uint32_t m = 1u << R.depth, lines = (uint32_t)(((uint64_t)R.n + 31) / 32);
    const uint32_t hl = R.heads ? (uint32_t)heads_len(R.n) : 0u, tail = (uint32_t)((uint64_t)lines * 32 - R.n);
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < 2u * (m + tail + hl); t += gridDim.x * blockDim.x) {
        if (t < 2u * m) {
            const uint32_t k = t & (m - 1u);
            R.tree[t] = k && R.n ? R.k[t < m ? 0 : 1][tree_rank(k, R.n) - 1] : 0u;
        } else if (t < 2u * (m + tail)) {
            const uint32_t k = t - 2u * m, a = k >= tail ? 1u : 0u;
            R.k[a][(uint64_t)R.n + (k - a * tail)] = 0xFFFFFFFFu;
        } else {
            const uint32_t k = t - 2u * (m + tail), a = k >= hl ? 1u : 0u, j = k - a * hl;
            R.heads[k] = j < lines ? R.k[a][32u * (uint64_t)j] : 0xFFFFFFFFu;
        }
    }
}

struct WsLayout {
    size_t descs, plan, seg_hist, lb, zero_end, ping, vping, total;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The tile a sort takes, from its segments' sizes.
constexpr int kShapes = 3;
struct SortShape {
    bool vals, lone;   // lone: every segment fits one workgroup
    int k, rounds;
    uint64_t ntiles;
};

static uint64_t tiles_at(const uint64_t* n, uint32_t nseg, int rounds) {
    const uint64_t tile = (uint64_t)rounds * kSweepThreads;
    uint64_t t = 0;
    for (uint32_t s = 0; s < nseg; ++s) t += (n[s] + tile - 1) / tile;
    return t;
}

// Tile k of the list that fits the segments; k < 0: the one wanted for their sizes.
static SortShape sort_shape(const uint64_t* n, uint32_t nseg, const uint32_t* vmode, int k = -1) {
    SortShape S{false, true, 0, 0, 0};
    uint64_t most = 0;
    for (uint32_t s = 0; s < nseg; ++s) {
        S.vals |= vmode && vmode[s];
        most = n[s] > most ? n[s] : most;
    }
    S.lone = most <= kLoneTile;
    const int* R = S.vals ? kRoundsVals : kRoundsKeys;
    const uint64_t* want = S.vals ? kWantVals : kWantKeys;
    if (k < 0) {
        k = kShapes - 1;
        while (k > 0 && tiles_at(n, nseg, R[k]) < want[k]) --k;
    }
    S.k = k;
    S.rounds = R[k];
    if (S.lone) S.rounds = most <= 4u * kSweepThreads ? 4 : 8;
    S.ntiles = tiles_at(n, nseg, S.rounds);
    return S;
}

static WsLayout ws_layout(const uint64_t* n, uint32_t nseg, const uint32_t* vmode, const SortShape& S) {
    uint64_t nkeys = 0, nvals = 0;
    for (uint32_t s = 0; s < nseg; ++s) {
        nkeys += n[s];
        if (vmode && vmode[s]) nvals += n[s];
    }
    WsLayout L;
    size_t o = 0;
    // cleared by the first launch: [plan, zero_end)
    L.plan = o; o = align256(o + sizeof(SortPlan));
    L.seg_hist = o; o = align256(o + (S.lone ? 0 : (size_t)nseg * 1024 * 4));
    L.lb = o; o = align256(o + (S.lone ? 0 : (size_t)S.ntiles * 256 * 8));
    L.zero_end = S.lone ? L.lb : L.lb + (size_t)S.ntiles * 256 * 8;
    L.descs = o; o = align256(o + sizeof(SegDesc) * nseg);
    L.ping = o; o = align256(o + (S.lone ? 0 : (size_t)nkeys * 4));
    L.vping = o; o = align256(o + (S.lone ? 0 : (size_t)nvals * 4));
    L.total = o;
    return L;
}

// The tile wanted for the segments, or the next larger one whose look-back
// words the workspace holds: a caller may have sized it for other segments, or
// for larger tiles (20 rounds of keys: an index of 5e7 1738 us, 1446 at 12).
static SortShape sort_shape_in(const uint64_t* n, uint32_t nseg, const uint32_t* vmode, size_t ws_bytes) {
    SortShape S = sort_shape(n, nseg, vmode);
    while (S.k + 1 < kShapes && ws_layout(n, nseg, vmode, S).total > ws_bytes) S = sort_shape(n, nseg, vmode, S.k + 1);
    return S;
}

}  // namespace

size_t sort_workspace_bytes(const uint64_t* n, uint32_t nseg, const uint32_t* vmode) {
    return ws_layout(n, nseg, vmode, sort_shape(n, nseg, vmode)).total;
}

size_t sort_workspace_least(const uint64_t* n, uint32_t nseg, const uint32_t* vmode) {
    return ws_layout(n, nseg, vmode, sort_shape(n, nseg, vmode, kShapes - 1)).total;
}

template <bool VALS, int ROUNDS>
static void launch_passes(SegDesc* descs, uint32_t nseg, SortPlan* plan, unsigned long long* lb, uint32_t ntiles,
                          const uint32_t* seg_hist, hipStream_t s) {
    for (int p = 0; p < 4; ++p)
        hipLaunchKernelGGL((k_onesweep<VALS, ROUNDS>), dim3(ntiles), dim3(kSweepThreads), 0, s, descs, nseg, plan, p, lb,
                           ntiles, seg_hist);
}

int launch_sort(const SortSeg* segs, uint32_t nseg, void* ws, size_t ws_bytes, hipStream_t s) {
    std::vector<uint64_t> ns(nseg);
    std::vector<uint32_t> vm(nseg);
    for (uint32_t i = 0; i < nseg; ++i) {
        if (segs[i].n > 0xFFFFFFFFull || segs[i].vmode > 2) return BITS_E_ARG;
        if ((segs[i].vmode == 1 && !segs[i].vin) || (segs[i].vmode && !segs[i].vout)) return BITS_E_ARG;
        ns[i] = segs[i].n;
        vm[i] = segs[i].vmode;
    }
    const SortShape S = sort_shape_in(ns.data(), nseg, vm.data(), ws_bytes);
    const WsLayout L = ws_layout(ns.data(), nseg, vm.data(), S);
    const uint32_t tile = (uint32_t)S.rounds * kSweepThreads;
    if (ws_bytes < L.total) return BITS_E_WORKSPACE;
    char* base = (char*)ws;
    SegDesc* descs = (SegDesc*)(base + L.descs);
    SortPlan* plan = (SortPlan*)(base + L.plan);
    uint32_t* seg_hist = (uint32_t*)(base + L.seg_hist);
    unsigned long long* lb = (unsigned long long*)(base + L.lb);
    uint32_t* ping = (uint32_t*)(base + L.ping);
    uint32_t* vping = (uint32_t*)(base + L.vping);

    // Descriptors, written by small kernels from by-value chunks so the call
    // stays asynchronous and capturable.
    uint32_t tile0 = 0;
    uint64_t koff = 0, voff = 0;
    for (uint32_t c0 = 0; c0 < nseg; c0 += kDescChunk) {
        DescChunk ch;
        memset(&ch, 0, sizeof(ch));
        const uint32_t cnt = (nseg - c0) < (uint32_t)kDescChunk ? (nseg - c0) : (uint32_t)kDescChunk;
        for (uint32_t i = 0; i < cnt; ++i) {
            const SortSeg& g = segs[c0 + i];
            ch.d[i].in = g.in;
            ch.d[i].out = g.out;
            ch.d[i].ping = ping + koff;
            ch.d[i].n = (uint32_t)g.n;
            ch.d[i].tile0 = tile0;
            ch.d[i].vmode = g.vmode;
            ch.d[i].status = g.status;
            ch.d[i].active = g.clear;
            if (g.vmode) {
                ch.d[i].vin = g.vmode == 1 ? g.vin : nullptr;
                ch.d[i].vping = vping + voff;
                ch.d[i].vout = g.vout;
                voff += g.n;
            }
            tile0 += (uint32_t)((g.n + tile - 1) / tile);
            koff += g.n;
        }
        const uint64_t nzero = c0 == 0 && !S.lone ? (L.zero_end - L.plan) / 16 : 0;
        const uint64_t gz = (nzero + 255) / 256;
        hipLaunchKernelGGL(k_sort_init, dim3((uint32_t)(gz < 1 ? 1 : gz > 2048 ? 2048 : gz)), dim3(256), 0, s,
                           descs + c0, ch, cnt, (uint4*)(base + L.plan), nzero);
    }
    const uint32_t ntiles = tile0;
    if (ntiles == 0) {
        BITS_CHECK_HIP(hipGetLastError());
        return BITS_OK;
    }
    if (S.lone) {
        if (S.vals && S.rounds == 4)
            hipLaunchKernelGGL((k_sort_lone<true, 4>), dim3(nseg), dim3(kSweepThreads), 0, s, descs);
        else if (S.vals)
            hipLaunchKernelGGL((k_sort_lone<true, 8>), dim3(nseg), dim3(kSweepThreads), 0, s, descs);
        else if (S.rounds == 4)
            hipLaunchKernelGGL((k_sort_lone<false, 4>), dim3(nseg), dim3(kSweepThreads), 0, s, descs);
        else
            hipLaunchKernelGGL((k_sort_lone<false, 8>), dim3(nseg), dim3(kSweepThreads), 0, s, descs);
        BITS_CHECK_HIP(hipGetLastError());
        return BITS_OK;
    }
    const uint32_t hg = ntiles < 2048u ? ntiles : 2048u;
    hipLaunchKernelGGL(k_hist_all, dim3(hg), dim3(kThreads), 0, s, descs, nseg, ntiles, tile, seg_hist);
    if (S.vals) {
        if (S.rounds == kRoundsVals[0]) launch_passes<true, kRoundsVals[0]>(descs, nseg, plan, lb, ntiles, seg_hist, s);
        else if (S.rounds == kRoundsVals[1]) launch_passes<true, kRoundsVals[1]>(descs, nseg, plan, lb, ntiles, seg_hist, s);
        else launch_passes<true, kRoundsVals[2]>(descs, nseg, plan, lb, ntiles, seg_hist, s);
    } else {
        if (S.rounds == kRoundsKeys[0]) launch_passes<false, kRoundsKeys[0]>(descs, nseg, plan, lb, ntiles, seg_hist, s);
        else if (S.rounds == kRoundsKeys[1]) launch_passes<false, kRoundsKeys[1]>(descs, nseg, plan, lb, ntiles, seg_hist, s);
        else launch_passes<false, kRoundsKeys[2]>(descs, nseg, plan, lb, ntiles, seg_hist, s);
    }
    BITS_CHECK_HIP(hipGetLastError());
    return BITS_OK;
}

hipError_t launch_finish_refs(const FinishRef* refs, uint32_t n_ref, hipStream_t s) {
    for (uint32_t j0 = 0; j0 < n_ref; j0 += kFinishRefs) {
        FinishChunk F;
        memset(&F, 0, sizeof(F));
        const uint32_t cnt = n_ref - j0 < kFinishRefs ? n_ref - j0 : kFinishRefs;
        uint64_t most = 0;
        for (uint32_t i = 0; i < cnt; ++i) {
            F.r[i] = refs[j0 + i];
            const uint64_t words = (2ull << refs[j0 + i].depth) + 64 + (refs[j0 + i].heads ? 2 * heads_len(refs[j0 + i].n) : 0);
            most = words > most ? words : most;
        }
        const uint64_t g = (most + 255) / 256;
        hipLaunchKernelGGL(k_finish_refs, dim3((uint32_t)(g < 4096 ? g : 4096), cnt), dim3(256), 0, s, F);
    }
    return hipGetLastError();
}

}  // namespace bits
