// Monte-Carlo shuffles binned by genome region (Sec. 3.2) for gfx950.
//
// A shuffle's total is a sum over its placements of first - last (Algorithm 1),
// so the placements may be counted in any order.  This path orders them by
// region of the genome, so that the slice of B_S and B_E a region needs is
// read from HBM once per batch of shuffles into LDS and every search runs in
// LDS, with no per-search memory request:
//   regions  each chromosome is cut into cells of 2^S bp; a region is a run of
//            consecutive cells of one chromosome, cut where the merged count of
//            B_S and B_E keys since the chromosome's start crosses a multiple
//            of kRegionKeys, so regions follow B's density;
//   binning  per (shuffle, chromosome): the placements of the chromosome's
//            queries are made (the Philox stream of the other Monte-Carlo
//            kernels), counted per region, made again and written, with their
//            ends, in region order: one segment per (shuffle, region).  When
//            the chromosome has many regions, the second sweep goes in chunks
//            that are counting-sorted by region in LDS and written out in
//            region runs, so that a record line is filled in one go;
//   search   per region (or per share of a region's records when regions
//            are few): both slices are staged in LDS (B_S with kMargin keys
//            past the region's end, for ends that cross it), with a table of
//            slice ranks at equally spaced coordinates (a piecewise-constant
//            CDF of the slice), and each placement of each shuffle of the
//            batch is counted by two table lookups, each followed by a
//            comparison with the few keys of its bucket, all in LDS; the
//            per-shuffle sums are written out;
//   reduce   per shuffle: the sums over regions (and shares) are added to the
//            totals.
// A region whose slices exceed the LDS capacity (very dense or duplicated
// keys) is searched in HBM by the same bisections; an end past the staged
// margin continues by galloping search in HBM.  Both only cost speed.
#include <algorithm>

#include "bits_internal.hpp"

namespace bits {

namespace {

constexpr uint32_t kMaxCells = 8192;       // cells per chromosome (LDS table of the binning kernel)
constexpr uint32_t kMinShift = 10;         // cells are at least 1 kbp
constexpr uint32_t kRegionKeys = 8192;     // merged B_S + B_E keys per region (target)
constexpr uint32_t kMargin = 256;          // B_S keys staged past a region's end
constexpr uint32_t kSliceWords = 12800;    // LDS slice capacity of the search kernel (50 KiB)
// Bucket tables of the search kernel: a region's coordinate range is cut into
// at most kBuckets equal buckets; entry b of a table (16 bits: a slice has
// fewer than 2^16 keys) is the number of slice keys in the buckets before b
// (b = 0 .. buckets, the last one closing the final bucket).
constexpr uint32_t kBuckets = 3072;
// Keys compared from a bucket's first on: kFirstKeys by every lane, the others
// by the lanes whose first ones all count, and past kBucketKeys (as many words
// of 0xFFFFFFFF follow each slice) a bisection.  LDS bank conflicts price each
// word a full wave reads: six by every lane took 1.5 times the LDS cycles.
constexpr uint32_t kFirstKeys = 2, kBucketKeys = 5;
// Record loads a wave of the search keeps in flight.  One is too few: 29 waves
// a CU x 512 B x 256 CUs in about 2 us is what the search then read per second.
// 1e9 records, all passes: 1, 2, 3, 4, 6 loads 3860, 3470, 3360, 3310, 3280 us.
constexpr uint32_t kAhead = 4;
// Records per shuffle of a region from which a wave walks the shuffles with
// scalars, each end costing it an LDS read's wait; with fewer, every lane looks
// for itself (1000 queries x 2200 against 2.3e6, two a region and shuffle: 453
// and 264 us; at 82 both take 3.31 ms for 1e9).
constexpr uint32_t kWalkRecords = 64;
static_assert(kSliceWords < (1u << 16), "slice ranks are 16-bit");
constexpr uint32_t kBinThreads = 1024;
constexpr int ILP = 4;   // table entries each binning thread loads before it places them
// A reference with few regions (a small B) would leave most of the chip idle
// in the search; each region's records are then split over up to kMaxSplits
// workgroups, aiming at kSearchWorkgroups per pass.
constexpr uint32_t kSearchWorkgroups = 2048;
constexpr uint32_t kMaxSplits = 16;

// Per-chromosome geometry, passed by value: off[k] = first coordinate of
// chromosome k (off[n] = genome size), cb[k] = its first cell (cb[n] = cells).
struct BinGeom {
    uint32_t n_chrom, shift;
    uint32_t off[BITS_MAX_CHROM + 1];
    uint32_t cb[BITS_MAX_CHROM + 1];
};

// The first key of region r, and #{B_S < key_lo}, #{B_E < key_lo}.
struct RegionDesc {
    uint32_t key_lo, s_lo, e_lo, pad;
};

__device__ __forceinline__ uint32_t chrom_of_cell(const BinGeom& g, uint32_t c) {
    uint32_t lo = 0, hi = g.n_chrom;   // last k with cb[k] <= c (chromosomes without cells are skipped)
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (g.cb[mid] <= c) lo = mid; else hi = mid;
    }
    return lo;
}

// #{K[0..m) < x} (STRICT) or #{K[0..m) <= x}; the same number of steps for
// every lane at a given m.  (Staging the slices with a spare word per 32
// keys spreads the probes over more LDS banks, but its two extra VALU
// operations per probe cost more than the conflicts it saves.)
template <bool STRICT>
__device__ __forceinline__ uint32_t rank_in(const uint32_t* K, uint32_t m, uint32_t x) {
    if (m == 0) return 0;
    uint32_t base = 0, len = m;
    while (len > 1) {
        const uint32_t half = len >> 1;
        const uint32_t k = K[base + half];
        if (STRICT ? (k < x) : (k <= x)) base += half;
        len -= half;
    }
    const uint32_t k = K[base];
    return base + (STRICT ? (k < x) : (k <= x));
}

// rank_in for the few keys of one bucket: no early exit for m = 0 (K[0] is
// then still read, at most one word past the slices, and ignored), so that
// the lanes of a wave do not branch around each other.
template <bool STRICT>
__device__ __forceinline__ uint32_t rank_bucket(const uint32_t* K, uint32_t m, uint32_t x) {
    uint32_t base = 0, len = m;
    while (len > 1) {
        const uint32_t half = len >> 1;
        const uint32_t k = K[base + half];
        if (STRICT ? (k < x) : (k <= x)) base += half;
        len -= half;
    }
    const uint32_t k = K[base];
    return base + ((m != 0u) & (STRICT ? (k < x) : (k <= x)));
}

// #{bs <= x} over the whole array, given that bs[j - 1] <= x (j >= 1) or j = 0.
__device__ uint32_t gallop_le(const uint32_t* __restrict__ bs, uint32_t n, uint32_t j, uint32_t x) {
    uint32_t lo = j, hi = n;
    uint64_t step = 1;
    while (true) {
        const uint64_t probe = (uint64_t)lo + step - 1;
        if (probe >= n) break;
        if (bs[probe] <= x) {
            lo = (uint32_t)probe + 1u;
            step <<= 1;
        } else {
            hi = (uint32_t)probe;
            break;
        }
    }
    return lo + rank_in<false>(bs + lo, hi - lo, x);
}

// Exclusive scan of h[0..m) in place (m <= per * blockDim with per <= 8);
// returns the total.  wsum holds blockDim / 64 words.
__device__ uint32_t block_scan_u32(uint32_t* h, uint32_t m, uint32_t* wsum) {
    const uint32_t per = (m + blockDim.x - 1) / blockDim.x;
    const uint32_t b0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < m) mine += h[b0 + k];
    const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t x = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= (uint32_t)o) x += y;
    }
    if (lane == kWave - 1) wsum[w] = x;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (uint32_t k = 0; k < blockDim.x / kWave; ++k) {
        if (k < w) pre += wsum[k];
        tot += wsum[k];
    }
    pre += x - mine;
    for (uint32_t k = 0; k < per; ++k) {
        if (b0 + k < m) {
            const uint32_t v = h[b0 + k];
            h[b0 + k] = pre;
            pre += v;
        }
    }
    __syncthreads();
    return tot;
}

// A (shuffle, chromosome)'s work in 256 entries, counting what it takes besides
// them: about 1.8 us with none, 3.9 with 830, 6.9 with 4200, 0.9 ns for each
// further one.
__host__ __device__ __forceinline__ uint32_t group_cost(uint32_t h) {
    const uint32_t more = h >> 6;
    return (h >> 8) + 8u + (more < 24u ? more : 24u);
}

// What a chromosome may cost while every workgroup takes the same number of shuffles.
uint32_t bin_most(uint64_t na, uint32_t n_chrom) { return 2u * group_cost((uint32_t)(na / n_chrom)); }

// Ranks of every cell's first coordinate in B_S and B_E, both bisections in
// step so that their dependent loads overlap.
__global__ void __launch_bounds__(256) k_bin_cells(BinGeom g, const uint32_t* __restrict__ bs,
                                                   const uint32_t* __restrict__ be, uint32_t n,
                                                   uint32_t* __restrict__ rs, uint32_t* __restrict__ re, uint64_t* nreg) {
    const uint32_t ncells = g.cb[g.n_chrom];
    if (blockIdx.x == 0 && threadIdx.x == 0) nreg[1] = 0ull;
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < ncells; c += gridDim.x * blockDim.x) {
        const uint32_t k = chrom_of_cell(g, c);
        const uint32_t lo = g.off[k] + ((c - g.cb[k]) << g.shift);
        uint32_t b0 = 0, b1 = 0, len = n;   // n > 0
        while (len > 1) {
            const uint32_t half = len >> 1;
            const uint32_t k0 = bs[b0 + half], k1 = be[b1 + half];
            if (k0 < lo) b0 += half;
            if (k1 < lo) b1 += half;
            len -= half;
        }
        rs[c] = b0 + (bs[b0] < lo);
        re[c] = b1 + (be[b1] < lo);
    }
}

// Regions of one chromosome per workgroup.  A region starts at the
// chromosome's first cell and wherever the merged count since the chromosome's
// start enters a new multiple of kRegionKeys.  Chromosome k's regions take the
// numbers from sum over k' < k of bound(k') on, bound = min(cells, keys /
// kRegionKeys + 1) being the most it can have, so that no scan over
// chromosomes is needed; the numbers it leaves unused are empty regions at its
// end.  Writes cell -> region, the descriptors, with the last chromosome
// the sentinel {genome size, n, n} and the number of regions, and in nreg[1]
// whether a chromosome's queries cost more than `heavy`.
__global__ void __launch_bounds__(kBinThreads) k_bin_regions(BinGeom g, const uint32_t* __restrict__ rs,
                                                             const uint32_t* __restrict__ re, uint32_t n,
                                                             uint32_t nreg_max, uint32_t* __restrict__ cell_region,
                                                             RegionDesc* __restrict__ desc, uint64_t* nreg,
                                                             const uint32_t* __restrict__ hist, uint32_t heavy,
                                                             uint32_t* status) {
    constexpr uint32_t kPer = kMaxCells / kBinThreads, kWaves = kBinThreads / kWave;
    __shared__ uint32_t found[kPer * kWaves], wsum[kWaves], sh_total;
    const uint32_t k = blockIdx.x, c0 = g.cb[k], nc = g.cb[k + 1] - c0, ncells = g.cb[g.n_chrom];
    if (nc == 0) return;
    if (threadIdx.x == 0 && group_cost(hist[k]) > heavy) atomicOr((unsigned long long*)&nreg[1], 1ull);
    const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    auto merged = [&](uint32_t c) -> uint64_t { return c < ncells ? (uint64_t)rs[c] + re[c] : 2ull * n; };
    auto bound = [&](uint32_t q) -> uint32_t {
        const uint32_t a = g.cb[q], m = g.cb[q + 1] - a;
        return m ? (uint32_t)min((uint64_t)m, (merged(a + m) - merged(a)) / kRegionKeys + 1u) : 0u;
    };
    const uint64_t base = merged(c0);
    // thread t holds cells t, t + 1024, ...; all loads (indices clamped) are in flight together
    uint32_t r_s[kPer], r_e[kPer];
    uint64_t prev[kPer];
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
        const uint32_t c = min(u * kBinThreads + threadIdx.x, nc - 1u);
        r_s[u] = rs[c0 + c];
        r_e[u] = re[c0 + c];
        prev[u] = merged(c0 + (c ? c - 1u : 0u));
    }
    uint32_t before = threadIdx.x < k ? bound(threadIdx.x) : 0u;
    uint64_t starts[kPer];   // the wave's cells that start a region
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
        const uint32_t c = u * kBinThreads + threadIdx.x;
        const uint64_t m = ((uint64_t)r_s[u] + r_e[u] - base) / kRegionKeys, q = (prev[u] - base) / kRegionKeys;
        starts[u] = __ballot(c < nc && (c == 0u || m != q));
        if (lane == 0) found[u * kWaves + w] = (uint32_t)__popcll(starts[u]);
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) before += __shfl_xor(before, o);
    if (lane == 0) wsum[w] = before;
    __syncthreads();
    if (w == 0) {   // exclusive prefix of the 128 counts, two a lane
        static_assert(kPer * kWaves == 2 * kWave, "one wave scans the counts");
        const uint32_t a = found[2 * lane], b = found[2 * lane + 1];
        uint32_t x = a + b;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= (uint32_t)o) x += y;
        }
        found[2 * lane] = x - a - b;
        found[2 * lane + 1] = x - b;
        if (lane == kWave - 1) sh_total = x;
    }
    __syncthreads();
    uint32_t first = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) first += wsum[j];   // at most 256 chromosomes before this one
    const uint32_t total = sh_total, most = bound(k);
    if ((first + most > nreg_max || total > most) && threadIdx.x == 0)   // only for unsorted arrays;
        atomicOr(status, BITS_FLAG_CHROM);                               // never index past the table
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
        const uint32_t c = u * kBinThreads + threadIdx.x;
        if (c >= nc) continue;
        // the region of cell c: as many as started up to it, less one
        const uint32_t rid = first + found[u * kWaves + w] + (uint32_t)__popcll(starts[u] & (~0ull >> (63 - lane))) - 1u;
        if (((starts[u] >> lane) & 1u) && rid < nreg_max)
            desc[rid] = RegionDesc{g.off[k] + (c << g.shift), r_s[u], r_e[u], 0u};
        cell_region[c0 + c] = min(rid, nreg_max - 1u);
    }
    // the unused numbers: empty regions where the next chromosome starts
    const uint32_t next = c0 + nc;
    const RegionDesc end = next < ncells ? RegionDesc{g.off[k + 1], rs[next], re[next], 0u}
                                         : RegionDesc{g.off[g.n_chrom], n, n, 0u};
    for (uint32_t r = first + total + threadIdx.x; r < min(first + most, nreg_max); r += kBinThreads) desc[r] = end;
    if (next == ncells && threadIdx.x == 0) {
        const uint32_t all = min(first + most, nreg_max);
        desc[all] = end;   // desc has nreg_max + 1
        *nreg = all;
    }
}

// Inclusive prefix sum over the 64 lanes of a wave, moving data between lanes
// with DPP only (no LDS instruction, so it does not queue behind the
// bisections): four row_shr steps (1, 2, 4, 8) build the prefix inside each
// row of 16 lanes, then row_bcast:15 adds row 0's total to row 1 and row 2's
// to row 3, and row_bcast:31 adds the total of rows 0-1 to rows 2 and 3.
// Lanes whose source lies outside the row, and rows the row mask leaves out,
// receive 0 (the `old` operand), so every step is a plain add.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_in0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_step(uint32_t& x) {
    x += dpp_in0<CTRL, ROWS>(x);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_step(uint64_t& x) {
    const uint32_t lo = dpp_in0<CTRL, ROWS>((uint32_t)x), hi = dpp_in0<CTRL, ROWS>((uint32_t)(x >> 32));
    x += ((uint64_t)hi << 32) | lo;
}

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    scan_step<0x111, 0xF>(x);   // row_shr:1
    scan_step<0x112, 0xF>(x);   // row_shr:2
    scan_step<0x114, 0xF>(x);   // row_shr:4
    scan_step<0x118, 0xF>(x);   // row_shr:8
    scan_step<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
    scan_step<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
    return x;
}

// Lane i's value in every lane of the wave (i uniform).
__device__ __forceinline__ uint32_t lane_value(uint32_t x, uint32_t i) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)i);
}

__device__ __forceinline__ uint64_t lane_value(uint64_t x, uint32_t i) {
    return ((uint64_t)lane_value((uint32_t)(x >> 32), i) << 32) | lane_value((uint32_t)x, i);
}

// Staged binning (second sweep): chromosomes with kStageMinRegions..kStageRegions
// regions; kStageRecs records staged at a time, so that the workgroup's LDS (about
// 76 KB) still lets two workgroups share a CU.
constexpr uint32_t kStageRegions = 2048;
constexpr uint32_t kStageMinRegions = 128;
constexpr uint32_t kStageRecs = 5632;      // 44 KB
// A group of at most kGroupRecs entries is placed once and held in registers.
constexpr int kGroupPer = 8;
constexpr uint32_t kGroupRecs = kGroupPer * kBinThreads;
static_assert(kGroupRecs < (1u << 16), "places in a group are 16-bit");
static_assert(kStageRegions <= 2 * kBinThreads, "one thread owns two regions' chunk counters");
static_assert(kMaxCells <= (1u << 16), "cell-to-region table entries are 16-bit");

// Entry j of an array of 16-bit values packed two per word.
__device__ __forceinline__ uint32_t half16(const uint32_t* w, uint32_t j) {
    return (w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
}

// Binning of shuffles [sb, sb + nb): a workgroup makes the placements of one
// chromosome k's queries (table positions [cursor[k] - hist[k], cursor[k])) in
// one shuffle s, or in several in turn (MANY, place_share), counts them per region,
// writes the segment table of (s, every region of k), and writes the records
// {start, end} in region order to recs[s * na + table position range].  A group
// of at most kGroupRecs entries is placed once and held in registers; a larger
// one is placed twice, to count and to write, either one by one (few regions,
// or more than kStageRegions) or chunk by chunk through LDS.
// (8 waves per SIMD: two workgroups per CU, at most 64 VGPRs.)
// The scattered write-out bounds large groups: with 3 Philox rounds for 10 the
// 4920 us of 1e9 placements become 4560, and without the counting sweep, every
// region having slots for five standard deviations more than its mean, 5600.
// A workgroup of 4000 entries spends half its time on its start, the region
// table and the chain of loads and barriers before its first store, so it takes
// several shuffles (1e5 entries in 24 chromosomes x 2000 shuffles: 800 -> 648 us;
// 2000 x 100: 21.3 -> 18.9 us): as many as place_share gives it.

// The chromosome and the shuffles [s0, s1) of workgroup b when workgroups take
// several and a chromosome costs more than bin_most: of n_chrom * wgs workgroups
// each chromosome has its part by group_cost (rounded, at least 1 and at most
// nb), which split the shuffles evenly, so that a workgroup's work does not
// depend on how the queries lie over the chromosomes (1e6 queries x 100 shuffles
// on one of 256 chromosomes: 13370 us with as many shuffles for every
// workgroup, 1960 so, 2210 with one; 1e5 x 1000 on 24 of 256: 5140, 1330,
// 2250).  Sets spread more evenly keep the same number for all: to find the
// shares costs every workgroup a microsecond (3e4 x 2000: 720 and 755 us).
// There are less than n_chrom more of them; false past the last.  All lanes call it.
__device__ __forceinline__ bool place_share(const uint32_t* __restrict__ hist, uint32_t n_chrom, uint32_t nb, uint32_t wgs,
                                            uint32_t b, uint32_t& k, uint32_t& s0, uint32_t& s1) {
    constexpr uint32_t kPer = BITS_MAX_CHROM / kWave;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    uint32_t cost[kPer], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t c = j * kWave + lane;
        cost[j] = c < n_chrom ? group_cost(hist[c]) : 0u;
        sum += cost[j];
    }
    const float inv = (float)(n_chrom * wgs) / (float)lane_value(wave_inclusive_scan<uint32_t>(sum), kWave - 1);
    uint32_t before = 0;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t v = cost[j] ? min(nb, max(1u, (uint32_t)((float)cost[j] * inv + 0.5f))) : 0u;
        const uint32_t x = wave_inclusive_scan<uint32_t>(v);
        const uint64_t past = __ballot(before + x > b);
        if (past) {
            const uint32_t l = (uint32_t)__builtin_ctzll(past), n = lane_value(v, l);
            const uint32_t i = b - (before + lane_value(x, l) - n);
            k = j * kWave + l;
            s0 = nb * i / n;
            s1 = nb * (i + 1u) / n;
            return true;
        }
        before += lane_value(x, kWave - 1);
    }
    return false;
}

template <bool MANY>
__global__ void __launch_bounds__(kBinThreads, 8) k_bin_place(
    BinGeom g, const uint2* __restrict__ packed, const uint32_t* __restrict__ hist, const uint32_t* __restrict__ cursor,
    uint64_t na, uint64_t seed, uint64_t sb, uint32_t nb, uint32_t per, const uint32_t* __restrict__ cell_region,
    const uint64_t* __restrict__ nreg_p, uint32_t nreg_max, uint32_t* __restrict__ seg_start,
    uint32_t* __restrict__ seg_cnt, uint2* __restrict__ recs) {
    constexpr int kChunkPer = MANY ? 6 : 10;   // a chunk's entries per thread
    constexpr uint32_t kChunkRecs = kChunkPer * kBinThreads;
    static_assert(kChunkRecs < (1u << 16), "chunk counts and offsets are 16-bit");
    __shared__ uint16_t cr[kMaxCells];
    __shared__ uint32_t hs[kStageRegions];          // segment cursors (staged path)
    __shared__ uint32_t cc[kStageRegions / 2];      // chunk counts, 16 bits each
    __shared__ uint32_t co[kStageRegions / 2];      // chunk offsets (exclusive), 16 bits each
    __shared__ uint2 stage[kStageRecs];             // the chunk's records in region order; h of the direct path
    __shared__ uint32_t wsum[kBinThreads / kWave];
    __shared__ uint32_t staged_total;
    const uint32_t wgs = MANY ? (nb + per - 1u) / per : nb;
    uint32_t k = blockIdx.x / wgs, s0 = (blockIdx.x - k * wgs) * (MANY ? per : 1u), s1 = MANY ? min(nb, s0 + per) : s0 + 1u;
    if (MANY) {
        if (nreg_p[1]) {
            if (!place_share(hist, g.n_chrom, nb, wgs, blockIdx.x, k, s0, s1)) return;
        } else if (k >= g.n_chrom) {
            return;
        }
    }
    const uint32_t c0 = g.cb[k], nc = g.cb[k + 1] - c0;
    if (nc == 0) return;
    const uint32_t nreg = (uint32_t)*nreg_p;
    const uint32_t rb = cell_region[c0];
    const uint32_t rl = (k + 1 < g.n_chrom && g.cb[k + 1] < g.cb[g.n_chrom]) ? cell_region[g.cb[k + 1]] : nreg;
    const uint32_t nr = rl > rb ? min(min(rl - rb, nc), nreg_max - rb) : 0u;
    // staging pays when a chromosome spreads its records over many regions (many open
    // record lines); with few regions the direct writes already merge in L2
    const bool staged = nr >= kStageMinRegions && nr <= kStageRegions;
    uint32_t* h = staged ? hs : reinterpret_cast<uint32_t*>(stage);   // kMaxCells words fit the stage buffer
    const uint32_t g1 = cursor[k], g0 = g1 - hist[k];
    const bool whole = g1 - g0 <= kGroupRecs && nr <= kStageRegions;
    for (uint32_t j = threadIdx.x; j < nc; j += kBinThreads) cr[j] = (uint16_t)(cell_region[c0 + j] - rb);
    const uint32_t ok = g.off[k], sh = g.shift, clen = g.off[k + 1] - g.off[k];
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint32_t nw2 = (nr + 1) >> 1;
    const bool owner = threadIdx.x < nw2;
    if (whole) {
        // Every entry is placed once and kept, with its rank in its region, in registers;
        // the counts give the segment table directly, and the records in region order are
        // the group's final layout, written out sequentially in windows of kStageRecs.  The
        // next shuffle's ranking touches only the counters, so it may overlap the write-out.
        if (owner) cc[threadIdx.x] = 0u;
        __syncthreads();
        for (uint32_t s = s0; s < s1; ++s) {
            const uint64_t gs = (sb + s) * na;
            uint32_t st_[kGroupPer], len[kGroupPer], key[kGroupPer];   // key: region << 16 | rank in it, or ~0
            // the entries are read again for every shuffle (they stay in L2): held, they and
            // what the compiler derives from them spill
            uint32_t from = g0 + threadIdx.x;
            if (MANY) asm volatile("" : "+v"(from));
#pragma unroll
            for (int u = 0; u < kGroupPer; ++u) {
                key[u] = 0xFFFFFFFFu;
                st_[u] = len[u] = 0u;
                if (g0 + (uint32_t)u * kBinThreads >= g1) continue;   // uniform
                const uint32_t p = from + (uint32_t)u * kBinThreads;
                const uint2 q = p < g1 ? packed[p] : make_uint2(0u, 0u);
                len[u] = q.y;
                if (!q.y) continue;
                const uint32_t st = mc_place(gs + q.x, k0, k1, ok, clen - q.y + 1u);
                const uint32_t lr = cr[(st - ok) >> sh];
                if (lr >= nr) continue;
                const uint32_t sft = 16u * (lr & 1u);
                const uint32_t old = atomicAdd(&cc[lr >> 1], 1u << sft);
                st_[u] = st;
                key[u] = (lr << 16) | ((old >> sft) & 0xFFFFu);
            }
            __syncthreads();   // counts complete; the previous shuffle is written out
            const uint32_t wv = owner ? cc[threadIdx.x] : 0u;
            const uint32_t a0 = wv & 0xFFFFu, a1 = wv >> 16, tsum = a0 + a1;
            const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
            uint32_t pre = 0;
            if (nw2 <= kWave) {   // the first wave owns all the counters
                if (w == 0) {
                    const uint32_t x = wave_inclusive_scan<uint32_t>(tsum);
                    if (lane == kWave - 1) staged_total = x;
                    pre = x - tsum;
                }
            } else {
                const uint32_t x = wave_inclusive_scan<uint32_t>(tsum);
                if (lane == kWave - 1) wsum[w] = x;
                __syncthreads();
                uint32_t tot = 0;
                for (uint32_t j = 0; j < kBinThreads / kWave; ++j) {
                    if (j < w) pre += wsum[j];
                    tot += wsum[j];
                }
                pre += x - tsum;
                if (threadIdx.x == 0) staged_total = tot;
            }
            if (owner) {
                uint32_t* ss = seg_start + (uint64_t)s * nreg_max + rb;
                uint32_t* sc = seg_cnt + (uint64_t)s * nreg_max + rb;
                const uint32_t r0 = 2u * threadIdx.x, lo1 = pre + a0;
                cc[threadIdx.x] = 0u;   // ready for the next shuffle
                co[threadIdx.x] = pre | (lo1 << 16);
                ss[r0] = g0 + pre;
                sc[r0] = a0;
                if (r0 + 1u < nr) {
                    ss[r0 + 1u] = g0 + lo1;
                    sc[r0 + 1u] = a1;
                }
            }
            __syncthreads();
            const uint32_t tot = staged_total;
#pragma unroll
            for (int u = 0; u < kGroupPer; ++u)   // now the place in the group, or ~0
                if (key[u] != 0xFFFFFFFFu) key[u] = half16(co, key[u] >> 16) + (key[u] & 0xFFFFu);
            uint2* out = recs + (uint64_t)s * na + g0;
            for (uint32_t w0 = 0; w0 < tot; w0 += kStageRecs) {
                if (w0) __syncthreads();   // the last window is written out
#pragma unroll
                for (int u = 0; u < kGroupPer; ++u)
                    if (key[u] - w0 < kStageRecs) stage[key[u] - w0] = make_uint2(st_[u], st_[u] + (len[u] - 1u));
                __syncthreads();
                const uint32_t m = min(kStageRecs, tot - w0);
                for (uint32_t j = threadIdx.x; j < m; j += kBinThreads) out[w0 + j] = stage[j];
            }
        }
        return;
    }
    for (uint32_t s = s0; s < s1; ++s) {
        const uint64_t gs = (sb + s) * na;
        if (MANY) __syncthreads();   // the last shuffle's counters are read
        for (uint32_t j = threadIdx.x; j < nr; j += kBinThreads) h[j] = 0u;
        __syncthreads();
        for (uint32_t p0 = g0 + threadIdx.x; p0 < g1; p0 += ILP * kBinThreads) {
            uint2 q[ILP];
#pragma unroll
            for (int u = 0; u < ILP; ++u) {
                const uint32_t p = p0 + u * kBinThreads;
                q[u] = p < g1 ? packed[p] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < ILP; ++u) {
                if (!q[u].y) continue;
                const uint32_t st = mc_place(gs + q[u].x, k0, k1, ok, clen - q[u].y + 1u);
                const uint32_t lr = cr[(st - ok) >> sh];
                if (lr < nr) atomicAdd(&h[lr], 1u);
            }
        }
        __syncthreads();
        uint32_t* ss = seg_start + (uint64_t)s * nreg_max + rb;
        uint32_t* sc = seg_cnt + (uint64_t)s * nreg_max + rb;
        for (uint32_t j = threadIdx.x; j < nr; j += kBinThreads) sc[j] = h[j];
        __syncthreads();
        block_scan_u32(h, nr, wsum);
        for (uint32_t j = threadIdx.x; j < nr; j += kBinThreads) ss[j] = g0 + h[j];
        __syncthreads();
        uint2* out = recs + (uint64_t)s * na;
        if (!staged) {
            for (uint32_t p0 = g0 + threadIdx.x; p0 < g1; p0 += ILP * kBinThreads) {
                uint2 q[ILP];
#pragma unroll
                for (int u = 0; u < ILP; ++u) {
                    const uint32_t p = p0 + u * kBinThreads;
                    q[u] = p < g1 ? packed[p] : make_uint2(0u, 0u);
                }
#pragma unroll
                for (int u = 0; u < ILP; ++u) {
                    if (!q[u].y) continue;
                    const uint32_t st = mc_place(gs + q[u].x, k0, k1, ok, clen - q[u].y + 1u);
                    const uint32_t lr = cr[(st - ok) >> sh];
                    if (lr >= nr) continue;
                    const uint32_t at = atomicAdd(&h[lr], 1u);
                    out[g0 + at] = make_uint2(st, st + (q[u].y - 1u));
                }
            }
            continue;
        }
        // staged: chunks of kChunkRecs table entries are placed into registers, counting-sorted
        // by region in LDS, in windows of kStageRecs, and written out in region runs.  The runs
        // are the longer the larger the chunk (1e9 placements, 82 a region and shuffle: 6, 8,
        // 10, 11 entries a thread 5240, 5030, 4920, 4940 us; 14 spill: 6100).  Thread t < nw2 owns regions 2t and 2t + 1
        // (counter word t) for the whole loop.  During a chunk, hs[r] holds region r's cursor
        // minus the offset of r's run in the chunk, so the chunk's record j goes to
        // g0 + hs[r] + j; the next chunk's scan adds back the end of that run (kept in the
        // owner's registers) to get the cursor again.  The next chunk's ranking touches only
        // the counters, so it may overlap the last write-out.
        if (owner) cc[threadIdx.x] = 0u;
        uint32_t end0 = 0u, end1 = 0u;   // the owner's run ends in the previous chunk
        __syncthreads();
        for (uint32_t cb = g0; cb < g1; cb += kChunkRecs) {
            const uint32_t ce = min(g1, cb + kChunkRecs);
            uint32_t st_[kChunkPer], len_[kChunkPer], key_[kChunkPer];   // key = lr << 16 | rank, or ~0
#pragma unroll
            for (int u = 0; u < kChunkPer; ++u) {
                const uint32_t p = cb + threadIdx.x + (uint32_t)u * kBinThreads;
                const uint2 q = p < ce ? packed[p] : make_uint2(0u, 0u);
                key_[u] = 0xFFFFFFFFu;
                st_[u] = 0u;
                len_[u] = q.y;
                if (!q.y) continue;
                const uint32_t st = mc_place(gs + q.x, k0, k1, ok, clen - q.y + 1u);
                const uint32_t lr = cr[(st - ok) >> sh];
                if (lr >= nr) continue;
                const uint32_t sft = 16u * (lr & 1u);
                const uint32_t old = atomicAdd(&cc[lr >> 1], 1u << sft);
                st_[u] = st;
                key_[u] = (lr << 16) | ((old >> sft) & 0xFFFFu);
            }
            __syncthreads();   // counts complete; the previous chunk is written out
            // exclusive offsets of the chunk's region counts (two per word) into co, and the
            // owners' cursors turned into this chunk's deltas
            {
                const uint32_t wv = owner ? cc[threadIdx.x] : 0u;
                if (owner) cc[threadIdx.x] = 0u;   // ready for the next chunk
                const uint32_t a0 = wv & 0xFFFFu, a1 = wv >> 16, tsum = a0 + a1;
                const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
                const uint32_t x = wave_inclusive_scan<uint32_t>(tsum);
                if (lane == kWave - 1) wsum[w] = x;
                __syncthreads();
                uint32_t pre = 0, tot = 0;
                for (uint32_t j = 0; j < kBinThreads / kWave; ++j) {
                    if (j < w) pre += wsum[j];
                    tot += wsum[j];
                }
                pre += x - tsum;
                if (owner) {
                    const uint32_t r0 = 2u * threadIdx.x, lo1 = pre + a0;
                    co[threadIdx.x] = pre | (lo1 << 16);
                    hs[r0] = hs[r0] + end0 - pre;
                    end0 = lo1;
                    if (r0 + 1u < nr) {
                        hs[r0 + 1u] = hs[r0 + 1u] + end1 - lo1;
                        end1 = lo1 + a1;
                    }
                }
                if (threadIdx.x == 0) staged_total = tot;
            }
            __syncthreads();
            const uint32_t tot = staged_total;
#pragma unroll
            for (int u = 0; u < kChunkPer; ++u)   // now the place in the chunk, or ~0
                if (key_[u] != 0xFFFFFFFFu) key_[u] = half16(co, key_[u] >> 16) + (key_[u] & 0xFFFFu);
            for (uint32_t w0 = 0; w0 < tot; w0 += kStageRecs) {
                if (w0) __syncthreads();   // the last window is written out
#pragma unroll
                for (int u = 0; u < kChunkPer; ++u)
                    if (key_[u] - w0 < kStageRecs) stage[key_[u] - w0] = make_uint2(st_[u], st_[u] + (len_[u] - 1u));
                __syncthreads();
                const uint32_t m = min(kStageRecs, tot - w0);
                for (uint32_t j = threadIdx.x; j < m; j += kBinThreads) {
                    const uint2 rec = stage[j];
                    const uint32_t lr = cr[(rec.x - ok) >> sh];
                    out[g0 + hs[lr] + w0 + j] = rec;
                }
            }
        }
    }
}

// A wave-uniform word read from LDS, in a scalar register.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// Buckets over the coordinates [lo, lo + span): bucket of x = (x - lo) scale >> 32.
// T[b] = #{keys of the slice in the buckets before b}; the keys of bucket b
// are ranks [T[b], T[b + 1]).
struct Buckets {
    const uint16_t* T;
    uint32_t lo, scale;
    __device__ __forceinline__ uint32_t of(uint32_t x) const { return __umulhi(x - lo, scale); }
};

// The number of buckets over `span` > 0 coordinates for m keys (three for four
// keys: a small slice is not worth a long table), and the scale.  The
// factor 1 - 2^-20 covers the float roundings (3 x 2^-24), so that
// scale <= 2^32 nb / span and the last coordinate's bucket is below nb.
__device__ __forceinline__ uint32_t bucket_scale(uint32_t m, uint32_t span, uint32_t* scale) {
    const uint32_t nb = min(min(kBuckets, m - m / 4u + 1u), span);
    *scale = (uint32_t)((float)nb * 4294967296.f / (float)span * (1.f - 0x1p-20f));
    return nb;
}

// T[b] for b = 0 .. nb, K[0..m) sorted with K[0] >= bk.lo.  With F(x) the
// bucket of x, or nb past the last, key j writes j to the buckets in
// (F(K[j - 1]), F(K[j])] and a final step j = m fills the rest up to nb: every
// bucket is written once, in one pass over the keys.
__device__ void bucket_ranks(const uint32_t* K, uint32_t m, const Buckets& bk, uint32_t nb, uint16_t* T) {
    for (uint32_t j = threadIdx.x; j <= m; j += blockDim.x) {
        const uint32_t lo = j == 0 ? 0u : min(bk.of(K[j - 1]), nb) + 1u;
        const uint32_t hi = j == m ? nb : min(bk.of(K[j]), nb);
        for (uint32_t b = lo; b <= hi; ++b) T[b] = (uint16_t)j;
    }
}

// #{K < x} (STRICT) or #{K <= x} in a slice, x inside the buckets: the keys
// before x's bucket, and those of its first kBucketKeys keys that count.  Keys
// of later buckets are above x, and so is the padding (x < 0xFFFFFFFF), so no
// bound is looked up; only a bucket with more keys below x is bisected on.
template <bool STRICT>
__device__ __forceinline__ uint32_t rank_buckets(const uint32_t* K, const Buckets& bk, uint32_t x) {
    const uint32_t b = bk.of(x), lo = bk.T[b];
    const uint32_t* k = K + lo;
    uint32_t c = 0;
#pragma unroll
    for (uint32_t i = 0; i < kFirstKeys; ++i) c += STRICT ? (k[i] < x) : (k[i] <= x);
    if (c != kFirstKeys) return lo + c;
#pragma unroll
    for (uint32_t i = kFirstKeys; i < kBucketKeys; ++i) c += STRICT ? (k[i] < x) : (k[i] <= x);
    if (c == kBucketKeys) c += rank_bucket<STRICT>(k + kBucketKeys, bk.T[b + 1] - lo - kBucketKeys, x);
    return lo + c;
}

// Wave-level segmented sum: lanes carry (key, value) with the keys of the
// valid lanes non-decreasing in lane order; each run of equal keys adds its
// sum to acc[key] with at most two LDS atomics (the run's inclusive prefix at
// its last lane, minus the prefix before its first lane, which is that lane's
// inclusive prefix minus its own value).  T = uint32_t only when 64 values
// cannot reach 2^32.
template <typename T>
__device__ __forceinline__ void wave_segment_add(uint32_t key, T v, bool valid, unsigned long long* acc) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const T x = wave_inclusive_scan<T>(v);
    // the neighbours' keys by whole-wave DPP shifts (wave_shr:1, wave_shl:1); lane 0's kp and
    // lane 63's kn are never used
    const uint32_t kp = dpp_in0<0x138, 0xF>(key), kn = dpp_in0<0x130, 0xF>(key);
    if (!valid) return;
    if (lane == kWave - 1 || kn != key) atomicAdd(&acc[key], (unsigned long long)x);
    if (lane != 0 && kp != key) atomicAdd(&acc[key], 0ull - (unsigned long long)(x - v));
}

// The placements of one region, counted against slices S = B_S[s_lo, s_lo + ns)
// and E = B_E[e_lo, e_lo + ne) (in LDS, or in HBM for an oversize region):
// the workgroup's share [q0, q1) of the region's records.  Each wave takes a
// contiguous range of it, 64 records per step; record p of the pass
// (p < pre[nb] < 2^32) is recs[base[s] + p], s its shuffle, pre[s] <= p <
// pre[s + 1].  The wave walks the shuffles with scalars: a step's counts are
// summed up to every lane, and where a shuffle ends its part of the sums, read
// from its last lane, goes to acc[s].
// Vector issue (75% of the cycles) and the LDS (58%) bound this loop, 81 vector
// instructions per 64 records.  Half as many buckets of power-of-two widths,
// bisected, shuffles tracked by each lane, a segmented sum with two LDS atomics
// a run and one load ahead took 124 (1e9 records against 5e7 keys: 3700 -> 3310
// us; 2e8 against 1e6: 775 -> 684 us).
// LANES, for few records a shuffle (many shuffles end in a step): every lane
// finds its own record's shuffle, moving forward, and a segmented sum adds up.
template <bool LDS, bool LANES, typename T>
__device__ __forceinline__ void bin_count_region(const uint32_t* S, uint32_t ns, const uint32_t* E, uint32_t ne,
                                                 const uint32_t* __restrict__ bs, uint32_t n, uint32_t s_lo,
                                                 uint32_t e_lo, const Buckets& bks, const Buckets& bke,
                                                 uint32_t key_top, const uint2* __restrict__ recs,
                                                 const uint32_t* pre, const uint32_t* base, uint32_t nb,
                                                 uint64_t q0, uint64_t q1, unsigned long long* acc) {
    const uint32_t lane = threadIdx.x & (kWave - 1), wv = uniform(threadIdx.x / kWave), nw = blockDim.x / kWave;
    const uint64_t steps = (q1 - q0 + kWave - 1) / kWave, per = (steps + nw - 1) / nw;
    const uint64_t p0 = q0 + (uint64_t)wv * per * kWave, p1 = min(q1, p0 + per * kWave);
    if (p0 >= p1) return;
    const uint32_t s_end = s_lo + ns;
    // shuffle of the wave's first record: the last s with pre[s] <= p0
    uint32_t sc = 0, hi = nb;
    while (hi - sc > 1) {
        const uint32_t mid = (sc + hi) >> 1;
        if (uniform(pre[mid]) <= p0) sc = mid; else hi = mid;
    }
    uint32_t end_c = uniform(pre[sc + 1]);   // the end of the counted step's shuffle
    // the shuffle of the records being loaded, kAhead steps ahead, so that a wave has
    // that many record loads in flight
    uint32_t sn = sc, end_n = end_c, base_n = uniform(base[sc]), lane_s = sc;
    auto load = [&](uint64_t b, uint32_t& of) {   // records [b, min(b + 64, p1)), b < p1
        const uint32_t e = (uint32_t)min(p1, b + kWave), p = (uint32_t)b + lane;
        if (LANES) {
            if (lane >= e - (uint32_t)b) return make_uint2(bke.lo, bke.lo);
            while (pre[lane_s + 1] <= p) ++lane_s;   // ends at lane_s < nb: p < pre[nb]
            of = lane_s;
            return recs[base[lane_s] + p];
        }
        uint32_t at = base_n + p;
        while (end_n < e) {   // ends at sn < nb: e <= pre[nb]
            const uint32_t from = end_n;
            ++sn;
            end_n = uniform(pre[sn + 1]);
            base_n = uniform(base[sn]);
            if (p >= from) at = base_n + p;
        }
        return lane < e - (uint32_t)b ? recs[at] : make_uint2(bke.lo, bke.lo);
    };
    unsigned long long run = 0ull;   // of shuffle sc, in the steps so far
    auto count = [&](uint64_t b, uint2 r, uint32_t of) {   // the step of records [b, min(b + 64, p1))
        uint32_t first, last;
        if (LDS && r.y < key_top) {   // every key <= r.y is inside the slice
            first = s_lo + rank_buckets<false>(S, bks, r.y);
        } else if (r.y == 0xFFFFFFFFu) {
            first = n;
        } else {
            const uint32_t c = rank_in<false>(S, ns, r.y);
            first = (c == ns && s_end < n) ? gallop_le(bs, n, s_end, r.y) : s_lo + c;
        }
        if (LDS)   // the start lies in the region
            last = e_lo + rank_buckets<true>(E, bke, r.x);
        else
            last = e_lo + rank_in<true>(E, ne, r.x);
        const uint32_t e = (uint32_t)min(p1, b + kWave), got = e - (uint32_t)b;
        if (LANES) {
            const bool valid = lane < got;
            wave_segment_add<T>(valid ? of : 0xFFFFFFFFu, valid ? (T)(first - last) : (T)0, valid, acc);
            return;
        }
        const T x = wave_inclusive_scan<T>(lane < got ? (T)(first - last) : (T)0);
        T before = 0;
        while (end_c <= e) {   // end_c > b: shuffle sc ends in this step
            const T upto = lane_value(x, end_c - 1u - (uint32_t)b);
            run += (T)(upto - before);
            before = upto;
            if (lane == 0) atomicAdd(&acc[sc], run);
            run = 0ull;
            if (++sc == nb) break;
            end_c = uniform(pre[sc + 1]);
        }
        run += (T)(lane_value(x, kWave - 1) - before);
    };
    uint2 rn[kAhead];
    uint32_t of[kAhead];   // the lanes' shuffles
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u)
        if (p0 + u * kWave < p1) rn[u] = load(p0 + u * kWave, of[u]);
    for (uint64_t b0 = p0; b0 < p1; b0 += kAhead * kWave) {
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) {
            const uint64_t b = b0 + u * kWave;
            if (b >= p1) break;
            const uint2 r = rn[u];
            const uint32_t s = LANES ? of[u] : 0u;
            if (b + kAhead * kWave < p1) rn[u] = load(b + kAhead * kWave, of[u]);
            count(b, r, s);
        }
    }
    if (lane == 0 && run) atomicAdd(&acc[sc], run);   // run = 0 once sc = nb
}

// `splits` workgroups per region r < nreg (nreg on the device; workgroups past
// it return): stage the slices, count the workgroup's share of the placements
// of the batch that start in the region, write partial[(r * splits + part) * nb + s].
// SPLIT = false is the one-workgroup-per-region form (splits = 1).
template <bool SPLIT>
__global__ void __launch_bounds__(kBinThreads) k_bin_search(
    const uint32_t* __restrict__ bs, const uint32_t* __restrict__ be, uint32_t n,
    const RegionDesc* __restrict__ desc, const uint64_t* __restrict__ nreg_p, const uint32_t* __restrict__ seg_start,
    const uint32_t* __restrict__ seg_cnt, uint32_t nreg_max, uint32_t nb, const uint2* __restrict__ recs,
    uint64_t na, uint32_t splits, unsigned long long* __restrict__ partial) {
    __shared__ uint32_t slice[kSliceWords + 2 * kBucketKeys];   // both slices, each with its padding
    __shared__ uint16_t tabs[2][kBuckets + 1];
    __shared__ uint32_t pre[BITS_MC_BIN_MAX_BATCH + 1];
    __shared__ uint32_t base[BITS_MC_BIN_MAX_BATCH];
    __shared__ unsigned long long acc[BITS_MC_BIN_MAX_BATCH];
    __shared__ uint32_t w32[kBinThreads / kWave];
    const uint32_t r = SPLIT ? blockIdx.x / splits : blockIdx.x, part = SPLIT ? blockIdx.x - r * splits : 0u;
    if (r >= *nreg_p) return;
    const RegionDesc d0 = desc[r], d1 = desc[r + 1];
    const uint32_t s_lo = d0.s_lo, e_lo = d0.e_lo;
    const uint32_t s_end = (uint32_t)min((uint64_t)d1.s_lo + kMargin, (uint64_t)n);
    const uint32_t ns = s_end - s_lo, ne = d1.e_lo - e_lo;
    // per-shuffle prefix of the segment lengths, and each shuffle's record base: record p of
    // the pass (in shuffle s) is recs[s * na + seg_start + (p - pre[s])]; nb * na < 2^32
    uint32_t cnt = 0, sst = 0;
    if (threadIdx.x < nb) {
        sst = seg_start[(uint64_t)threadIdx.x * nreg_max + r];
        cnt = seg_cnt[(uint64_t)threadIdx.x * nreg_max + r];
        acc[threadIdx.x] = 0ull;
    }
    {
        const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
        uint32_t x = cnt;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= (uint32_t)o) x += y;
        }
        if (lane == kWave - 1) w32[w] = x;
        __syncthreads();
        uint32_t before = 0;
        for (uint32_t j = 0; j < w; ++j) before += w32[j];
        const uint32_t pr = before + x - cnt;
        if (threadIdx.x < nb) {
            pre[threadIdx.x] = pr;
            base[threadIdx.x] = threadIdx.x * (uint32_t)na + sst - pr;
        }
        if (threadIdx.x == nb - 1) pre[nb] = before + x;
    }
    __syncthreads();
    if (pre[nb] == 0u) {   // no placement starts here (uniform)
        if (threadIdx.x < nb)
            partial[(SPLIT ? (uint64_t)r * splits + part : (uint64_t)r) * nb + threadIdx.x] = 0ull;
        return;
    }
    const uint32_t eo = ns + kBucketKeys;   // E's first word
    const bool in_lds = (uint64_t)ns + ne <= kSliceWords;
    // E's buckets cover the region, S's an eighth more, for the ends that cross
    // the region's end (not past the last staged key: up to it, every key is staged)
    const uint32_t key_lo = d0.key_lo, span = d1.key_lo - key_lo;   // > 0: a region holds at least one cell
    uint32_t key_top = d1.key_lo + min(span / 8u, 0xFFFFFFFFu - d1.key_lo);
    Buckets bks{tabs[0], key_lo, 0u}, bke{tabs[1], key_lo, 0u};
    if (in_lds) {
        for (uint32_t j = threadIdx.x; j < ns; j += blockDim.x) slice[j] = bs[s_lo + j];
        for (uint32_t j = threadIdx.x; j < ne; j += blockDim.x) slice[eo + j] = be[e_lo + j];
        if (threadIdx.x < kBucketKeys) slice[ns + threadIdx.x] = slice[eo + ne + threadIdx.x] = 0xFFFFFFFFu;
        __syncthreads();
        if (s_end < n) key_top = min(key_top, max(slice[ns - 1], d1.key_lo));
        const uint32_t nbs = bucket_scale(ns, key_top - key_lo, &bks.scale), nbe = bucket_scale(ne, span, &bke.scale);
        bucket_ranks(slice, ns, bks, nbs, tabs[0]);
        bucket_ranks(slice + eo, ne, bke, nbe, tabs[1]);
    }
    __syncthreads();
    // this workgroup's share of the region's records
    const uint64_t total = pre[nb];
    const uint64_t q0 = SPLIT ? total * part / splits : 0ull, q1 = SPLIT ? total * (part + 1) / splits : total;
    // per-step sums fit 32 bits when 64 counts of at most n cannot reach 2^32
    const bool narrow = n < (1u << 26);
    const bool lanes = total < (uint64_t)kWalkRecords * nb;
    if (in_lds && lanes && narrow)
        bin_count_region<true, true, uint32_t>(slice, ns, slice + eo, ne, bs, n, s_lo, e_lo, bks, bke, key_top,
                                               recs, pre, base, nb, q0, q1, acc);
    else if (in_lds && lanes)
        bin_count_region<true, true, uint64_t>(slice, ns, slice + eo, ne, bs, n, s_lo, e_lo, bks, bke, key_top,
                                               recs, pre, base, nb, q0, q1, acc);
    else if (in_lds && narrow)
        bin_count_region<true, false, uint32_t>(slice, ns, slice + eo, ne, bs, n, s_lo, e_lo, bks, bke, key_top,
                                               recs, pre, base, nb, q0, q1, acc);
    else if (in_lds)
        bin_count_region<true, false, uint64_t>(slice, ns, slice + eo, ne, bs, n, s_lo, e_lo, bks, bke, key_top,
                                               recs, pre, base, nb, q0, q1, acc);
    else if (narrow)
        bin_count_region<false, false, uint32_t>(bs + s_lo, ns, be + e_lo, ne, bs, n, s_lo, e_lo, bks, bke, key_top,
                                                 recs, pre, base, nb, q0, q1, acc);
    else
        bin_count_region<false, false, uint64_t>(bs + s_lo, ns, be + e_lo, ne, bs, n, s_lo, e_lo, bks, bke, key_top,
                                                 recs, pre, base, nb, q0, q1, acc);
    __syncthreads();
    if (threadIdx.x < nb)
        partial[(SPLIT ? (uint64_t)r * splits + part : (uint64_t)r) * nb + threadIdx.x] = acc[threadIdx.x];
}

// totals[s] += sum over the nreg * splits region shares j of partial[j * nb + s];
// blockIdx.y takes every gridDim.y-th share.
__global__ void __launch_bounds__(256) k_bin_reduce(const unsigned long long* __restrict__ partial,
                                                    const uint64_t* __restrict__ nreg_p, uint32_t splits,
                                                    uint32_t nb, unsigned long long* __restrict__ totals) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nb) return;
    const uint64_t shares = *nreg_p * splits;
    unsigned long long v = 0ull;
    for (uint64_t j = blockIdx.y; j < shares; j += gridDim.y) v += partial[j * nb + s];
    if (v) atomicAdd(totals + s, v);
}

// Cell shift and per-chromosome cell bases of a genome; false if no shift
// keeps every chromosome within kMaxCells cells (impossible below 2^32 bp).
bool bin_geometry(const uint32_t* chrom_len, uint32_t n_chrom, BinGeom* g) {
    uint64_t maxlen = 0, acc = 0;
    for (uint32_t k = 0; k < n_chrom; ++k) maxlen = chrom_len[k] > maxlen ? chrom_len[k] : maxlen;
    uint32_t sh = kMinShift;
    while (sh < 32 && ((maxlen + (1ull << sh) - 1) >> sh) > kMaxCells) ++sh;
    if (sh >= 32) return false;
    g->n_chrom = n_chrom;
    g->shift = sh;
    uint64_t cells = 0;
    for (uint32_t k = 0; k < n_chrom; ++k) {
        g->off[k] = (uint32_t)acc;
        g->cb[k] = (uint32_t)cells;
        acc += chrom_len[k];
        cells += ((uint64_t)chrom_len[k] + (1ull << sh) - 1) >> sh;
    }
    if (acc > 0xFFFFFFFFull || cells > 0xFFFFFFFFull) return false;
    for (uint32_t k = n_chrom; k <= BITS_MAX_CHROM; ++k) {
        g->off[k] = (uint32_t)acc;
        g->cb[k] = (uint32_t)cells;
    }
    return true;
}

}  // namespace

bool bin_layout(const uint32_t* chrom_len, uint32_t n_chrom, uint64_t n, BinLayout* L) {
    BinGeom g;
    if (!bin_geometry(chrom_len, n_chrom, &g)) return false;
    L->ncells = g.cb[n_chrom];
    uint64_t with_cells = 0;
    for (uint32_t k = 0; k < n_chrom; ++k) with_cells += g.cb[k + 1] > g.cb[k];
    const uint64_t bound = with_cells + (2 * n) / kRegionKeys;
    L->nreg_max = L->ncells < bound ? L->ncells : bound;
    const uint64_t sp = L->nreg_max ? (kSearchWorkgroups + L->nreg_max - 1) / L->nreg_max : 1;
    L->splits = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(sp, 1), kMaxSplits);
    return true;
}

hipError_t launch_bin_regions(const uint32_t* chrom_len, uint32_t n_chrom, const McTable& tab, uint64_t na, const uint32_t* bs, const uint32_t* be,
                              uint32_t n, const BinWs& w, uint32_t* status, hipStream_t s) {
    BinGeom g;
    if (!bin_geometry(chrom_len, n_chrom, &g)) return hipErrorInvalidValue;
    const uint32_t ncells = g.cb[n_chrom];
    if (!ncells || !n) return hipErrorInvalidValue;
    const uint32_t gr = (uint32_t)std::min<uint64_t>((ncells + 255) / 256, 4096);
    hipLaunchKernelGGL(k_bin_cells, dim3(gr), dim3(256), 0, s, g, bs, be, n, w.rs, w.re, w.nreg);
    hipLaunchKernelGGL(k_bin_regions, dim3(n_chrom), dim3(kBinThreads), 0, s, g, w.rs, w.re, n, w.nreg_max,
                       w.cell_region, reinterpret_cast<RegionDesc*>(w.desc), w.nreg, tab.hist, bin_most(na, n_chrom), status);
    return hipGetLastError();
}

hipError_t launch_bin_batch(const uint32_t* chrom_len, uint32_t n_chrom, const McTable& tab, uint64_t na,
                            const uint32_t* bs, const uint32_t* be, uint32_t n, uint64_t seed, uint64_t sb,
                            uint32_t nb, const BinWs& w, unsigned long long* totals, hipStream_t s,
                            hipEvent_t* ev) {
    BinGeom g;
    if (!bin_geometry(chrom_len, n_chrom, &g)) return hipErrorInvalidValue;
    if (nb == 0 || nb > BITS_MC_BIN_MAX_BATCH) return hipErrorInvalidValue;
    hipError_t e;
    if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
    // Shuffles per workgroup: groups of more than kGroupRecs entries take long enough
    // by themselves; of the others, as many as leave `rounds` workgroups for each of the
    // two slots a CU has: one when a workgroup's few shuffles are mostly latency, two when
    // they are many (a few workgroups too many are a second round of them: 2e4 entries x
    // 1000 184 us of placement at one round, 141 at two; 2000 x 100 18.6, 23.9), up to 6
    // so that the last round costs little (1e5 entries x 2000: 3, 6, 10 rounds 671, 648, 658 us).
    const uint64_t groups = (uint64_t)n_chrom * nb, mean = na / n_chrom;
    const uint64_t few = groups < 32u * (uint64_t)device_cu_count() ? 1 : 2;
    const uint64_t rounds = std::min<uint64_t>(std::max<uint64_t>(mean / 512, few), 6);
    const uint64_t slots = 2u * rounds * (uint64_t)device_cu_count();
    const uint32_t per = mean > kGroupRecs ? 1u : (uint32_t)std::min<uint64_t>((groups + slots - 1) / slots, nb);
    const uint64_t wgs = n_chrom * ((nb + per - 1ull) / per);
    const auto place = per == 1 ? k_bin_place<false> : k_bin_place<true>;
    hipLaunchKernelGGL(place, dim3((uint32_t)(per == 1 ? wgs : wgs + n_chrom)), dim3(kBinThreads), 0, s, g,
                       reinterpret_cast<const uint2*>(w.packed), tab.hist, tab.cursor, na, seed, sb, nb, per,
                       w.cell_region, w.nreg, w.nreg_max, w.seg_start, w.seg_cnt, reinterpret_cast<uint2*>(w.recs));
    if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
    if (w.splits > 1)
        hipLaunchKernelGGL(k_bin_search<true>, dim3(w.nreg_max * w.splits), dim3(kBinThreads), 0, s, bs, be, n,
                           reinterpret_cast<const RegionDesc*>(w.desc), w.nreg, w.seg_start, w.seg_cnt,
                           w.nreg_max, nb, reinterpret_cast<const uint2*>(w.recs), na, w.splits, w.partial);
    else
        hipLaunchKernelGGL(k_bin_search<false>, dim3(w.nreg_max), dim3(kBinThreads), 0, s, bs, be, n,
                           reinterpret_cast<const RegionDesc*>(w.desc), w.nreg, w.seg_start, w.seg_cnt,
                           w.nreg_max, nb, reinterpret_cast<const uint2*>(w.recs), na, 1u, w.partial);
    if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
    // about 8 region shares per thread, at most 512 partial sums per shuffle into the atomics
    const uint32_t gy = (uint32_t)std::min<uint64_t>(std::max<uint64_t>((uint64_t)w.nreg_max * w.splits / 8, 1), 512);
    hipLaunchKernelGGL(k_bin_reduce, dim3((nb + 255) / 256, gy), dim3(256), 0, s, w.partial, w.nreg,
                       w.splits, nb, totals);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[3], s)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace bits
