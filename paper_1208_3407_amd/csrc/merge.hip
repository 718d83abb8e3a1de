// All pairs of many query sets and many references at once (the many-pairs
// screen of Sec. 3.3), for gfx950.
//
// A pair's total is sum over its queries of #{B_S <= a.end} minus the same
// sum of #{B_E < a.start} (Algorithm 1), and each of the two sums may take
// the query keys in any order.  So the ends of all query sets are sorted
// into one list, tagged with their set, and the starts into another (once per
// replay, for all references), and the lists are walked in chunks:
//   splits  the rank of every chunk's first key in every reference;
//   count   one workgroup per chunk and 64 references, one reference per
//           lane: the references' keys that fall inside the chunk are placed
//           between its query keys by bisection in LDS (a histogram over
//           position and reference), and a running sum down the positions is
//           then the rank of each query key in 64 references at once, added
//           to the accumulators of the key's set;
//   reduce  the workgroups' accumulators are added into the pair totals.
// Every reference key is read once and every query key costs one LDS read
// and one LDS add per 64 references, in place of a search per pair.
#include <algorithm>

#include "bits_internal.hpp"

namespace bits {

namespace {

constexpr uint32_t kMergeThreads = 1024;
constexpr uint32_t kMergeWaves = kMergeThreads / kWave;
constexpr uint32_t kChunk = 256;                     // query keys per chunk
constexpr uint32_t kPerWave = kChunk / kMergeWaves;  // positions a wave walks
// Reference keys of a chunk counted through the histogram (16-bit counters); a
// reference with more in one chunk is searched by the chunk's keys instead, and
// where all have more than kDenseChunk together, already one with more than
// kDenseSlice.  Placing a key costs a chain of reads (1024 keys in about a
// microsecond), the searches one of steps (four references at once in 10 to 15).
// 8 sets of 1e5 against 64 references of 1e4 to 5e5 that all lie within 4e6 bp:
// 1310 us searched by 256 threads a reference at a time, 333 so (452 pair by pair).
constexpr uint32_t kLongSlice = 4096, kDenseSlice = 512, kDenseChunk = 1u << 16;
constexpr uint32_t kNoSet = 0xFFFFFFFFu;
constexpr uint32_t kQuarters = kMergeThreads / kChunk;
static_assert(kWave % kQuarters == 0, "long slices");
static_assert(kLongSlice < 65536, "histogram counters are 16-bit");

// The query sets' keys one after another (set i at offs[i]): ends into ks,
// starts into ke, the set number into sid (kNoSet and the interval flag for a
// query with start > end, which counts nothing).
__global__ void __launch_bounds__(256) k_merge_gather(const BatchQuery* __restrict__ qs, const uint32_t* __restrict__ offs,
                                                      uint32_t n_q, uint32_t total, uint32_t* __restrict__ ks,
                                                      uint32_t* __restrict__ ke, uint32_t* __restrict__ sid,
                                                      uint32_t* status) {
    uint32_t bad = 0;
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
        uint32_t lo = 0, hi = n_q;   // last set with offs[lo] <= t
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (offs[mid] <= t) lo = mid; else hi = mid;
        }
        const uint32_t i = t - offs[lo];
        const uint32_t s = qs[lo].as[i], e = qs[lo].ae[i];
        ks[t] = e;
        ke[t] = s;
        sid[t] = s <= e ? lo : kNoSet;
        bad |= s > e ? 1u : 0u;
    }
    if (bad) atomicOr(status, BITS_FLAG_INTERVAL);
}

// #{K[0..n) <= x} (ends against B_S) or #{K[0..n) < x} (starts against B_E).
__device__ __forceinline__ uint32_t rank_of(const uint32_t* __restrict__ K, uint32_t lo, uint32_t n, uint32_t x,
                                            bool strict) {
    uint32_t len = n;
    while (len) {
        const uint32_t half = len >> 1, k = K[lo + half];
        const bool below = strict ? k < x : k <= x;
        lo = below ? lo + half + 1 : lo;
        len = below ? len - half - 1 : half;
    }
    return lo;
}

// splits[(a * (chunks + 1) + c) * n_ref + j]: the rank of chunk c's first key
// of list a in reference j, and for c = chunks that of the list's last key.
// A thread bisects for kSplitPer chunks at once, so that their dependent
// loads overlap.
constexpr int kSplitPer = 4;
__global__ void __launch_bounds__(256) k_merge_splits(const BatchRef* __restrict__ refs, uint32_t n_ref,
                                                      const uint32_t* __restrict__ ks, const uint32_t* __restrict__ ke,
                                                      uint32_t total, uint32_t chunks, uint32_t* __restrict__ splits) {
    const uint32_t c0 = blockIdx.x * 256 * kSplitPer + threadIdx.x, j = blockIdx.y, a = blockIdx.z;
    const BatchRef R = refs[j];
    const uint32_t* __restrict__ K = a ? R.be : R.bs;
    uint32_t x[kSplitPer], lo[kSplitPer];
#pragma unroll
    for (int u = 0; u < kSplitPer; ++u) {
        x[u] = (a ? ke : ks)[min((uint64_t)(c0 + 256u * u) * kChunk, (uint64_t)total - 1u)];
        lo[u] = 0u;
    }
    uint32_t len = R.n;   // #{K <= x} or #{K < x} is in [lo, lo + len]
    while (len) {
        const uint32_t half = (len + 1u) >> 1;   // the same steps for every key; lo + half may pass n by rounding
        uint32_t k[kSplitPer];
#pragma unroll
        for (int u = 0; u < kSplitPer; ++u) k[u] = K[min(lo[u] + half, R.n) - 1u];
#pragma unroll
        for (int u = 0; u < kSplitPer; ++u) {
            const bool below = a ? k[u] < x[u] : k[u] <= x[u];
            lo[u] = below ? min(lo[u] + half, R.n) : lo[u];
        }
        len = len > 1u ? len - half : 0u;
    }
#pragma unroll
    for (int u = 0; u < kSplitPer; ++u) {
        const uint32_t c = c0 + 256u * u;
        if (c <= chunks) splits[((uint64_t)a * (chunks + 1) + c) * n_ref + j] = lo[u];
    }
}

// Sum over the lanes up to this one.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= (uint32_t)o) x += y;
    }
    return x;
}

// Workgroup w of group g (64 references) takes every W-th, from the w-th on, of
// the group's 2 * chunks (list, chunk) tasks and writes its sums,
// ends' ranks minus starts' ranks modulo 2^64, to part[((g W + w) n_q + i) 64 + lane].
// Dynamic LDS: the accumulators, n_q * 64 uint64.
// (Neighbouring chunks go to different workgroups so that none has all the
// chunks of a place where the references are dense: 333 us for those 64
// references, 804 with tasks in a row; elsewhere within 2%, mostly faster.)
// What bounds it: the latency of a chunk's steps between its six barriers
// (slice bounds, reference keys, bisections), so waves per CU decide: 32 sets
// of 3e6 keys in all against 64 references of 5e6 took 395 us with 512 threads
// a workgroup and three a CU, 307 with 1024 and a third one waiting, 284 with
// two of 1024 (chunks of 128 keys and four of 512: 263, but the splits then
// cost more).
__global__ void __launch_bounds__(kMergeThreads, 8) k_merge_count(
    const BatchRef* __restrict__ refs, uint32_t n_ref, uint32_t n_q, const uint32_t* __restrict__ ks,
    const uint32_t* __restrict__ ke, const uint32_t* __restrict__ ss, const uint32_t* __restrict__ se, uint32_t total,
    uint32_t chunks, const uint32_t* __restrict__ splits, unsigned long long* __restrict__ part) {
    extern __shared__ __align__(16) unsigned long long acc[];   // [n_q][64]
    __shared__ __align__(16) uint32_t hist[kChunk * kWave / 2];  // 16-bit counters [position][reference]
    __shared__ uint32_t key[kChunk], set[kChunk];
    __shared__ uint32_t first[kWave], base[kWave], pre[kWave + 1], len[kWave];
    __shared__ uint32_t wsum[kMergeWaves][kWave];
    __shared__ const uint32_t* arr[2][kWave];   // the group's B_S and B_E
    const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const uint32_t g = blockIdx.y, j0 = g * kWave;
    if (threadIdx.x < 2 * kWave) {
        const BatchRef& R = refs[min(j0 + lane, n_ref - 1u)];
        arr[wv][lane] = wv ? R.be : R.bs;
    }
    for (uint32_t k = threadIdx.x; k < n_q * kWave; k += kMergeThreads) acc[k] = 0ull;
    const uint32_t tasks = 2u * chunks;
    for (uint32_t t = blockIdx.x; t < tasks; t += gridDim.x) {
        const uint32_t a = t >= chunks ? 1u : 0u, c = t - a * chunks;
        const uint32_t b0 = c * kChunk, cnt = min(kChunk, total - b0);
        __syncthreads();   // the previous task is done with the LDS
        for (uint32_t k = threadIdx.x; k < kChunk * kWave / 8; k += kMergeThreads)
            reinterpret_cast<uint4*>(hist)[k] = make_uint4(0u, 0u, 0u, 0u);
        if (threadIdx.x < kChunk) {
            const bool in = threadIdx.x < cnt;
            key[threadIdx.x] = in ? (a ? ke : ks)[b0 + threadIdx.x] : 0xFFFFFFFFu;
            set[threadIdx.x] = in ? (a ? se : ss)[b0 + threadIdx.x] : kNoSet;
        } else if (wv == kMergeWaves - 1) {   // one lane per reference: its slice of the chunk
            const uint32_t* sp = splits + ((uint64_t)a * (chunks + 1) + c) * n_ref + j0;
            const bool in = j0 + lane < n_ref;
            const uint32_t r0 = in ? sp[lane] : 0u, r1 = in ? sp[n_ref + lane] : 0u;
            const uint32_t l = r1 - r0;
            uint32_t s = l <= kLongSlice ? l : 0u, x = wave_prefix(s);
            if (__shfl(x, kWave - 1) > kDenseChunk) {   // uniform
                s = l <= kDenseSlice ? l : 0u;
                x = wave_prefix(s);
            }
            first[lane] = r0;
            len[lane] = l - s;   // searched
            base[lane] = s == l ? r0 : 0u;
            pre[lane] = x - s;
            if (lane == kWave - 1) pre[kWave] = x;
        }
        __syncthreads();
        // every reference key of the slices, between the chunk's query keys
        const uint32_t m = pre[kWave];
        for (uint32_t q = threadIdx.x; q < m; q += kMergeThreads) {
            uint32_t lo = 0, hi = kWave;   // last reference with pre <= q
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (pre[mid] <= q) lo = mid; else hi = mid;
            }
            const uint32_t b = arr[a][lo][first[lo] + (q - pre[lo])];
            // first position whose key counts b: key >= b (ends) or key > b (starts)
            uint32_t p = 0;
#pragma unroll
            for (uint32_t h = kChunk / 2; h; h >>= 1) {
                const uint32_t x = key[p + h - 1];
                p += (a ? x <= b : x < b) ? h : 0u;
            }
            p += (a ? key[p] <= b : key[p] < b) ? 1u : 0u;
            if (p < cnt) atomicAdd(&hist[p * (kWave / 2) + lo / 2], 1u << (16 * (lo & 1u)));
        }
        // references with long slices: a search per query key, each quarter of the workgroup
        // for another reference
        for (uint64_t left = __ballot(len[lane] != 0u); left;) {
            const uint32_t j1 = (uint32_t)__builtin_ctzll(left) / kQuarters * kQuarters;
            left &= ~(((1ull << kQuarters) - 1ull) << j1);
            const uint32_t k = threadIdx.x % kChunk, j = j1 + threadIdx.x / kChunk;
            if (k < cnt && len[j] && set[k] != kNoSet) {
                const uint64_t r = rank_of(arr[a][j], first[j], len[j], key[k], a != 0);
                atomicAdd(&acc[set[k] * kWave + j], (unsigned long long)(a ? 0ull - r : r));
            }
        }
        __syncthreads();
        // lane j walks reference j: the wave's positions, after the sums of the waves before it
        const uint16_t* H = reinterpret_cast<const uint16_t*>(hist) + wv * kPerWave * kWave + lane;
        uint32_t h[kPerWave], sum = 0;
#pragma unroll
        for (uint32_t k = 0; k < kPerWave; ++k) {
            h[k] = H[k * kWave];
            sum += h[k];
        }
        wsum[wv][lane] = sum;
        __syncthreads();
        uint32_t r = base[lane];
        for (uint32_t k = 0; k < wv; ++k) r += wsum[k][lane];
#pragma unroll
        for (uint32_t k = 0; k < kPerWave; ++k) {
            r += h[k];
            const uint32_t i = __builtin_amdgcn_readfirstlane(set[wv * kPerWave + k]);
            if (i != kNoSet) atomicAdd(&acc[i * kWave + lane], a ? 0ull - (unsigned long long)r : (unsigned long long)r);
        }
    }
    __syncthreads();
    unsigned long long* out = part + ((uint64_t)g * gridDim.x + blockIdx.x) * n_q * kWave;
    for (uint32_t k = threadIdx.x; k < n_q * kWave; k += kMergeThreads) out[k] = acc[k];
}

// totals[i * n_ref + j] = sum over the workgroups of reference j's group.
// blockIdx.x = i, blockIdx.y = g; wave w of the workgroup takes every 16th.
__global__ void __launch_bounds__(1024) k_merge_reduce(const unsigned long long* __restrict__ part, uint32_t n_wg,
                                                       uint32_t n_q, uint32_t n_ref,
                                                       unsigned long long* __restrict__ totals) {
    constexpr uint32_t kWaves = 1024 / kWave;
    __shared__ unsigned long long s[kWaves][kWave];
    const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, i = blockIdx.x, g = blockIdx.y;
    const unsigned long long* P = part + ((uint64_t)g * n_wg * n_q + i) * kWave + lane;
    const uint64_t step = (uint64_t)n_q * kWave;
    unsigned long long v = 0ull;
#pragma unroll 8
    for (uint32_t w = wv; w < n_wg; w += kWaves) v += P[w * step];
    s[wv][lane] = v;
    __syncthreads();
    const uint32_t j = g * kWave + lane;
    if (wv == 0 && j < n_ref) {
        v = 0ull;
        for (uint32_t k = 0; k < kWaves; ++k) v += s[k][lane];
        totals[(uint64_t)i * n_ref + j] = v;
    }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

bool merge_layout(const uint64_t* na, uint32_t n_q, uint32_t n_ref, MergeLayout* L) {
    uint64_t total = 0;
    for (uint32_t i = 0; i < n_q; ++i) {
        if (na[i] > kMergeMaxKeys) return false;
        total += na[i];
    }
    if (n_q > kMergeMaxSets || n_ref > kMergeMaxRefs || total > kMergeMaxKeys ||
        total * n_ref < kMergeMinEvaluations)
        return false;
    L->total = (uint32_t)total;
    L->chunks = (uint32_t)((total + kChunk - 1) / kChunk);
    L->groups = (n_ref + kWave - 1) / kWave;
    // two workgroups per CU while their LDS (42 KB and the accumulators) fits it
    const uint32_t per_cu = (42u << 10) + n_q * kWave * 8u <= (80u << 10) ? 2u : 1u;
    L->wgs = std::max(1u, std::min(2u * L->chunks, kMergeCus * per_cu / L->groups));
    size_t o = 0;
    const size_t col = align256((size_t)total * 4);
    L->offs = o; o = align256(o + (size_t)(n_q + 1) * 4);
    L->in = o; o += 2 * col;
    L->sid = o; o += col;
    L->out = o; o += 2 * col;
    L->sets = o; o += 2 * col;
    L->splits = o; o = align256(o + (size_t)2 * (L->chunks + 1) * n_ref * 4);
    L->part = o; o = align256(o + (size_t)L->groups * L->wgs * n_q * kWave * 8);
    L->sort = o;
    const uint64_t ns[2] = {total, total};
    const uint32_t vm[2] = {1u, 1u};
    L->sort_bytes = sort_workspace_bytes(ns, 2, vm);
    o = align256(o + L->sort_bytes);
    L->bytes = o;
    return true;
}

// Microseconds of both forms from measured rates (8 sets of 2e3 to 5e5 queries
// against 2 to 128 references of 2e4, 2e5 and 2e6): a search takes 17, 25 and
// 60 ps per query by the reference's size; the sorted form 140 us (its
// launches), 0.13 ns per query key and 64 references and 13 ps per reference
// key.  Either side of the line: 1e6 queries against 8 of 2e6 keys 521 us
// searched and 433 sorted, against 16 of 2e4 320 and 262, against 8 of 2e4 172
// and 260; 2.6e5 against 32 of 2e6 542 and 1031, against 64 of 2e5 713 and 334.
bool merge_pays(const MergeLayout& L, const uint64_t* nb, uint32_t n_ref) {
    double search = 0.0, merge = 140.0 + 0.13e-3 * L.total * L.groups;
    for (uint32_t j = 0; j < n_ref; ++j) {
        search += L.total * (nb[j] < (1u << 16) ? 17e-6 : nb[j] < (1u << 19) ? 25e-6 : 60e-6);
        merge += 13e-6 * (double)nb[j];
    }
    return search > merge;
}

int launch_merge(const BatchRef* refs, uint32_t n_ref, const BatchQuery* qs, uint32_t n_q, const MergeLayout& L, void* ws,
                 unsigned long long* totals, uint32_t* status, hipStream_t s) {
    char* b = (char*)ws;
    const size_t col = align256((size_t)L.total * 4);
    uint32_t* offs = (uint32_t*)(b + L.offs);
    uint32_t *in_s = (uint32_t*)(b + L.in), *in_e = (uint32_t*)(b + L.in + col), *sid = (uint32_t*)(b + L.sid);
    uint32_t *out_s = (uint32_t*)(b + L.out), *out_e = (uint32_t*)(b + L.out + col);
    uint32_t *set_s = (uint32_t*)(b + L.sets), *set_e = (uint32_t*)(b + L.sets + col);
    uint32_t* splits = (uint32_t*)(b + L.splits);
    auto* part = (unsigned long long*)(b + L.part);
    const uint32_t gg = std::min<uint32_t>((L.total + 255) / 256, 4096);
    hipLaunchKernelGGL(k_merge_gather, dim3(gg), dim3(256), 0, s, qs, offs, n_q, L.total, in_s, in_e, sid, status);
    const SortSeg segs[2] = {{in_s, out_s, L.total, 1u, sid, set_s, status}, {in_e, out_e, L.total, 1u, sid, set_e, status}};
    const int rc = launch_sort(segs, 2, b + L.sort, L.sort_bytes, s);
    if (rc != BITS_OK) return rc;
    hipLaunchKernelGGL(k_merge_splits, dim3((L.chunks + 256 * kSplitPer) / (256 * kSplitPer), n_ref, 2), dim3(256), 0, s, refs, n_ref, out_s,
                       out_e, L.total, L.chunks, splits);
    hipLaunchKernelGGL(k_merge_count, dim3(L.wgs, L.groups), dim3(kMergeThreads), (size_t)n_q * kWave * 8, s, refs,
                       n_ref, n_q, out_s, out_e, set_s, set_e, L.total, L.chunks, splits, part);
    hipLaunchKernelGGL(k_merge_reduce, dim3(n_q, L.groups), dim3(1024), 0, s, part, L.wgs, n_q, n_ref, totals);
    BITS_CHECK_HIP(hipGetLastError());
    return BITS_OK;
}

}  // namespace bits
