// Search kernels of libbits.so (gfx950): ICount (Algorithm 1) over the plain
// index (LDS Eytzinger top tree + bisection of the bucket in HBM), the same
// tree with interpolated windows of line heads or keys, or the
// learned CDF index (route -> leaf model -> one cooperative 128-byte line
// probe at the predicted rank -> bisection of what is left of the error
// window -> verification), the per-query / total counters (Algorithm 2),
// the Monte-Carlo loop of Sec. 3.2 as one persistent launch, the
// batched-pairs kernel, projection and small helpers.
//
// Every lane carries QPL queries, i.e. 2*QPL independent search chains (one
// over B_S for a.end, one over B_E for a.start per query); the chains advance
// in lock-step so their dependent loads overlap.  Loads of the sorted arrays
// that have no reuse are non-temporal, so the learned leaf records and the
// shared top of the bisections stay in L2.
#include <mutex>
#include <unordered_map>

#include "bits_internal.hpp"
#include "near.hpp"

// Waves per SIMD the search kernels are compiled for (caps their VGPRs).
#ifndef BITS_SEARCH_WAVES_PER_EU
#define BITS_SEARCH_WAVES_PER_EU 4
#endif
#define BITS_SEARCH_KERNEL __global__ void __launch_bounds__(1024) \
    __attribute__((amdgpu_waves_per_eu(BITS_SEARCH_WAVES_PER_EU)))

namespace bits {

using u32x4 = uint32_t __attribute__((ext_vector_type(4)));

template <bool NT>
__device__ __forceinline__ uint32_t ld_key(const uint32_t* p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The sorted arrays a search of several chains runs over, with their line heads
// and models: even chains take k[0], odd ones k[1].  A search of one array has
// it in both places.
struct Arrays {
    const uint32_t* k[2];
    const uint32_t* h[2];
    const bits_rmi_model* m[2];
    uint32_t n;
};
__device__ __forceinline__ Arrays both_arrays(const SearchArgs& sa) {
    return Arrays{{sa.bs, sa.be}, {sa.hs, sa.he}, {sa.rmi, sa.rmi ? sa.rmi + 1 : nullptr}, sa.n};
}
__device__ __forceinline__ Arrays one_array(const SearchArgs& sa, int which) {
    const Arrays a = both_arrays(sa);
    return Arrays{{a.k[which], a.k[which]}, {a.h[which], a.h[which]}, {a.m[which], a.m[which]}, a.n};
}

// ------------------------------------------------------------------ bisection
// For each chain c: base[c] += #{K_c[base[c] .. base[c] + len[c]) < x[c]};
// K_c is B_S for even c and B_E for odd c.  Leaves len[c] == 0.  The first
// `hot` probes are ordinary (cached) loads, later ones non-temporal.
template <int NC>
__device__ __forceinline__ void bisect_multi(const uint32_t* __restrict__ ks, const uint32_t* __restrict__ ke,
                                             uint32_t (&base)[NC], uint32_t (&len)[NC], const uint32_t (&x)[NC],
                                             uint32_t hot) {
    for (uint32_t step = 0;; ++step) {
        uint32_t v[NC];
        bool any = false;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t* K = (c & 1) ? ke : ks;
            const uint32_t half = len[c] >> 1;
            // a finished chain reads key 0 (always in bounds); its value is unused.
            // A probe is streamed (non-temporal) unless it is one of the shared
            // first probes or the range is down to ~2 lines, which the next
            // probes read again.
            const uint32_t idx = half ? base[c] + half - 1 : 0u;
            if (step < hot || len[c] <= 64u)
                v[c] = ld_key<false>(K + idx);
            else
                v[c] = ld_key<true>(K + idx);
            any |= half != 0;
        }
        if (!any) break;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t half = len[c] >> 1;
            if (half) {
                base[c] += (v[c] < x[c]) ? half : 0u;
                len[c] -= half;
            }
        }
    }
    uint32_t v[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t* K = (c & 1) ? ke : ks;
        v[c] = len[c] ? ld_key<false>(K + base[c]) : 0u;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (len[c]) base[c] += (v[c] < x[c]) ? 1u : 0u;
        len[c] = 0;
    }
}

// ------------------------------------------------------------------ line probe
// For every lane's chains with start[c] != kNoLine:
//   cnt[c] = #{i in [start[c], start[c] + 32) : K_c[i] < x[c]},
// start a multiple of 4 (16-byte aligned).  On a sorted array probed at a
// 128-byte line (start = 32 line), 0 < cnt < 32 pins the global lower bound
// to start + cnt exactly.  The sorted arrays are 256-byte aligned inside the
// reference block and the rest of their last 128-byte line holds 0xFFFFFFFF
// (never < x), so every line read is in bounds and needs no masking; the
// line-head arrays are padded the same way.  The whole wave cooperates:
// kProbeLanes lanes read one 32-word window with 16-byte loads (each load
// instruction covering a contiguous 16 * kProbeLanes bytes of every window
// it touches) and their partial counts are summed with DPP lane moves.  NT
// selects non-temporal loads (data lines, no reuse) over cached ones (line
// heads, kept in L2).  `scr` is this wave's LDS scratch of 4 * NC * 64
// words.  Must be called by all 64 lanes.

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

__device__ __forceinline__ uint32_t count_lt4(u32x4 v, uint32_t x) {
    return (v.x < x ? 1u : 0u) + (v.y < x ? 1u : 0u) + (v.z < x ? 1u : 0u) + (v.w < x ? 1u : 0u);
}

#ifndef BITS_QUAD_SHFL
#define BITS_QUAD_SHFL 0
#endif
#ifndef BITS_PROBE_LANES
#define BITS_PROBE_LANES 8
#endif
constexpr int kProbeLanes = BITS_PROBE_LANES;        // lanes reading one line

// Sum over each aligned group of L lanes, in every lane of the group.
template <int L>
__device__ __forceinline__ uint32_t group_sum(uint32_t t) {
    if constexpr (L >= 2) t += dpp_u32<0xB1>(t);    // quad_perm [1,0,3,2]
    if constexpr (L >= 4) t += dpp_u32<0x4E>(t);    // quad_perm [2,3,0,1]
    if constexpr (L >= 8) t += dpp_u32<0x141>(t);   // row_half_mirror
    return t;
}

// WIN words per window (32: a 128-byte line; 16: half a line), read by
// LANES lanes with WIN / (4 LANES) 16-byte loads each.
template <int NC, bool NT, int WIN = 32, int LANES = kProbeLanes>
__device__ __forceinline__ void probe_lines(const uint32_t* __restrict__ ks, const uint32_t* __restrict__ ke,
                                            const uint32_t (&start)[NC], const uint32_t (&x)[NC],
                                            uint32_t (&cnt)[NC], uint32_t* scr) {
    constexpr int kLanes = LANES;
    constexpr int kLoads = WIN / 4 / LANES;      // 16-byte loads per lane per window
    constexpr int kGroups = kWave / LANES;       // windows per instruction
    static_assert(kLoads >= 1 && WIN % (4 * LANES) == 0, "window geometry");
    const uint32_t lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        // an idle lane probes words 0..31 against x = 0 (counts nothing, result unused)
        const bool on = start[c] != kNoLine;
        scr[(2 * c + 0) * 2 * kWave + 2 * lane] = on ? start[c] : 0u;
        scr[(2 * c + 0) * 2 * kWave + 2 * lane + 1] = on ? x[c] : 0u;
    }
    wave_lds_sync();
    const uint32_t sub = lane % kLanes, grp = lane / kLanes;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t* K = (c & 1) ? ke : ks;
        u32x4 v[kLanes][kLoads];
        uint32_t xx[kLanes];
#pragma unroll
        for (int j = 0; j < kLanes; ++j) {
            const uint32_t owner = (uint32_t)j * kGroups + grp;
            const uint2 lx = *reinterpret_cast<const uint2*>(scr + (2 * c + 0) * 2 * kWave + 2 * owner);
            xx[j] = lx.y;
            // load k covers bytes [16 k L, 16 (k + 1) L) of the window (L lanes), contiguous per group
            const u32x4* P = reinterpret_cast<const u32x4*>(K + lx.x) + sub;
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                if constexpr (NT)
                    v[j][k] = __builtin_nontemporal_load(P + k * kLanes);
                else
                    v[j][k] = P[k * kLanes];
            }
        }
#pragma unroll
        for (int j = 0; j < kLanes; ++j) {
            const uint32_t owner = (uint32_t)j * kGroups + grp;
            uint32_t t = 0;
#pragma unroll
            for (int k = 0; k < kLoads; ++k) t += count_lt4(v[j][k], xx[j]);
            t = group_sum<LANES>(t);
            if (sub == 0) scr[(2 * c + 1) * 2 * kWave + owner] = t;
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < NC; ++c) cnt[c] = scr[(2 * c + 1) * 2 * kWave + lane];
    wave_lds_sync();
}

// ------------------------------------------------------------------ probes in registers
// The same counts without LDS memory, for the search that keeps its LDS for
// the top trees.  A group of lanes serves its own lanes in turn: in pass j the
// group counts lane j's window, whose start and key the others read by a lane
// broadcast, each lane taking 16 bytes of it.
//   quads  windows of WIN words, 64 contiguous bytes per load and quad
//          (quad_perm broadcasts);
//   octs   128-byte windows, one load each: a line read by one instruction is
//          one request, by two it is two (1e7 queries against 1e7: 702 us with
//          the data lines read by octs, 798 by quads); ds_swizzle broadcasts.
template <int J>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v) {
    int r = __builtin_amdgcn_update_dpp(0, (int)v, J * 0x55, 0xF, 0xF, true);
    asm volatile("" : "+v"(r));   // kept a move of its own, not folded into its use
    return (uint32_t)r;
}

template <int J>
__device__ __forceinline__ uint32_t oct_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (J << 5) | 0x18);   // lane (l & 24) | J of each 32
}

// The 16-byte pieces of the windows of the quad's lane J.
template <int J, int LOADS>
__device__ __forceinline__ void quad_load(const uint32_t* __restrict__ K, uint32_t start, u32x4 (&v)[LOADS]) {
    const u32x4* P = reinterpret_cast<const u32x4*>(K + quad_bcast<J>(start)) + (threadIdx.x & 3u);
#pragma unroll
    for (int k = 0; k < LOADS; ++k) v[k] = P[4 * k];
}

template <int J, int LOADS>
__device__ __forceinline__ void quad_sum(const u32x4 (&v)[LOADS], uint32_t x, uint32_t& res) {
    const uint32_t xx = quad_bcast<J>(x);
    uint32_t t = 0;
#pragma unroll
    for (int k = 0; k < LOADS; ++k) t += count_lt4(v[k], xx);
    t = group_sum<4>(t);
    if ((threadIdx.x & 3u) == (uint32_t)J) res = t;
}

// cnt[c] = #{i in [start[c], start[c] + WIN) : K_c[i] < x[c]}, start a
// multiple of 4 with the whole window inside K_c; all 64 lanes call it, an
// idle chain passes any start in bounds.  The loads of all chains are issued
// before the first count.
template <int NC, int WIN>
__device__ __forceinline__ void quad_windows(const uint32_t* __restrict__ ks, const uint32_t* __restrict__ ke,
                                             const uint32_t (&start)[NC], const uint32_t (&x)[NC],
                                             uint32_t (&cnt)[NC]) {
    constexpr int kLoads = WIN / 16;
    static_assert(WIN % 16 == 0, "window geometry");
    u32x4 v[NC][4][kLoads];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t* K = (c & 1) ? ke : ks;
        quad_load<0, kLoads>(K, start[c], v[c][0]);
        quad_load<1, kLoads>(K, start[c], v[c][1]);
        quad_load<2, kLoads>(K, start[c], v[c][2]);
        quad_load<3, kLoads>(K, start[c], v[c][3]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        uint32_t r = 0;
        quad_sum<0, kLoads>(v[c][0], x[c], r);
        quad_sum<1, kLoads>(v[c][1], x[c], r);
        quad_sum<2, kLoads>(v[c][2], x[c], r);
        quad_sum<3, kLoads>(v[c][3], x[c], r);
        cnt[c] = r;
    }
}

template <int J, bool NT>
__device__ __forceinline__ u32x4 oct_load(const uint32_t* __restrict__ K, uint32_t start) {
    const u32x4* P = reinterpret_cast<const u32x4*>(K + oct_bcast<J>(start)) + (threadIdx.x & 7u);
    if constexpr (NT)
        return __builtin_nontemporal_load(P);
    else
        return *P;
}

template <int J>
__device__ __forceinline__ void oct_sum(u32x4 v, uint32_t x, uint32_t& res) {
    const uint32_t t = group_sum<8>(count_lt4(v, oct_bcast<J>(x)));
    if ((threadIdx.x & 7u) == (uint32_t)J) res = t;
}

// As quad_windows for 32 words, by octs.
template <int NC, bool NT>
__device__ __forceinline__ void oct_windows(const uint32_t* __restrict__ ks, const uint32_t* __restrict__ ke,
                                            const uint32_t (&start)[NC], const uint32_t (&x)[NC], uint32_t (&cnt)[NC]) {
    u32x4 v[NC][8];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t* K = (c & 1) ? ke : ks;
        v[c][0] = oct_load<0, NT>(K, start[c]);
        v[c][1] = oct_load<1, NT>(K, start[c]);
        v[c][2] = oct_load<2, NT>(K, start[c]);
        v[c][3] = oct_load<3, NT>(K, start[c]);
        v[c][4] = oct_load<4, NT>(K, start[c]);
        v[c][5] = oct_load<5, NT>(K, start[c]);
        v[c][6] = oct_load<6, NT>(K, start[c]);
        v[c][7] = oct_load<7, NT>(K, start[c]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        uint32_t r = 0;
        oct_sum<0>(v[c][0], x[c], r);
        oct_sum<1>(v[c][1], x[c], r);
        oct_sum<2>(v[c][2], x[c], r);
        oct_sum<3>(v[c][3], x[c], r);
        oct_sum<4>(v[c][4], x[c], r);
        oct_sum<5>(v[c][5], x[c], r);
        oct_sum<6>(v[c][6], x[c], r);
        oct_sum<7>(v[c][7], x[c], r);
        cnt[c] = r;
    }
}

// Windows of 32 words for the few lanes of `on` (not empty): the lowest eight
// of them are served at once, the k-th by oct k.  Returns the count in the
// lanes served, and in `on` the lanes that are.  All 64 lanes call it.
template <bool NT>
__device__ __forceinline__ uint32_t few_windows(const uint32_t* __restrict__ K, uint32_t start, uint32_t x, uint64_t& on) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    uint32_t owner = 0;
    uint64_t m = on, served = 0ull;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {   // m is uniform: the k-th lane of `on`, for oct k
        const uint32_t i = m ? (uint32_t)__builtin_ctzll(m) : (uint32_t)__builtin_ctzll(on);
        owner = lane / 8 == k ? i : owner;
        served |= m & (0ull - m);
        m &= m - 1;
    }
    const uint32_t w = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4 * owner), (int)start);
    const uint32_t y = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4 * owner), (int)x);
    const u32x4* P = reinterpret_cast<const u32x4*>(K + w) + (lane & 7u);
    u32x4 v;
    if constexpr (NT)
        v = __builtin_nontemporal_load(P);
    else
        v = *P;
    const uint32_t t = group_sum<8>(count_lt4(v, y));
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(on >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)on, 0u));
    on = served;
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(32 * (rank & 7u)), (int)t);
}

// Lower bounds by windows: on entry r_c = #{K_c < x[c]} lies in
// [lo[c], hi[c]] and near g[c]; on return lo[c] = r_c.  The first window sits
// around the guess, the second next to it on the side its count points to,
// later ones around the middle of what is left, so a bad guess costs speed
// only.  K_c is readable (and 0xFFFFFFFF past its keys) up to `lim`, a
// multiple of 4 and at least WIN.  All 64 lanes call it.
template <int NC, int WIN>
__device__ __forceinline__ void window_search(const uint32_t* __restrict__ ks, const uint32_t* __restrict__ ke,
                                              uint32_t lim, uint32_t (&lo)[NC], uint32_t (&hi)[NC],
                                              const uint32_t (&g)[NC], const uint32_t (&x)[NC]) {
    uint32_t w[NC], cnt[NC];
    bool any = false;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        // a range that one window covers needs no guess
        const uint32_t near = (g[c] > WIN / 2 - 4 ? g[c] - (WIN / 2 - 4) : 0u) & ~7u;
        w[c] = min(hi[c] - lo[c] <= WIN - 4 ? lo[c] & ~3u : near, lim - WIN);
        any |= lo[c] < hi[c];
    }
    for (uint32_t step = 0; __ballot(any); ++step) {
        quad_windows<NC, WIN>(ks, ke, w, x, cnt);
        any = false;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (lo[c] >= hi[c]) continue;
            const uint32_t r = w[c] + cnt[c];   // keys before the window are below x unless cnt is 0
            const bool left = cnt[c] == 0u, right = cnt[c] == (uint32_t)WIN;
            const uint32_t at = min(max(r, lo[c]), hi[c]);
            if (!left) lo[c] = at;
            if (!right) hi[c] = at;
            if (lo[c] >= hi[c]) continue;
            any = true;
            const uint32_t half = (hi[c] - lo[c]) / 2;
            uint32_t s = lo[c];                                  // covers the range, or its left end
            if (hi[c] - lo[c] > WIN - 4) {
                if (step)
                    s += half > WIN / 2 ? half - WIN / 2 : 0u;   // around the middle
                else if (left)
                    s = hi[c] - (WIN - 4);                       // up to the right end
            }
            w[c] = min(s & ~3u, lim - WIN);
        }
    }
}

// ------------------------------------------------------------------ leaf model
// Evaluates the leaf of every lane's chains cooperatively, 4 lanes per leaf:
// in pass p the quad k of the wave serves owner lane 16 p + k.  Lane q of
// the quad reads 16 bytes at 16 q and 16 bytes at 64 + 16 q of the owner's
// 128-byte leaf record (each instruction covers 64 contiguous bytes per
// quad): two header words and the binary16 weights of hidden units
// 4q..4q+3.  The quad adds its 4 partial sums with two lane-pair moves (the
// order b2 + ((s0 + s1) + (s2 + s3)) of rmi_pred_offset) and writes, per
// owner, {kmin, kmax, rlo, cnt, y, err} to LDS.  `scr` is this wave's
// scratch; chain c uses words [c * kLeafScr, (c + 1) * kLeafScr): 128 words
// of (leaf, x) pairs, then 6 result words per owner.  Must be called by all
// 64 lanes.

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_quad(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

template <int NC>
__device__ __forceinline__ void quad_leaves(const Arrays& A, const uint32_t (&leaf)[NC],
                                            const uint32_t (&x)[NC], uint32_t* scr) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        scr[c * kLeafScr + 2 * lane] = leaf[c];
        scr[c * kLeafScr + 2 * lane + 1] = x[c];
    }
    wave_lds_sync();
    const uint32_t quad = lane >> 2, q = lane & 3u;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const bits_rmi_model* M = A.m[c & 1];
        uint4 Q[4], B[4];
        uint32_t xo[4];
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const uint32_t owner = (uint32_t)pass * 16u + quad;
            const uint2 lx = *reinterpret_cast<const uint2*>(scr + c * kLeafScr + 2 * owner);
            xo[pass] = lx.y;
            const uint4* rec = reinterpret_cast<const uint4*>(M->leaf + lx.x);
            Q[pass] = rec[q];
            B[pass] = rec[4 + q];
        }
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const uint32_t owner = (uint32_t)pass * 16u + quad;
            // kmin from quad lane 0, kinv from quad lane 2 (lane exchanges: a quad_perm
            // broadcast DPP folded into the using instruction gave wrong values here)
            const uint32_t kmin = (uint32_t)__shfl((int)Q[pass].x, (int)(lane & ~3u));
            const uint32_t kinvb = (uint32_t)__shfl((int)Q[pass].x, (int)((lane & ~3u) + 2u));
            const float u = rmi_u(xo[pass] - kmin, __uint_as_float(kinvb));
            const float w1[4] = {h2f(Q[pass].z & 0xFFFFu), h2f(Q[pass].z >> 16), h2f(Q[pass].w & 0xFFFFu),
                                 h2f(Q[pass].w >> 16)};
            const float b1[4] = {h2f(B[pass].x & 0xFFFFu), h2f(B[pass].x >> 16), h2f(B[pass].y & 0xFFFFu),
                                 h2f(B[pass].y >> 16)};
            const float w2[4] = {h2f(B[pass].z & 0xFFFFu), h2f(B[pass].z >> 16), h2f(B[pass].w & 0xFFFFu),
                                 h2f(B[pass].w >> 16)};
            float t = rmi_quad_partial(w1, b1, w2, u);
#if BITS_QUAD_SHFL
            t += __shfl_xor(t, 1);   // s0+s1, s2+s3
            t += __shfl_xor(t, 2);   // (s0+s1)+(s2+s3)
#else
            t += __uint_as_float(dpp_quad<0xB1>(__float_as_uint(t)));   // s0+s1, s2+s3
            t += __uint_as_float(dpp_quad<0x4E>(__float_as_uint(t)));   // (s0+s1)+(s2+s3)
#endif
            // lane 0: {kmin, kmax}; 1: {rlo, cnt}; 2: y = b2 + sum; 3: err
            uint32_t* res = scr + c * kLeafScr + 2 * kWave + 6 * owner;
            if (q < 2)
                *reinterpret_cast<uint2*>(res + 2 * q) = make_uint2(Q[pass].x, Q[pass].y);
            else if (q == 2)
                res[4] = __float_as_uint(__uint_as_float(Q[pass].y) + t);
            else
                res[5] = Q[pass].x;
        }
    }
    wave_lds_sync();
}


// ------------------------------------------------------------------ ICount
// first = #{B_S <= a.end} = #{B_S < a.end + 1}; last = #{B_E < a.start};
// count = first - last (Sec. 2.1).  a.end == 2^32-1 means first = |B|.
//
// A lane without a query (past the end of its tile or round, or a query
// left out) still runs the wave-cooperative searches with the interval
// [0, kIdleEnd]: both search keys are then 0, below every key routed to a
// leaf, so the learned searches resolve it from the leaf header without a
// single probe.  (An idle [0, 0] would search B_S for 1, which a reference
// with many intervals starting at 0 turns into a fallback bisection.)
constexpr uint32_t kIdleEnd = 0xFFFFFFFFu;

// Mean length of B's intervals less one, for predictions only: the mean
// distance of equal ranks of B_E and B_S at four places.
__device__ __forceinline__ float mean_length(const SearchArgs& sa) {
    float m = 0.0f;
#pragma unroll
    for (uint32_t k = 1; k < 8; k += 2) {
        const uint32_t i = (uint32_t)((uint64_t)sa.n * k / 8);
        const uint32_t a = sa.bs[i], b = sa.be[i];
        m += b > a ? (float)(b - a) : 0.0f;
    }
    return 0.25f * m;
}

// Bisection probes kept in L2 on the plain path: the first few probes of a
// bucket are shared by every query landing in it.
constexpr uint32_t kPlainHotSteps = 3;

// The LDS top tree's bucket for each chain: the lower bound #{K_c < x[c]}
// lies in [base[c], base[c] + len[c]] (the whole array when depth is 0).
template <int NC>
__device__ __forceinline__ void tree_bucket(const SearchArgs& sa, const uint32_t* lds, const uint32_t (&x)[NC],
                                            uint32_t (&base)[NC], uint32_t (&len)[NC]) {
    const uint32_t d = sa.depth;
    if (d) {
        const uint32_t m = 1u << d;
        uint32_t k[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) k[c] = 1u;
        for (uint32_t l = 0; l < d; ++l) {
#pragma unroll
            for (int c = 0; c < NC; ++c) k[c] = 2u * k[c] + (lds[(c & 1) * m + k[c]] < x[c] ? 1u : 0u);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint64_t qb = k[c] - m;
            base[c] = (uint32_t)((qb * sa.n) >> d);
            len[c] = (uint32_t)(((qb + 1) * sa.n) >> d) - base[c];
        }
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            base[c] = 0u;
            len[c] = sa.n;
        }
    }
}

template <int QPL>
__device__ __forceinline__ void icount_plain(const SearchArgs& sa, const uint32_t* lds,
                                             const uint32_t (&as)[QPL], const uint32_t (&ae)[QPL],
                                             uint32_t (&cnt)[QPL],
                                             uint32_t (&fst)[QPL]) {
    constexpr int NC = 2 * QPL;
    uint32_t x[NC], base[NC], len[NC];
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        x[2 * q] = ae[q] + 1u;
        x[2 * q + 1] = as[q];
    }
    tree_bucket<NC>(sa, lds, x, base, len);
    bisect_multi<NC>(sa.bs, sa.be, base, len, x, kPlainHotSteps);
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        const uint32_t first = (ae[q] == 0xFFFFFFFFu) ? sa.n : base[2 * q];
        cnt[q] = first - base[2 * q + 1];
        fst[q] = first;
    }
}

// Leaf stage of both learned searches for NC chains (even chains search B_S,
// odd ones B_E): route each key and evaluate its leaf model.  Per chain:
// the leaf's rank range [rlo, rhi]; inside = (kmin < x <= kmax); pred = the
// model's rank for an inside key, else the resolved rank (rhi if x > kmax,
// rlo if x <= kmin: routing is monotone, so no key of another leaf lies
// between); err = the leaf's packed error bounds; dens = the leaf's keys per
// coordinate.  Must be called by all 64 lanes.
template <int NC>
__device__ __forceinline__ void leaf_stage(const Arrays& A, uint32_t* scr, const uint32_t (&x)[NC],
                                           uint32_t (&rlo)[NC], uint32_t (&rhi)[NC], uint32_t (&pred)[NC],
                                           uint32_t (&err)[NC], bool (&inside)[NC], float (&dens)[NC]) {
    uint32_t leaf[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const bits_rmi_model* M = A.m[c & 1];
        leaf[c] = rmi_route(M->root_a, M->root_b, x[c]);
    }
    quad_leaves<NC>(A, leaf, x, scr);
    const uint32_t lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t* res = scr + c * kLeafScr + 2 * kWave + 6 * lane;
        const uint2 ra = *reinterpret_cast<const uint2*>(res), rb = *reinterpret_cast<const uint2*>(res + 2),
                    rc = *reinterpret_cast<const uint2*>(res + 4);
        // ra = {kmin, kmax}, rb = {rlo, cnt}, rc = {y, err}
        // clamped to [0, n] so that no header value can send a search out of bounds
        rhi[c] = min(rb.x + rb.y, A.n);
        rlo[c] = min(rb.x, rhi[c]);
        err[c] = rc.y;
        dens[c] = (float)rb.y * __builtin_amdgcn_rcpf((float)(ra.y - ra.x));
        inside[c] = x[c] > ra.x && x[c] <= ra.y;
        if (inside[c])
            pred[c] = min(rlo[c] + (uint32_t)rmi_offset_from_y(__uint_as_float(rc.x), rb.y), rhi[c]);
        else
            pred[c] = x[c] > ra.y ? rhi[c] : rlo[c];
    }
}

// Learned search, leaf part: either the resolved rank (base, win = false) or
// the recorded error window [wl, wr] around the prediction (base = wl).  Must
// be called by all 64 lanes.
template <int NC>
__device__ __forceinline__ void learned_windows(const Arrays& A, uint32_t* scr, const uint32_t (&x)[NC],
                                                uint32_t (&base)[NC], uint32_t (&wl)[NC], uint32_t (&wr)[NC],
                                                uint32_t (&rlo)[NC], uint32_t (&rhi)[NC], bool (&win)[NC],
                                                float (&dens)[NC]) {
    uint32_t pred[NC], err[NC];
    leaf_stage<NC>(A, scr, x, rlo, rhi, pred, err, win, dens);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        base[c] = pred[c];
        wl[c] = wr[c] = 0;
        if (win[c]) {
            const int32_t p = (int32_t)pred[c];
            const int32_t lo = p - (int32_t)(err[c] & 0xFFFFu), hi = p + (int32_t)(err[c] >> 16);
            wl[c] = (uint32_t)max(lo, (int32_t)rlo[c]);
            wr[c] = (uint32_t)min(hi, (int32_t)rhi[c]);
            if (wr[c] < wl[c]) wr[c] = wl[c];
            base[c] = wl[c];
        }
    }
}

// Learned search through the line heads (H[j] = K[32 j], the first key of
// every 128-byte line of a sorted array, padded with 0xFFFFFFFF).  With
// r = #{K < x} the lower bound and j = #{H < x} = ceil(r / 32), the lower
// bound lies in line j - 1: r = 32 (j - 1) + #{keys < x in that line}, or
// r = 0 when j = 0.  Per chain:
//   1. leaf model -> predicted rank -> line p = pred / 32;
//   2. one cooperative probe of a window of kHeadWin heads with p at least
//      kHeadLead lines from either end (cached loads: a workgroup that serves
//      one part of the key range keeps that part's heads in its L2) gives j
//      exactly when 0 < count < kHeadWin (or the window starts at 0);
//   3. otherwise the window next to it on the side the count points to is
//      probed (only if some lane of the wave needs it), and what is still
//      unresolved is bisected over the heads of the leaf's rank range (the
//      fallback counter counts these);
//   4. one cooperative non-temporal probe of line j - 1 gives r.
// Exact whatever the model predicts (no verification step), and every read
// stays inside the arrays whatever the leaf records hold.  Must be called by
// all 64 lanes.
#ifndef BITS_HEAD_WIN
#define BITS_HEAD_WIN 16
#endif
#ifndef BITS_HEAD_ALIGN
#define BITS_HEAD_ALIGN 8
#endif
#ifndef BITS_HEAD_LEAD
#define BITS_HEAD_LEAD 4
#endif
constexpr uint32_t kHeadWin = BITS_HEAD_WIN;      // heads per window
constexpr uint32_t kHeadAlign = BITS_HEAD_ALIGN;  // window start is a multiple of this (>= 4: 16-byte loads)
constexpr uint32_t kHeadLead = BITS_HEAD_LEAD;    // the predicted line sits >= this many lines into the window
constexpr int kHeadLanes = kHeadWin == 32 ? kProbeLanes : 4;
// windows reach at most 2 kHeadWin - kHeadLead heads past the predicted line
// (second window on the right), which the >= 32 padding heads cover
static_assert(kHeadLead + kHeadAlign <= kHeadWin && 2 * kHeadWin <= 32 + kHeadLead && kHeadAlign % 4 == 0,
              "head window");

// j from a window count: resolved (0 < cnt < kHeadWin, or cnt = 0 at the
// start of the array), else left (j <= w) or right (j >= w + kHeadWin).
enum : uint32_t { kHeadHit = 0, kHeadLeft = 1, kHeadRight = 2 };
__device__ __forceinline__ uint32_t head_outcome(uint32_t w, uint32_t cnt) {
    if (cnt >= kHeadWin) return kHeadRight;
    return (cnt == 0u && w != 0u) ? kHeadLeft : kHeadHit;
}

// Learned rank: the leaf's recorded error window [wl, wr] holds the lower
// bound r = #{K < x}, so j = #{H < x} = ceil(r / 32) over the line heads
// (H[j] = K[32 j], kept in L2 / the Infinity Cache) lies in [ceil(wl / 32),
// ceil(wr / 32)].  One cooperative probe of the kHeadWin heads starting at
// or below ceil(wl / 32) - 1 resolves j when that range fits in the probe,
// else the heads of the leaf's whole range [rlo, rhi] are bisected; a probe
// whose count shows that j left the window (the model erred past its
// recorded error) falls back to that bisection too, and is counted.  One
// cooperative probe of line j - 1 then gives r (r = 0 when j = 0).  Must be
// called by all 64 lanes.
template <int NC>
__device__ __forceinline__ void rank_learned(const Arrays& A, unsigned long long* fallbacks, uint32_t* scr,
                                             const uint32_t (&x)[NC], uint32_t (&r)[NC], float (&dens)[NC]) {
    uint32_t wl[NC], wr[NC], rlo[NC], rhi[NC];
    bool win[NC];
    learned_windows<NC>(A, scr, x, r, wl, wr, rlo, rhi, win, dens);
    const uint32_t m = (A.n + 31u) >> 5;     // heads in use
    uint32_t w[NC], pc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t jlo = min((wl[c] + 31u) >> 5, m), jhi = min((wr[c] + 31u) >> 5, m);
        const uint32_t w0 = (jlo > 0u ? jlo - 1u : 0u) & ~(kHeadAlign - 1u);
        w[c] = (win[c] && jhi < w0 + kHeadWin) ? w0 : kNoLine;
    }
    probe_lines<NC, false, kHeadWin, kHeadLanes>(A.h[0], A.h[1], w, x, pc, scr);
    uint32_t j[NC], jl[NC];
    bool again = false;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        j[c] = 0u;
        jl[c] = 0u;
        if (!win[c]) continue;
        if (w[c] != kNoLine && head_outcome(w[c], pc[c]) == kHeadHit) {
            j[c] = w[c] + pc[c];
            continue;
        }
        if (w[c] != kNoLine) atomicAdd(fallbacks, 1ull);   // the window missed
        j[c] = min((rlo[c] + 31u) >> 5, m);
        jl[c] = min((rhi[c] + 31u) >> 5, m) - j[c];
        again = true;
    }
    if (__ballot(again)) bisect_multi<NC>(A.h[0], A.h[1], j, jl, x, 32u);
    uint32_t dw[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) dw[c] = (win[c] && j[c] != 0u) ? (min(j[c], m) - 1u) * 32u : kNoLine;
    probe_lines<NC, true>(A.k[0], A.k[1], dw, x, pc, scr);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (win[c]) r[c] = dw[c] == kNoLine ? 0u : dw[c] + pc[c];
}

template <int QPL>
__device__ __forceinline__ void icount_heads(const SearchArgs& sa, uint32_t* scr, const uint32_t (&as)[QPL],
                                             const uint32_t (&ae)[QPL], uint32_t (&cnt)[QPL],
                                             uint32_t (&fst)[QPL]) {
    constexpr int NC = 2 * QPL;
    uint32_t x[NC], rlo[NC], rhi[NC], pred[NC], err[NC], w[NC], pc[NC], st[NC];
    bool inside[NC];
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        x[2 * q] = ae[q] + 1u;
        x[2 * q + 1] = as[q];
    }
    float dens[NC];
    leaf_stage<NC>(both_arrays(sa), scr, x, rlo, rhi, pred, err, inside, dens);
    const uint32_t m = (sa.n + 31u) >> 5;     // heads in use
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t p = pred[c] >> 5;
        w[c] = inside[c] ? ((p > kHeadLead ? p - kHeadLead : 0u) & ~(kHeadAlign - 1u)) : kNoLine;
    }
    probe_lines<NC, false, kHeadWin, kHeadLanes>(sa.hs, sa.he, w, x, pc, scr);
    bool again = false;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        st[c] = w[c] == kNoLine ? kHeadHit : head_outcome(w[c], pc[c]);
        pc[c] = w[c] + pc[c];                 // j when resolved
        if (st[c] == kHeadLeft) w[c] = w[c] >= kHeadWin ? w[c] - kHeadWin : 0u;
        if (st[c] == kHeadRight) w[c] += kHeadWin;
        again |= st[c] != kHeadHit;
    }
    uint32_t j[NC], jl[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        j[c] = pc[c];
        jl[c] = 0;
    }
    if (__ballot(again)) {
        uint32_t w2[NC], pc2[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) w2[c] = st[c] != kHeadHit ? w[c] : kNoLine;
        probe_lines<NC, false, kHeadWin, kHeadLanes>(sa.hs, sa.he, w2, x, pc2, scr);
        uint32_t nmiss = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (st[c] == kHeadHit) continue;
            const uint32_t o = head_outcome(w2[c], pc2[c]);
            if (o == kHeadHit) {
                j[c] = w2[c] + pc2[c];
                continue;
            }
            // still unresolved: j lies in [ceil(rlo/32), ceil(rhi/32)] (rlo <= r <= rhi),
            // on the side of w2 the count points to
            const uint32_t hi = min((rhi[c] + 31u) >> 5, m), lo = min((rlo[c] + 31u) >> 5, hi);
            uint32_t a = lo, b = hi;
            if (o == kHeadLeft && w2[c] >= lo && w2[c] <= hi) b = w2[c];
            if (o == kHeadRight && w2[c] + kHeadWin >= lo && w2[c] + kHeadWin <= hi) a = w2[c] + kHeadWin;
            j[c] = a;
            jl[c] = b - a;
            ++nmiss;
        }
        if (nmiss) {
            atomicAdd(sa.fallbacks, (unsigned long long)nmiss);
            bisect_multi<NC>(sa.hs, sa.he, j, jl, x, 32u);
        }
    }
    uint32_t dw[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        dw[c] = (inside[c] && j[c] != 0u) ? (min(j[c], m) - 1u) * 32u : kNoLine;
    probe_lines<NC, true>(sa.bs, sa.be, dw, x, pc, scr);
    uint32_t r[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) r[c] = !inside[c] ? pred[c] : (dw[c] == kNoLine ? 0u : dw[c] + pc[c]);
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        const uint32_t first = (ae[q] == 0xFFFFFFFFu) ? sa.n : r[2 * q];
        cnt[q] = first - r[2 * q + 1];
        fst[q] = first;
    }
}

// Search without a model.  The LDS top tree narrows the lower bound
// r = #{K < x} to its bucket [base, base + len] and, on the way down, leaves
// the bucket's bounding keys; keys are dense enough inside a bucket that a
// straight line between them predicts r to a few keys (about sqrt(len)).
//   direct_form        a window of 32 keys around the prediction gives r; a
//                      bucket of at most 28 keys is covered whole.
//   else               j = #{H < x} = ceil(r / 32) over the line heads
//                      H[j] = K[32 j] (1/32 of the array, kept in L2 / the
//                      Infinity Cache) by windows of 32 heads around the
//                      predicted line (the median error is 2 heads at 1e7
//                      half-clustered keys and 8 at 5e7; windows of 16 miss more
//                      often: 702 us against 647 for 1e7 queries), then one window
//                      over line j - 1 (r = 0 when j = 0): one data line per search.
// A key outside the array's first and last needs no read, and a wave of them
// makes none (5e6 sorted queries of a genome against 1e6 keys of its third
// chromosome 101 us with reads for all, 65 so, 69 bisected).
// dens = the bucket's keys per coordinate.  Exact whatever the prediction
// (window_search).  All 64 lanes call it.
// Bound by random reads: one window of heads (L2) and one data line per
// search.  1e7 queries against 1e7 (half clustered): 0.55 ms, against
// 3.85 ms for the bisection of the bucket in HBM and about 0.35 ms for the
// data lines alone; 5e7 against 5e7: 3.8 against 18.5 ms.  A whole bisection
// of the heads costs one L2 request per step where the window costs two.
template <int NC, bool DIRECT>
__device__ __forceinline__ void rank_tiered(const Arrays& A, const uint32_t* tree0, const uint32_t* tree1, uint32_t d,
                                            const uint32_t (&x)[NC], uint32_t (&r)[NC], float (&dens)[NC]) {
    const uint32_t n = A.n, m = 1u << d;
    uint32_t k[NC], klo[NC], khi[NC];
    bool in[NC], any = false;   // between the first key and the last: the others need no read
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t* K = A.k[c & 1];
        k[c] = 1u;
        klo[c] = K[0];
        khi[c] = K[n - 1];
        in[c] = x[c] > klo[c] && x[c] <= khi[c];
        r[c] = x[c] > klo[c] ? n : 0u;
        any |= in[c];
    }
    for (uint32_t l = 0; l < d; ++l) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t v = ((c & 1) ? tree1 : tree0)[k[c]];
            const bool right = v < x[c];
            klo[c] = right ? v : klo[c];
            khi[c] = right ? khi[c] : v;
            k[c] = 2u * k[c] + (right ? 1u : 0u);
        }
    }
    uint32_t lo[NC], hi[NC], g[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint64_t qb = k[c] - m;
        const uint32_t base = (uint32_t)((qb * n) >> d), len = (uint32_t)(((qb + 1) * n) >> d) - base;
        const float inv = __builtin_amdgcn_rcpf((float)(khi[c] - klo[c]));
        const float f = x[c] > klo[c] ? (float)(x[c] - klo[c]) * inv : 0.0f;
        dens[c] = (float)len * inv;
        const uint32_t pos = base + (uint32_t)(fminf(f, 1.0f) * (float)len);   // equal bounding keys give f = inf
        lo[c] = DIRECT ? base : (uint32_t)(((uint64_t)base + 31u) >> 5);
        hi[c] = DIRECT ? base + len : (uint32_t)(((uint64_t)base + len + 31u) >> 5);
        g[c] = DIRECT ? pos : (uint32_t)(((uint64_t)pos + 31u) >> 5);
        if (!in[c]) lo[c] = hi[c];
    }
    if (!__ballot(any)) return;
    if constexpr (DIRECT) {
        window_search<NC, 32>(A.k[0], A.k[1], (n + 31u) & ~31u, lo, hi, g, x);
#pragma unroll
        for (int c = 0; c < NC; ++c) r[c] = in[c] ? lo[c] : r[c];
    } else {
        window_search<NC, 32>(A.h[0], A.h[1], (uint32_t)heads_len(n), lo, hi, g, x);
        uint32_t w[NC], pc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) w[c] = lo[c] ? (lo[c] - 1u) * 32u : 0u;
        oct_windows<NC, true>(A.k[0], A.k[1], w, x, pc);
#pragma unroll
        for (int c = 0; c < NC; ++c) r[c] = !in[c] ? r[c] : lo[c] ? w[c] + pc[c] : 0u;
    }
}

// ------------------------------------------------------------------ last from first
// #{B_E < a.start} is first = #{B_S <= a.end} less the count, so it is looked
// for next to rank `first` of B_E instead of by a search of its own: with the
// local density of starts, est = dens (length of a + mean length of B)
// intervals are expected, and the 128-byte line of rank first - 1 - est, or
// its neighbour on the side the count of the line points to, holds the answer
// for all but long queries (near_step; a rank on the boundary of two lines is
// decided by the two together: 3% of the queries, in 88% of the waves, took
// the full search when it was not, 1e7 queries against 5e6 through the model
// 617 us, 555 now).  Nothing is assumed about the count: a key range
// that the two lines do not decide, an interval set whose starts and ends do
// not belong together, or a query with more than kNearCount expected hits
// takes the full search.
// That halves the requests (9.5 -> 4.2 L2 requests per query at 1e7) but makes
// one chain of waits of two, so it pays where reads miss the nearest caches.
// 1e7 queries with both searches in step and so: through the model against 2e4
// keys 316 and 339 us, 5e4 371 and 297, 1e5 485 and 379, 1e6 601 and 510, 5e6
// 632 and 556, 5e7 766 and 615; without a model (line heads) against 1e6 560
// and 484, 5e6 603 and 533, 2e7 775 and 633, 5e7 1225 and 761.
// Lines after the first: 2% of the queries with 40 expected hits need the
// second, 0.02% a third.
constexpr int kNearLooks = 2;
// Lanes served eight at a time, more by a probe of the whole wave (1e7 queries
// with 110 expected hits: 8, 16, 24 lanes 429, 422, 398 us).
constexpr uint32_t kNearFew = 24;

// RANK(array, 0 = B_S or 1 = B_E, x[NC], r[NC], dens[NC]) is the full search of
// NC chains, LINE(K, w[NC], x[NC], cnt[NC]) counts lines (kNoLine: idle).
template <int QPL, class RANK, class LINE>
__device__ __forceinline__ void icount_near(const SearchArgs& sa, const uint32_t (&as)[QPL], const uint32_t (&ae)[QPL],
                                            uint32_t (&cnt)[QPL], uint32_t (&fst)[QPL], RANK rank, LINE line) {
    uint32_t x[QPL], r[QPL], w[QPL], c[QPL];
    float dens[QPL];
    bool open[QPL];
#pragma unroll
    for (int q = 0; q < QPL; ++q) x[q] = ae[q] + 1u;
    rank(one_array(sa, 0), 0, x, r, dens);
    bool any = false;
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        fst[q] = (ae[q] == 0xFFFFFFFFu) ? sa.n : r[q];
        x[q] = as[q];
        bool done;
        w[q] = near_line(sa.n, fst[q], dens[q], sa.mean_len, as[q], ae[q], done);
        r[q] = done ? 0u : kNoLine;
        open[q] = !done;
        // one lane's full search is the whole wave's work: no line is then looked at for the others
        if (__ballot(open[q] && w[q] == kNoLine)) w[q] = kNoLine;
        any |= w[q] != kNoLine;
    }
    if (__ballot(any)) {
        line(sa.be, w, x, c);
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            if (w[q] != kNoLine && near_step(sa.n, c[q], w[q], r[q])) {
                open[q] = false;
                w[q] = kNoLine;
            }
        }
    }
    // the neighbouring line for lanes that the first did not decide: as many looks for
    // each of them, whatever the other lanes need
#pragma unroll 1
    for (int look = 0; look < kNearLooks; ++look) {
        uint32_t most = 0;
#pragma unroll
        for (int q = 0; q < QPL; ++q) most = max(most, (uint32_t)__popcll(__ballot(w[q] != kNoLine)));
        if (!most) break;
        if (most > kNearFew) {
            line(sa.be, w, x, c);
#pragma unroll
            for (int q = 0; q < QPL; ++q) {
                if (w[q] != kNoLine && near_step(sa.n, c[q], w[q], r[q])) {
                    open[q] = false;
                    w[q] = kNoLine;
                }
            }
            continue;
        }
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            uint64_t left = __ballot(w[q] != kNoLine);
#pragma unroll 1
            while (left) {
                uint64_t on = left;
                const uint32_t k = few_windows<true>(sa.be, w[q], x[q], on);
                left &= ~on;
                if (((on >> (threadIdx.x & (kWave - 1))) & 1u) && near_step(sa.n, k, w[q], r[q])) {
                    open[q] = false;
                    w[q] = kNoLine;
                }
            }
        }
    }
    any = false;
#pragma unroll
    for (int q = 0; q < QPL; ++q) any |= open[q];
    if (__ballot(any)) {
        uint32_t r2[QPL];
#pragma unroll
        for (int q = 0; q < QPL; ++q) x[q] = open[q] ? as[q] : 0u;   // 0 is below every key of a leaf
        rank(one_array(sa, 1), 1, x, r2, dens);
#pragma unroll
        for (int q = 0; q < QPL; ++q)
            if (open[q]) r[q] = r2[q];
    }
#pragma unroll
    for (int q = 0; q < QPL; ++q) cnt[q] = fst[q] - r[q];
}

// The count through the model: the recorded error windows searched.
template <int QPL>
__device__ __forceinline__ void icount_learned(const SearchArgs& sa, uint32_t* scr, const uint32_t (&as)[QPL],
                                               const uint32_t (&ae)[QPL], uint32_t (&cnt)[QPL], uint32_t (&fst)[QPL]) {
    icount_near<QPL>(
        sa, as, ae, cnt, fst,
        [&](const Arrays& A, int, const uint32_t (&x)[QPL], uint32_t (&r)[QPL], float (&dens)[QPL]) {
            rank_learned<QPL>(A, sa.fallbacks, scr, x, r, dens);
        },
        [&](const uint32_t* K, const uint32_t (&w)[QPL], const uint32_t (&x)[QPL], uint32_t (&c)[QPL]) {
            probe_lines<QPL, true>(K, K, w, x, c, scr);
        });
}

// The same with both searches of a query in step, for references up to
// kPairedKeys keys: their lines are in L2, where a second wait costs more than
// the requests it saves (measured at icount_near).
template <int QPL>
__device__ __forceinline__ void icount_paired(const SearchArgs& sa, uint32_t* scr, const uint32_t (&as)[QPL],
                                              const uint32_t (&ae)[QPL], uint32_t (&cnt)[QPL], uint32_t (&fst)[QPL]) {
    uint32_t x[2 * QPL], r[2 * QPL];
    float dens[2 * QPL];
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        x[2 * q] = ae[q] + 1u;
        x[2 * q + 1] = as[q];
    }
    rank_learned<2 * QPL>(both_arrays(sa), sa.fallbacks, scr, x, r, dens);
#pragma unroll
    for (int q = 0; q < QPL; ++q) {
        fst[q] = (ae[q] == 0xFFFFFFFFu) ? sa.n : r[2 * q];
        cnt[q] = fst[q] - r[2 * q + 1];
    }
}

// One query at a time: the windows of more would not fit the registers.  In
// windows of keys both searches of a query run in step, which hides their waits
// in each other's; through the line heads the second starts from the first one's rank.
template <int QPL, bool DIRECT>
__device__ __forceinline__ void icount_tiered(const SearchArgs& sa, const uint32_t* lds, const uint32_t (&as)[QPL],
                                              const uint32_t (&ae)[QPL], uint32_t (&cnt)[QPL],
                                              uint32_t (&fst)[QPL]) {
    const uint32_t* tree_e = lds + (1u << sa.depth);
#pragma unroll 1
    for (int q = 0; q < QPL; ++q) {
        if constexpr (DIRECT) {
            const uint32_t x[2] = {ae[q] + 1u, as[q]};
            uint32_t r[2];
            float dens[2];
            rank_tiered<2, true>(both_arrays(sa), lds, tree_e, sa.depth, x, r, dens);
            const uint32_t first = (ae[q] == 0xFFFFFFFFu) ? sa.n : r[0];
            cnt[q] = first - r[1];
            fst[q] = first;
        } else {
            const uint32_t s1[1] = {as[q]}, e1[1] = {ae[q]};
            uint32_t c1[1], f1[1];
            icount_near<1>(
                sa, s1, e1, c1, f1,
                [&](const Arrays& A, int which, const uint32_t (&x)[1], uint32_t (&r)[1], float (&dens)[1]) {
                    const uint32_t* tree = which ? tree_e : lds;
                    rank_tiered<1, false>(A, tree, tree, sa.depth, x, r, dens);
                },
                [&](const uint32_t* K, const uint32_t (&w)[1], const uint32_t (&x)[1], uint32_t (&c)[1]) {
                    const uint32_t at[1] = {w[0] == kNoLine ? 0u : w[0]};
                    oct_windows<1, true>(K, K, at, x, c);
                });
            cnt[q] = c1[0];
            fst[q] = f1[0];
        }
    }
}

template <int QPL, int MODE>
__device__ __forceinline__ void icount(const SearchArgs& sa, uint32_t* lds, const uint32_t (&as)[QPL],
                                       const uint32_t (&ae)[QPL], uint32_t (&cnt)[QPL], uint32_t (&fst)[QPL]) {
    if constexpr (MODE == kModeLearned)
        icount_learned<QPL>(sa, lds + (threadIdx.x / kWave) * probe_scratch_words(QPL), as, ae, cnt, fst);
    else if constexpr (MODE == kModePaired)
        icount_paired<QPL>(sa, lds + (threadIdx.x / kWave) * probe_scratch_words(QPL), as, ae, cnt, fst);
    else if constexpr (MODE == kModePlain)
        icount_plain<QPL>(sa, lds, as, ae, cnt, fst);
    else
        icount_tiered<QPL, MODE == kModeDirect>(sa, lds, as, ae, cnt, fst);
}


// Adds the workgroup's sum of v to *out with one atomic: all workgroups add to
// one word, and thousands of such additions take longer than a small count
// (1e6 queries against 3e5 with 8192 waves: 129 us with an atomic per wave,
// 52 us with one per workgroup).  All threads call it.
__device__ __forceinline__ void add_block_sum(uint64_t v, unsigned long long* out) {
    __shared__ unsigned long long part[1024 / kWave];
    v = wave_sum_u64(v);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t k = 1; k < blockDim.x / kWave; ++k) v += part[k];
        if (v) atomicAdd(out, (unsigned long long)v);
    }
}

// ------------------------------------------------------------------ counting kernel
// Persistent grid over tiles of blockDim*QPL queries; query i of a tile is
// loaded by lane (i mod blockDim), so every load of a query round is
// coalesced.  Totals: uint64 sums, one atomic per workgroup.

// MODE: kModePlain (LDS tree + bisection), kModeLearned and kModePaired (learned
// index, error-window head probe + one line), kModeTiered (LDS tree + line-head
// window + one line) or kModeDirect (LDS tree + one window of keys).
template <int QPL, int MODE>
BITS_SEARCH_KERNEL k_count(SearchArgs sa, const uint32_t* __restrict__ a_start,
                                                const uint32_t* __restrict__ a_end, uint64_t na,
                                                uint32_t* __restrict__ counts, uint32_t* __restrict__ firsts,
                                                unsigned long long* total) {
    extern __shared__ __align__(16) uint32_t lds[];
    if (!learned_mode(MODE)) {
        stage_tree(lds, sa.tree, sa.tree_stride, sa.depth);
        __syncthreads();
    }
    if (MODE == kModeLearned || MODE == kModeTiered) sa.mean_len = mean_length(sa);
    const uint64_t tile = (uint64_t)blockDim.x * QPL;
    const uint64_t ntiles = (na + tile - 1) / tile;
    uint64_t acc = 0;
    uint32_t bad = 0;
    for (uint64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        uint32_t as[QPL], ae[QPL], cnt[QPL];
        bool valid[QPL];
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            const uint64_t i = t * tile + (uint64_t)q * blockDim.x + threadIdx.x;
            valid[q] = i < na;
            as[q] = valid[q] ? a_start[i] : 0u;
            ae[q] = valid[q] ? a_end[i] : kIdleEnd;
            if (as[q] > ae[q]) {
                bad = 1;
                valid[q] = false;
                ae[q] = as[q];
            }
        }
        uint32_t fst[QPL];
        icount<QPL, MODE>(sa, lds, as, ae, cnt, fst);
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            const uint64_t i = t * tile + (uint64_t)q * blockDim.x + threadIdx.x;
            const uint32_t c = valid[q] ? cnt[q] : 0u;
            if (counts && i < na) counts[i] = c;
            if (firsts && i < na) firsts[i] = fst[q];
            acc += c;
        }
    }
    if (bad) atomicOr(sa.status, BITS_FLAG_INTERVAL);
    if (total) add_block_sum(acc, total);
}

// ------------------------------------------------------------------ decision
// Sec. 1.1, sub-problem 1: does any a intersect any b?  The counting loop
// with an early exit: a workgroup checks the shared flag before each tile
// and stops once some query has a non-zero count.  *witness receives the
// smallest index with a hit among the tiles that ran (initialised to
// 2^64 - 1 by the caller).
template <int QPL, int MODE>
BITS_SEARCH_KERNEL k_decide(SearchArgs sa, const uint32_t* __restrict__ a_start, const uint32_t* __restrict__ a_end,
                            uint64_t na, uint32_t* found, unsigned long long* witness) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ uint32_t stop;
    if (!learned_mode(MODE)) stage_tree(lds, sa.tree, sa.tree_stride, sa.depth);
    __syncthreads();
    if (MODE == kModeLearned || MODE == kModeTiered) sa.mean_len = mean_length(sa);
    const uint64_t tile = (uint64_t)blockDim.x * QPL;
    const uint64_t ntiles = (na + tile - 1) / tile;
    uint32_t bad = 0;
    for (uint64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        if (threadIdx.x == 0) stop = __hip_atomic_load(found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (stop) break;
        uint32_t as[QPL], ae[QPL], cnt[QPL], fst[QPL];
        bool valid[QPL];
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            const uint64_t i = t * tile + (uint64_t)q * blockDim.x + threadIdx.x;
            valid[q] = i < na;
            as[q] = valid[q] ? a_start[i] : 0u;
            ae[q] = valid[q] ? a_end[i] : kIdleEnd;
            if (as[q] > ae[q]) {
                bad = 1;
                valid[q] = false;
                ae[q] = as[q];
            }
        }
        icount<QPL, MODE>(sa, lds, as, ae, cnt, fst);
        bool hit = false;
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            if (valid[q] && cnt[q]) {
                atomicMin(witness, (unsigned long long)(t * tile + (uint64_t)q * blockDim.x + threadIdx.x));
                hit = true;
            }
        }
        if (hit) atomicOr(found, 1u);
        __syncthreads();   // every lane has read `stop` before it is rewritten
    }
    if (bad) atomicOr(sa.status, BITS_FLAG_INTERVAL);
}

// ------------------------------------------------------------------ Monte-Carlo
// The per-query table (off, span, len, idx) is grouped by chromosome (see
// k_mc_prepare): position j holds query idx[j].  Work item = (tile of
// blockDim*QPL table positions, chunk of consecutive shuffles), walked by a
// persistent grid.  A workgroup reads its tile's table entries once per item
// and runs every shuffle of the chunk on them.  Query i of shuffle s starts at
// off_i + floor(u * span_i / 2^64), u = the first two Philox words of counter
// g = (s0 + s) * na + i.  Per-shuffle wave sums are added in LDS and flushed
// with one global atomic per shuffle per item.  OBSERVED counts the
// unshuffled queries instead (same exclusion of queries with span 0, i.e.
// outside their chromosome).
//
// XCD-aware split: workgroups are dispatched round-robin over the 8 XCDs,
// so workgroup b runs on XCD b mod 8.  The tiles are cut into 8 contiguous
// groups and group x is served only by workgroups b = x (mod 8).  A shuffle
// keeps every query inside its chromosome, and the table is grouped by
// chromosome, so each XCD searches one contiguous part of B and its L2 holds
// that part's leaves and line heads.  (With another placement the split only
// costs locality, never correctness.)
constexpr uint32_t kMaxChunk = 64;
constexpr uint32_t kXcds = 8;

template <int QPL, int MODE>
__device__ __forceinline__ void icount_mc(const SearchArgs& sa, uint32_t* lds, const uint32_t (&as)[QPL],
                                          const uint32_t (&ae)[QPL], uint32_t (&cnt)[QPL]) {
    uint32_t fst[QPL];
    if constexpr (MODE == kModeLearned)
        icount_heads<QPL>(sa, lds + (threadIdx.x / kWave) * probe_scratch_words(QPL), as, ae, cnt, fst);
    else
        icount<QPL, MODE>(sa, lds, as, ae, cnt, fst);
}

template <int QPL, int MODE, bool OBSERVED>
BITS_SEARCH_KERNEL k_mc(SearchArgs sa, const uint32_t* __restrict__ a_start, const uint32_t* __restrict__ a_end,
         const uint32_t* __restrict__ off, const uint32_t* __restrict__ span, const uint32_t* __restrict__ len,
         const uint32_t* __restrict__ idx, uint64_t na, uint64_t seed, uint64_t s0, uint64_t nshuf, uint64_t tiles,
         uint32_t chunk, unsigned long long* __restrict__ totals) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ unsigned long long acc[kMaxChunk];
    if (MODE != kModeLearned) stage_tree(lds, sa.tree, sa.tree_stride, sa.depth);
    for (uint32_t k = threadIdx.x; k < kMaxChunk; k += blockDim.x) acc[k] = 0ull;
    __syncthreads();
    if (MODE == kModeTiered) sa.mean_len = mean_length(sa);
    const uint64_t tile = (uint64_t)blockDim.x * QPL;
    const uint64_t nchunks = (nshuf + chunk - 1) / chunk;
    const uint32_t ng = (gridDim.x >= kXcds && tiles >= kXcds) ? kXcds : 1u;
    const uint32_t grp = blockIdx.x % ng, slot = blockIdx.x / ng;
    const uint32_t nslots = (gridDim.x - grp + ng - 1) / ng;   // workgroups b < gridDim with b = grp (mod ng)
    const uint64_t t_lo = tiles * grp / ng, gtiles = tiles * (grp + 1) / ng - t_lo;
    const uint64_t nitems = gtiles * nchunks;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    for (uint64_t it = slot; it < nitems; it += nslots) {
        const uint64_t kc = it / gtiles;
        const uint64_t t = t_lo + (it - kc * gtiles);
        uint32_t qo[QPL], qs[QPL], ql[QPL];
        uint64_t qi[QPL];
        bool valid[QPL];
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            const uint64_t pos = t * tile + (uint64_t)q * blockDim.x + threadIdx.x;
            const bool in = pos < na;
            qs[q] = in ? span[pos] : 0u;
            qi[q] = in ? idx[pos] : 0u;
            valid[q] = qs[q] != 0u;
            if (OBSERVED) {
                qo[q] = valid[q] ? a_start[qi[q]] : 0u;
                ql[q] = valid[q] ? a_end[qi[q]] : kIdleEnd;
            } else {
                qo[q] = valid[q] ? off[pos] : 0u;
                ql[q] = valid[q] ? len[pos] : 1u;
            }
        }
        const uint64_t sb = kc * chunk;
        const uint64_t se = min(nshuf, sb + chunk);
        for (uint64_t s = sb; s < se; ++s) {
            uint32_t as[QPL], ae[QPL], cnt[QPL];
#pragma unroll
            for (int q = 0; q < QPL; ++q) {
                if (OBSERVED) {
                    as[q] = qo[q];
                    ae[q] = ql[q];
                } else {
                    const uint64_t g = (s0 + s) * na + qi[q];
                    uint32_t c0 = (uint32_t)g, c1 = (uint32_t)(g >> 32), c2 = 0u, c3 = 0u;
                    philox4x32_10(c0, c1, c2, c3, k0, k1);
                    const uint64_t u = ((uint64_t)c1 << 32) | c0;
                    const uint32_t local = (uint32_t)__umul64hi(u, (uint64_t)qs[q]);
                    as[q] = valid[q] ? qo[q] + local : 0u;
                    ae[q] = valid[q] ? as[q] + ql[q] - 1u : kIdleEnd;
                }
            }
            icount_mc<QPL, MODE>(sa, lds, as, ae, cnt);
            uint64_t sum = 0;
#pragma unroll
            for (int q = 0; q < QPL; ++q) sum += valid[q] ? cnt[q] : 0u;
            sum = wave_sum_u64(sum);
            if ((threadIdx.x & (kWave - 1)) == 0 && sum) atomicAdd(&acc[s - sb], (unsigned long long)sum);
        }
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < (uint32_t)(se - sb); k += blockDim.x) {
            const unsigned long long v = acc[k];
            if (v) atomicAdd(totals + sb + k, v);
            acc[k] = 0ull;
        }
        __syncthreads();
    }
}

// Learned Monte-Carlo with placements sorted inside the work item.  An item
// (tile of blockDim/8 table positions, chunk of <= kMaxChunk shuffles)
// generates all its placements, counting-sorts them by start into
// kSortBuckets buckets over the tile's start range in LDS, and searches them
// in that order, so that lanes of a wave share leaf records and often head
// windows: the searches then take fewer L1/L2 requests, the resource that
// bounds the unsorted kernel.  Placements are made twice (histogram, then
// scatter) rather than staged unsorted, to fit LDS.  Totals are sums, so
// the order does not change them.  The placements (start, and query | shuffle
// << 8 in 16 bits) live in dynamic LDS after the per-wave probe scratch.
#ifndef BITS_MC_SORTED
#define BITS_MC_SORTED 1
#endif
#ifndef BITS_MC_SORTED_QPL
#define BITS_MC_SORTED_QPL 1
#endif
constexpr int kSortQpl = BITS_MC_SORTED_QPL;   // placements per lane per search round
constexpr uint32_t kSortBuckets = 1024;
constexpr uint32_t kSortMaxTileQ = 128;
constexpr uint32_t kSortQBits = 8;
__host__ __device__ constexpr uint32_t sort_tile_q(uint32_t block) { return block / 8u; }
__host__ __device__ constexpr size_t sort_lds_bytes(uint32_t block) {
    return (size_t)(block / kWave) * probe_scratch_words(kSortQpl) * 4u + (size_t)sort_tile_q(block) * kMaxChunk * 6u;
}
static_assert((kMaxChunk << kSortQBits) <= 65536, "sort meta");

// In-place exclusive scan of kSortBuckets counters by the whole workgroup;
// returns the total.
__device__ __forceinline__ uint32_t block_scan_buckets(uint32_t* h, uint32_t* wsum) {
    const uint32_t per = kSortBuckets / blockDim.x;            // 1, 2 or 4 (blocks of 1024, 512, 256)
    const uint32_t b0 = threadIdx.x * per;
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        if (k < per) v[k] = h[b0 + k];
        mine += v[k];
    }
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
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        if (k < per) h[b0 + k] = pre;
        pre += v[k];
    }
    __syncthreads();
    return tot;
}

BITS_SEARCH_KERNEL k_mc_sorted(SearchArgs sa, const uint32_t* __restrict__ off, const uint32_t* __restrict__ span,
                               const uint32_t* __restrict__ len, const uint32_t* __restrict__ idx, uint64_t na,
                               uint64_t seed, uint64_t s0, uint64_t nshuf, uint64_t tiles, uint32_t chunk,
                               unsigned long long* __restrict__ totals) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ uint32_t hist[kSortBuckets];
    __shared__ uint32_t t_off[kSortMaxTileQ], t_span[kSortMaxTileQ], t_len[kSortMaxTileQ], t_idx[kSortMaxTileQ];
    __shared__ unsigned long long acc[kMaxChunk];
    __shared__ uint32_t wsum[16], lo_key, hi_key;
    const uint32_t tile_q = sort_tile_q(blockDim.x);           // 32, 64 or 128
    uint32_t* scr = lds + (threadIdx.x / kWave) * probe_scratch_words(kSortQpl);
    uint32_t* p_start = lds + (blockDim.x / kWave) * probe_scratch_words(kSortQpl);
    uint16_t* p_meta = reinterpret_cast<uint16_t*>(p_start + tile_q * kMaxChunk);
    for (uint32_t k = threadIdx.x; k < kMaxChunk; k += blockDim.x) acc[k] = 0ull;
    const uint64_t nchunks = (nshuf + chunk - 1) / chunk;
    const uint32_t ng = (gridDim.x >= kXcds && tiles >= kXcds) ? kXcds : 1u;
    const uint32_t grp = blockIdx.x % ng, slot = blockIdx.x / ng;
    const uint32_t nslots = (gridDim.x - grp + ng - 1) / ng;
    const uint64_t t_lo = tiles * grp / ng, gtiles = tiles * (grp + 1) / ng - t_lo;
    const uint64_t nitems = gtiles * nchunks;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    __syncthreads();
    for (uint64_t it = slot; it < nitems; it += nslots) {
        const uint64_t kc = it / gtiles;
        const uint64_t t = t_lo + (it - kc * gtiles);
        const uint64_t sb = kc * chunk;
        const uint32_t nsh = (uint32_t)min((uint64_t)chunk, nshuf - sb);
        // 1. the tile's table and its start range
        if (threadIdx.x == 0) {
            lo_key = 0xFFFFFFFFu;
            hi_key = 0u;
        }
        for (uint32_t k = threadIdx.x; k < kSortBuckets; k += blockDim.x) hist[k] = 0u;
        __syncthreads();
        if (threadIdx.x < tile_q) {
            const uint64_t pos = t * tile_q + threadIdx.x;
            const bool in = pos < na;
            const uint32_t sp = in ? span[pos] : 0u;
            t_span[threadIdx.x] = sp;
            t_off[threadIdx.x] = in ? off[pos] : 0u;
            t_len[threadIdx.x] = in ? len[pos] : 1u;
            t_idx[threadIdx.x] = in ? idx[pos] : 0u;
            if (sp) {
                atomicMin(&lo_key, t_off[threadIdx.x]);
                atomicMax(&hi_key, t_off[threadIdx.x] + (sp - 1u));
            }
        }
        __syncthreads();
        const uint32_t lo = lo_key;
        const uint32_t range = hi_key >= lo ? hi_key - lo : 0u;
        const uint32_t bits = range ? 32u - __clz(range) : 0u;
        const uint32_t shift = bits > 10u ? bits - 10u : 0u;   // (range >> shift) < 1024
        const uint32_t P = tile_q * nsh;
        // 2. histogram of the placements' buckets
        for (uint32_t p = threadIdx.x; p < P; p += blockDim.x) {
            const uint32_t q = p & (tile_q - 1), sh = p / tile_q;
            if (!t_span[q]) continue;
            const uint32_t st = mc_place((s0 + sb + sh) * na + t_idx[q], k0, k1, t_off[q], t_span[q]);
            atomicAdd(&hist[(st - lo) >> shift], 1u);
        }
        __syncthreads();
        const uint32_t nvalid = block_scan_buckets(hist, wsum);
        // 3. the same placements again, scattered into bucket order
        for (uint32_t p = threadIdx.x; p < P; p += blockDim.x) {
            const uint32_t q = p & (tile_q - 1), sh = p / tile_q;
            if (!t_span[q]) continue;
            const uint32_t st = mc_place((s0 + sb + sh) * na + t_idx[q], k0, k1, t_off[q], t_span[q]);
            const uint32_t at = atomicAdd(&hist[(st - lo) >> shift], 1u);
            p_start[at] = st;
            p_meta[at] = (uint16_t)(q | (sh << kSortQBits));
        }
        __syncthreads();
        // 4. the searches, in start order (every lane runs every round: the probes are wave-cooperative)
        for (uint32_t r0 = 0; r0 < nvalid; r0 += kSortQpl * blockDim.x) {
            uint32_t as[kSortQpl], ae[kSortQpl], cnt[kSortQpl], fst[kSortQpl], m[kSortQpl];
            bool valid[kSortQpl];
#pragma unroll
            for (uint32_t q = 0; q < kSortQpl; ++q) {
                const uint32_t p = r0 + q * blockDim.x + threadIdx.x;
                valid[q] = p < nvalid;
                as[q] = valid[q] ? p_start[p] : 0u;
                m[q] = valid[q] ? p_meta[p] : 0u;
                ae[q] = valid[q] ? as[q] + t_len[m[q] & (tile_q - 1)] - 1u : kIdleEnd;
            }
            icount_heads<kSortQpl>(sa, scr, as, ae, cnt, fst);
#pragma unroll
            for (uint32_t q = 0; q < kSortQpl; ++q)
                if (valid[q] && cnt[q]) atomicAdd(&acc[m[q] >> kSortQBits], (unsigned long long)cnt[q]);
        }
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < nsh; k += blockDim.x) {
            const unsigned long long v = acc[k];
            if (v) atomicAdd(totals + sb + k, v);
            acc[k] = 0ull;
        }
        __syncthreads();
    }
}

struct ChromTab {
    uint32_t n;
    uint32_t off[BITS_MAX_CHROM + 1];   // off[c] = sum of lengths before c; off[n] = genome size
};

// Chromosome of a global coordinate: the last c with off[c] <= s.
__device__ __forceinline__ uint32_t chrom_of(const ChromTab& ct, uint32_t s) {
    uint32_t lo = 0, hi = ct.n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ct.off[mid] <= s) lo = mid; else hi = mid;
    }
    return lo;
}

// What a Monte-Carlo call starts from, in one launch: zero totals, observed
// total, chromosome histogram and cursors.
__global__ void __launch_bounds__(256) k_mc_zero(unsigned long long* __restrict__ totals, uint64_t ns,
                                                 unsigned long long* observed, uint32_t* hist, uint32_t* cursor) {
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < ns; k += (uint64_t)gridDim.x * blockDim.x)
        totals[k] = 0ull;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) *observed = 0ull;
        if (hist) {
            hist[threadIdx.x] = 0u;
            cursor[threadIdx.x] = 0u;
        }
    }
}
static_assert(BITS_MAX_CHROM == 256, "one thread per chromosome");

// Per-chromosome query counts (hist and cursor zeroed by the caller).  The
// last workgroup to add its counts (counted in cursor[0], which is 0 in the
// result) turns them into cursor[c] = queries on chromosomes before c.  Each
// workgroup waits for its additions' return values before it counts itself in,
// so no cache write-back (a device fence: 30 us for 1e5 queries) is needed; few
// large workgroups keep the shared counter cheap.
__global__ void __launch_bounds__(1024) k_mc_hist(const uint32_t* __restrict__ a_start, uint64_t na, ChromTab ct,
                                                  uint32_t* hist, uint32_t* cursor) {
    __shared__ uint32_t h[BITS_MAX_CHROM], wsum[4], last;
    if (threadIdx.x < BITS_MAX_CHROM) h[threadIdx.x] = 0u;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < na; i += (uint64_t)gridDim.x * blockDim.x)
        atomicAdd(&h[chrom_of(ct, a_start[i])], 1u);
    __syncthreads();
    if (threadIdx.x < BITS_MAX_CHROM && h[threadIdx.x]) {
        const uint32_t old = atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
        asm volatile("" ::"v"(old) : "memory");   // the addition has been made
    }
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&cursor[0], 1u) == gridDim.x - 1u ? 1u : 0u;
    __syncthreads();
    if (!last || threadIdx.x >= BITS_MAX_CHROM) return;
    const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t v = __hip_atomic_load(&hist[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= (uint32_t)o) x += y;
    }
    if (lane == kWave - 1) wsum[w] = x;
    __syncthreads();   // of the waves that are left
    for (uint32_t k = 0; k < w; ++k) x += wsum[k];
    cursor[threadIdx.x] = x - v;
}

// Per-query (chromosome offset, number of legal starts, length, index),
// computed once and reused by every shuffle, stored grouped by chromosome:
// each round of blockDim queries takes one slot range per chromosome from
// `cursor` and places its queries there.  The order inside a chromosome's
// range depends on scheduling; the totals do not (sums over the queries,
// each drawing from its own index).  span = 0 marks a query outside its
// chromosome (or start > end).  With packed != nullptr (the binned path) the
// table is span, idx and packed = {index, length, or 0 for such a query}; off
// and len are not written.
__global__ void __launch_bounds__(1024) k_mc_prepare(const uint32_t* __restrict__ a_start,
                                                     const uint32_t* __restrict__ a_end, uint64_t na, ChromTab ct,
                                                     uint32_t* __restrict__ cursor, uint32_t* __restrict__ off,
                                                     uint32_t* __restrict__ span, uint32_t* __restrict__ len,
                                                     uint32_t* __restrict__ idx, uint2* __restrict__ packed,
                                                     uint32_t* status) {
    __shared__ uint32_t cnt[BITS_MAX_CHROM], base[BITS_MAX_CHROM];
    uint32_t bad = 0;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x; i0 < na; i0 += (uint64_t)gridDim.x * blockDim.x) {
        for (uint32_t k = threadIdx.x; k < ct.n; k += blockDim.x) cnt[k] = 0u;
        __syncthreads();
        const uint64_t i = i0 + threadIdx.x;
        uint32_t s = 0, e = 0, c = 0, r = 0;
        if (i < na) {
            s = a_start[i];
            e = a_end[i];
            c = chrom_of(ct, s);
            r = atomicAdd(&cnt[c], 1u);
        }
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < ct.n; k += blockDim.x)
            if (cnt[k]) base[k] = atomicAdd(&cursor[k], cnt[k]);
        __syncthreads();
        if (i < na) {
            const bool ok = s <= e && s >= ct.off[c] && (uint64_t)e < (uint64_t)ct.off[c + 1];
            const uint32_t L = e - s + 1u;
            const uint32_t pos = base[c] + r;
            if (packed) {
                packed[pos] = make_uint2((uint32_t)i, ok ? L : 0u);
            } else {
                off[pos] = ct.off[c];
                len[pos] = ok ? L : 1u;
            }
            span[pos] = ok ? (ct.off[c + 1] - ct.off[c]) - L + 1u : 0u;
            idx[pos] = (uint32_t)i;
            if (!ok) bad |= (s > e) ? BITS_FLAG_INTERVAL : BITS_FLAG_CHROM;
        }
        __syncthreads();
    }
    if (bad) atomicOr(status, bad);
}

// ------------------------------------------------------------------ paper orientation
// The Monte-Carlo loop as Sec. 3.2 runs it: every round randomises the
// database set B and sorts it again, then counts the fixed query set A.
// Round r of a batch places interval idx[p] of B (table position p) by the
// rule and stream of k_mc with the roles swapped, g = (s0 + r) * nb + idx[p],
// and writes keys S[r * stride + p], E[r * stride + p] as one segment per round for
// the segmented sort.  An interval outside its chromosome (span 0) becomes
// the sentinel [2^32 - 1, 2^32 - 1], which no query with end < 2^32 - 1
// counts.  identity = true writes the unshuffled set (the observed round).
__global__ void k_place_rounds(const uint32_t* __restrict__ off, const uint32_t* __restrict__ span,
                               const uint32_t* __restrict__ len, const uint32_t* __restrict__ idx,
                               const uint32_t* __restrict__ b_start, uint64_t nb, uint64_t stride, uint64_t seed,
                               uint64_t s0, uint32_t rounds, uint32_t identity, uint32_t* __restrict__ S,
                               uint32_t* __restrict__ E) {
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint64_t total = (uint64_t)rounds * nb;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t r = t / nb, p = t - r * nb;
        const uint32_t sp = span[p];
        uint32_t st = 0xFFFFFFFFu, en = 0xFFFFFFFFu;
        if (sp) {
            if (identity) {
                st = b_start[idx[p]];
            } else {
                const uint64_t g = (s0 + r) * nb + idx[p];
                uint32_t c0 = (uint32_t)g, c1 = (uint32_t)(g >> 32), c2 = 0u, c3 = 0u;
                philox4x32_10(c0, c1, c2, c3, k0, k1);
                const uint64_t u = ((uint64_t)c1 << 32) | c0;
                st = off[p] + (uint32_t)__umul64hi(u, (uint64_t)sp);
            }
            en = st + len[p] - 1u;
        }
        S[r * stride + p] = st;
        E[r * stride + p] = en;
    }
}

// 0xFFFFFFFF from nb to stride of every round.
__global__ void k_fill_tails(uint32_t* __restrict__ S, uint32_t* __restrict__ E, uint64_t nb, uint64_t stride,
                             uint32_t rounds) {
    const uint32_t tail = (uint32_t)(stride - nb);
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < rounds * tail; t += gridDim.x * blockDim.x) {
        const uint64_t at = (uint64_t)(t / tail) * stride + nb + t % tail;
        S[at] = 0xFFFFFFFFu;
        E[at] = 0xFFFFFFFFu;
    }
}

// What the search without a model needs of every sorted round (segments
// S[r * stride ..], E[r * stride ..] of nb keys): the top trees of both arrays
// at trees + r * stride, and above kDirectKeys their line heads at
// heads + r * stride.  blockIdx.y = round.
__global__ void __launch_bounds__(256) k_round_index(const uint32_t* __restrict__ S, const uint32_t* __restrict__ E,
                                                     uint32_t nb, uint64_t stride, uint32_t depth,
                                                     uint32_t* __restrict__ trees, uint32_t* __restrict__ heads) {
    const uint64_t o = blockIdx.y * stride;
    const uint32_t m = 1u << depth, hl = nb > kDirectKeys ? (uint32_t)heads_len(nb) : 0u, lines = (nb + 31u) / 32u;
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < 2u * (m + hl); t += gridDim.x * blockDim.x) {
        if (t < 2u * m) {
            const uint32_t k = t & (m - 1u);
            const uint32_t* K = (t < m ? S : E) + o;
            trees[o + t] = k ? K[tree_rank(k, nb) - 1u] : 0u;
        } else {
            const uint32_t a = t - 2u * m >= hl ? 1u : 0u, k = t - 2u * m - a * hl;
            heads[o + t - 2u * m] = k < lines ? (a ? E : S)[o + 32u * (uint64_t)k] : 0xFFFFFFFFu;
        }
    }
}

// Counts the fixed query set A against every sorted round of a batch: `per`
// workgroups a round, each staging the round's top trees once for its share
// of A.  Random reads of the round's sorted arrays bound it, so a round
// belongs to one XCD (workgroups b = r mod 8) and few rounds are in flight on
// it, to be served from its L2: 64 rounds of 1e5 intervals against 1e5
// queries take 128 us with 16 workgroups a round (8: 159, 32: 161, 64: 229,
// from staging), 367 us with rounds spread over all XCDs, and 710 us for a
// bisection of the whole segment per search.  Fewer than 8 rounds are spread
// over the whole chip.
constexpr uint32_t kRoundParts = 16;   // most workgroups of a round
template <int MODE>
BITS_SEARCH_KERNEL k_count_rounds(SearchArgs sa0, uint64_t stride, uint32_t rounds, uint32_t per,
                                  const uint32_t* __restrict__ a_start, const uint32_t* __restrict__ a_end, uint64_t na,
                                  unsigned long long* __restrict__ totals) {
    extern __shared__ __align__(16) uint32_t lds[];
    const uint32_t xg = rounds >= kXcds ? kXcds : 1u;
    const uint32_t slot = blockIdx.x / xg, turn = slot / per, part = slot - turn * per;
    const uint32_t r = turn * xg + blockIdx.x % xg;
    if (r >= rounds) return;
    SearchArgs sa = sa0;
    sa.bs += r * stride;
    sa.be += r * stride;
    sa.tree += r * stride;
    sa.hs += r * stride;
    sa.he += r * stride;
    stage_tree(lds, sa.tree, sa.tree_stride, sa.depth);
    if (MODE == kModeTiered) sa.mean_len = mean_length(sa);
    __syncthreads();
    const uint64_t tiles = (na + blockDim.x - 1) / blockDim.x;
    uint32_t bad = 0;
    uint64_t sum = 0;
    for (uint64_t t = part; t < tiles; t += per) {
        const uint64_t i = t * blockDim.x + threadIdx.x;
        bool valid = i < na;
        uint32_t as[1] = {valid ? a_start[i] : 0u}, ae[1] = {valid ? a_end[i] : kIdleEnd}, cnt[1], fst[1];
        if (as[0] > ae[0]) {
            bad = 1;
            valid = false;
            ae[0] = as[0];
        }
        icount<1, MODE>(sa, lds, as, ae, cnt, fst);
        sum += valid ? cnt[0] : 0u;
    }
    add_block_sum(sum, totals + r);
    if (bad && sa.status) atomicOr(sa.status, BITS_FLAG_INTERVAL);
}

__global__ void k_mc_tail(const unsigned long long* __restrict__ totals, uint64_t nshuf,
                          const unsigned long long* observed, unsigned long long* n_ge,
                          unsigned long long* n_le) {
    __shared__ unsigned long long red[2][16];
    const unsigned long long obs = *observed;
    uint64_t ge = 0, le = 0;
    for (uint64_t s = threadIdx.x; s < nshuf; s += blockDim.x) {
        ge += totals[s] >= obs;
        le += totals[s] <= obs;
    }
    ge = wave_sum_u64(ge);
    le = wave_sum_u64(le);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][w] = ge;
        red[1][w] = le;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long g = 0, l = 0;
        for (int k = 0; k < (int)(blockDim.x / kWave); ++k) {
            g += red[0][k];
            l += red[1][k];
        }
        *n_ge = g;
        *n_le = l;
    }
}

// Order statistics of the per-shuffle totals (the median of Sec. 3.3): *out0
// and *out1 = the k0-th and k1-th smallest (0-based, k0 <= k1 <= k0 + 1) of
// v[0..n), exact for any n < 2^32, in one workgroup.  Most-significant-digit
// radix selection of the k0-th: the digits all values share are found first
// and skipped (totals of one run differ in their low two or three bytes), then
// each pass histograms the values that match the digits fixed so far, and one
// wave finds the bucket holding the rank with a prefix sum.  The k1-th is the
// same value if enough values are not above it, else the least value above.
// Latency of a pass bounds it; 1000 totals took 49 us with sixteen passes and
// a serial walk of the histogram, 5 us now.
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const unsigned long long y = __shfl_xor(v, o);
        v = y < v ? y : v;
    }
    return v;
}

__global__ void __launch_bounds__(1024) k_select_u64(const unsigned long long* __restrict__ v, uint64_t n,
                                                     uint64_t k0, uint64_t k1, unsigned long long* out0,
                                                     unsigned long long* out1) {
    __shared__ uint32_t hist[256];
    __shared__ unsigned long long red[2][16], sh_prefix, sh_diff;
    __shared__ uint64_t sh_rank;
    __shared__ uint32_t sh_same;
    const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    constexpr int kHeld = 4;   // values a thread keeps in registers; the rest are read again each pass
    unsigned long long held[kHeld];
    const unsigned long long ref = v[0];
    unsigned long long diff = 0ull;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const uint64_t i = threadIdx.x + (uint64_t)u * 1024;
        held[u] = i < n ? v[i] : ref;
        diff |= held[u] ^ ref;
    }
    for (uint64_t i = threadIdx.x + kHeld * 1024; i < n; i += 1024) diff |= v[i] ^ ref;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) diff |= __shfl_xor(diff, o);
    if (lane == 0) red[0][w] = diff;
    if (threadIdx.x < 256) hist[threadIdx.x] = 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long d = 0ull;
        for (int k = 0; k < 16; ++k) d |= red[0][k];
        const int top = d ? (63 - __clzll(d)) / 8 : -1;   // the highest byte in which values differ
        sh_diff = d;
        sh_prefix = top == 7 ? 0ull : ref & (~0ull << (8 * (top + 1)));
        sh_rank = k0;
        sh_same = 0u;
    }
    __syncthreads();
    const unsigned long long d = sh_diff;
    for (int p = d ? (63 - __clzll(d)) / 8 : -1; p >= 0; --p) {
        const unsigned long long mask = p == 7 ? 0ull : ~0ull << (8 * (p + 1)), prefix = sh_prefix;
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            if (threadIdx.x + (uint64_t)u * 1024 < n && (held[u] & mask) == prefix)
                atomicAdd(&hist[(uint32_t)(held[u] >> (8 * p)) & 255u], 1u);
        for (uint64_t i = threadIdx.x + kHeld * 1024; i < n; i += 1024)
            if ((v[i] & mask) == prefix) atomicAdd(&hist[(uint32_t)(v[i] >> (8 * p)) & 255u], 1u);
        __syncthreads();
        if (w == 0) {   // lane l owns buckets 4l .. 4l + 3
            uint32_t c[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) sum += c[k] = hist[4 * lane + k];
            uint32_t x = sum;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const uint32_t y = __shfl_up(x, o);
                if (lane >= (uint32_t)o) x += y;
            }
            const uint64_t r = sh_rank;
            uint64_t cum = x - sum;
            if (r >= cum && r < x) {   // the bucket is one of this lane's
                uint32_t k = 0;
                while (cum + c[k] <= r) cum += c[k++];
                sh_rank = r - cum;
                sh_same = c[k];
                sh_prefix = prefix | ((unsigned long long)(4 * lane + k) << (8 * p));
            }
        }
        __syncthreads();
        if (threadIdx.x < 256) hist[threadIdx.x] = 0u;
        __syncthreads();
    }
    // sh_prefix is the k0-th value, sh_rank its rank among its equals (k0 when all are equal)
    const unsigned long long v0 = sh_prefix;
    const uint64_t same = d ? sh_same : n;
    if (threadIdx.x == 0) *out0 = v0;
    if (sh_rank + (k1 - k0) < same) {
        if (threadIdx.x == 0) *out1 = v0;
        return;
    }
    unsigned long long m = ~0ull;
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (held[u] > v0 && held[u] < m) m = held[u];
    for (uint64_t i = threadIdx.x + kHeld * 1024; i < n; i += 1024) {
        const unsigned long long x = v[i];
        if (x > v0 && x < m) m = x;
    }
    m = wave_min_u64(m);
    if (lane == 0) red[1][w] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 16; ++k) m = red[1][k] < m ? red[1][k] : m;
        *out1 = m;
    }
}

// ------------------------------------------------------------------ projection
__global__ void k_project(ChromTab ct, const uint32_t* __restrict__ chrom, const uint32_t* __restrict__ ls,
                          const uint32_t* __restrict__ le, uint64_t n, uint32_t* __restrict__ gs,
                          uint32_t* __restrict__ ge, uint32_t* status) {
    uint32_t bad = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t c = chrom[i], s = ls[i], e = le[i];
        const bool cok = c < ct.n;
        const uint32_t o = cok ? ct.off[c] : 0u;
        const uint32_t clen = cok ? ct.off[c + 1] - ct.off[c] : 0u;
        if (!cok || e >= clen) bad |= BITS_FLAG_CHROM;
        if (s > e) bad |= BITS_FLAG_INTERVAL;
        gs[i] = o + s;
        ge[i] = o + e;
    }
    if (bad && status) atomicOr(status, bad);
}

// ------------------------------------------------------------------ batched pairs
// Each workgroup owns the contiguous item range [wg_begin[w], wg_begin[w+1]);
// items are sorted by reference, so (plain path) the LDS tree is re-staged
// only when the reference changes.  Consecutive logical workgroups run on the
// same XCD (hardware dispatches workgroups round-robin over the 8 XCDs), so
// an XCD's L2 sees few distinct references (and, on the learned path, their
// leaf records).  kModeTiered takes the form for each reference's size;
// kModeLearned searches every pair through the reference's learned
// index (leaf model, error-window head probe, one line), with the per-wave scratch in LDS.
template <int QPL, int MODE>
__global__ void __launch_bounds__(1024)
    k_batch(const BatchRef* __restrict__ refs, const BatchQuery* __restrict__ qs, const BatchItem* __restrict__ items,
            const uint32_t* __restrict__ wg_begin, uint32_t n_wg, uint32_t n_ref, uint32_t max_depth,
            unsigned long long* __restrict__ pair_totals, uint32_t* status) {
    extern __shared__ __align__(16) uint32_t lds[];
    constexpr bool LEARNED = MODE == kModeLearned;
    const uint32_t g = gridDim.x, b = blockIdx.x;
    const uint32_t per_xcd = g / 8u;
    const uint32_t w = (g % 8u == 0u) ? (b % 8u) * per_xcd + b / 8u : b;
    if (w >= n_wg) return;
    const uint32_t i0 = wg_begin[w], i1 = wg_begin[w + 1];
    uint32_t cur = 0xFFFFFFFFu;
    SearchArgs sa{};
    uint32_t bad = 0;
    // The lane's sum for the pair of the last items: one addition to a total per wave and run
    // of its items (with one per item, 2 x 2 pairs of 1e6 queries against 3e4 keys 295 us, 119 so).
    uint64_t acc = 0, pair = 0;
    auto flush = [&] {
        acc = wave_sum_u64(acc);
        if ((threadIdx.x & (kWave - 1)) == 0 && acc) atomicAdd(pair_totals + pair, (unsigned long long)acc);
        acc = 0;
    };
    for (uint32_t it = i0; it < i1; ++it) {
        const BatchItem item = items[it];
        const uint64_t p = (uint64_t)item.q * n_ref + item.r;
        if (p != pair) flush();
        pair = p;
        if (item.r != cur) {
            const BatchRef R = refs[item.r];
            sa.bs = R.bs;
            sa.be = R.be;
            sa.tree = R.tree;
            sa.rmi = R.rmi;
            sa.hs = R.hs;
            sa.he = R.he;
            sa.status = status;
            sa.fallbacks = R.fallbacks;
            sa.n = R.n;
            sa.tree_stride = R.tree_stride;
            sa.depth = LEARNED ? 0u : min(R.depth, max_depth);
            sa.mean_len = MODE != kModePlain && R.n ? mean_length(sa) : 0.0f;
            if (!LEARNED) {
                __syncthreads();
                stage_tree(lds, sa.tree, sa.tree_stride, sa.depth);
                __syncthreads();
            }
            cur = item.r;
        }
        const BatchQuery Q = qs[item.q];
        uint32_t as[QPL], ae[QPL], cnt[QPL];
        bool valid[QPL];
#pragma unroll
        for (int q = 0; q < QPL; ++q) {
            const uint32_t k = (uint32_t)q * blockDim.x + threadIdx.x;
            const uint64_t i = (uint64_t)item.begin + k;
            valid[q] = k < item.count;
            as[q] = valid[q] ? Q.as[i] : 0u;
            ae[q] = valid[q] ? Q.ae[i] : kIdleEnd;
            if (as[q] > ae[q]) {
                bad = 1;
                valid[q] = false;
                ae[q] = as[q];
            }
        }
        if (sa.n) {   // uniform over the workgroup: every item of the loop is one reference
            uint32_t fst[QPL];
            if (MODE == kModeTiered && direct_form(sa.n, sa.depth))
                icount<QPL, kModeDirect>(sa, lds, as, ae, cnt, fst);
            else
                icount<QPL, MODE>(sa, lds, as, ae, cnt, fst);
        } else {
#pragma unroll
            for (int q = 0; q < QPL; ++q) cnt[q] = 0;
        }
#pragma unroll
        for (int q = 0; q < QPL; ++q) acc += valid[q] ? cnt[q] : 0u;
    }
    flush();
    if (bad) atomicOr(status, BITS_FLAG_INTERVAL);
}

// ------------------------------------------------------------------ window hook
// For keys x[i]: the learned path's window for array `which` (0 = B_S,
// 1 = B_E): lo = wl, hi = wr, or lo = hi = the resolved rank.
__global__ void __launch_bounds__(256) k_rmi_window(SearchArgs sa, uint32_t which, const uint32_t* __restrict__ xs,
                                                    uint64_t n, uint32_t* __restrict__ lo, uint32_t* __restrict__ hi) {
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t* scr = lds + (threadIdx.x / kWave) * probe_scratch_words(1);
    const uint64_t tiles = (n + blockDim.x - 1) / blockDim.x;
    for (uint64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const uint64_t i = t * blockDim.x + threadIdx.x;
        const uint32_t xi = i < n ? xs[i] : 0u;
        uint32_t x[2] = {xi, xi}, base[2], wl[2], wr[2], rlo[2], rhi[2];
        float dens[2];
        bool win[2];
        learned_windows<2>(both_arrays(sa), scr, x, base, wl, wr, rlo, rhi, win, dens);
        if (i < n) {
            lo[i] = win[which] ? wl[which] : base[which];
            hi[i] = win[which] ? wr[which] : base[which];
        }
    }
}

hipError_t launch_rmi_window(const SearchArgs& sa, uint32_t which, const uint32_t* xs, uint64_t n, uint32_t* lo,
                             uint32_t* hi, hipStream_t s) {
    if (!n) return hipSuccess;
    uint64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_rmi_window, dim3((uint32_t)g), dim3(256), search_lds_bytes(true, 0, 1, 256), s, sa, which,
                       xs, n, lo, hi);
    return hipGetLastError();
}

// ------------------------------------------------------------------ fills
__global__ void k_fill_u64(unsigned long long* p, uint64_t n, unsigned long long v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ------------------------------------------------------------------ host side

int device_cu_count() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cached[dev]) {
        int cu = 0;
        if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0) cu = 256;
        cached[dev] = cu;
    }
    return cached[dev];
}

size_t device_lds_per_block() {
    static size_t cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 65536;
    if (!cached[dev]) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
            v = 65536;
        cached[dev] = (size_t)v;
    }
    return cached[dev];
}

// Workgroups resident per CU for a kernel/block/LDS combination (cached).
static int blocks_per_cu(const void* kernel, int block, size_t lds) {
    static std::mutex mu;
    static std::unordered_map<uint64_t, int> cache;
    int dev = 0;
    (void)hipGetDevice(&dev);
    const uint64_t key = ((uint64_t)(uintptr_t)kernel * 1315423911u) ^ ((uint64_t)block << 40) ^ ((uint64_t)lds << 8) ^ (uint64_t)dev;
    {
        std::lock_guard<std::mutex> g(mu);
        auto it = cache.find(key);
        if (it != cache.end()) return it->second;
    }
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, block, lds) != hipSuccess || nb <= 0) nb = 1;
    std::lock_guard<std::mutex> g(mu);
    cache[key] = nb;
    return nb;
}

static uint32_t persistent_grid(const void* kernel, const LaunchCfg& cfg, size_t lds, uint64_t work_items) {
    uint64_t g = cfg.grid ? cfg.grid : (uint64_t)device_cu_count() * blocks_per_cu(kernel, cfg.block, lds);
    if (g > work_items) g = work_items;
    if (g < 1) g = 1;
    return (uint32_t)g;
}

hipError_t launch_fill_u64(unsigned long long* p, uint64_t n, unsigned long long v, hipStream_t s) {
    if (!n) return hipSuccess;
    uint64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_fill_u64, dim3((uint32_t)g), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
    if (!n) return hipSuccess;
    uint64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)g), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// The kernel mode of a launch's path (the tiered path has two forms).
static int search_mode(const SearchArgs& sa, const LaunchCfg& cfg, bool counting = false) {
    if (cfg.path == BITS_PATH_LEARNED) return counting && sa.n <= kPairedKeys ? kModePaired : kModeLearned;
    if (cfg.path == BITS_PATH_TIERED) return direct_form(sa.n, sa.depth) ? kModeDirect : kModeTiered;
    return kModePlain;
}

template <int QPL, int MODE>
static hipError_t launch_count_t(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                                 uint64_t na, uint32_t* counts, uint32_t* firsts, unsigned long long* total,
                                 hipStream_t s) {
    const size_t lds = search_lds_bytes(learned_mode(MODE), sa.depth, QPL, cfg.block);
    const uint64_t tile = (uint64_t)cfg.block * QPL;
    const void* kern = (const void*)k_count<QPL, MODE>;
    const uint32_t grid = persistent_grid(kern, cfg, lds, (na + tile - 1) / tile);
    hipLaunchKernelGGL((k_count<QPL, MODE>), dim3(grid), dim3(cfg.block), lds, s, sa, as, ae, na, counts, firsts,
                       total);
    return hipGetLastError();
}

template <int QPL>
static hipError_t launch_count_q(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                                 uint64_t na, uint32_t* counts, uint32_t* firsts, unsigned long long* total,
                                 hipStream_t s) {
    switch (search_mode(sa, cfg, true)) {
        case kModeLearned:
            return launch_count_t<QPL, kModeLearned>(sa, cfg, as, ae, na, counts, firsts, total, s);
        case kModePaired:
            return launch_count_t<QPL, kModePaired>(sa, cfg, as, ae, na, counts, firsts, total, s);
        case kModeTiered:
            return launch_count_t<QPL, kModeTiered>(sa, cfg, as, ae, na, counts, firsts, total, s);
        case kModeDirect:
            return launch_count_t<QPL, kModeDirect>(sa, cfg, as, ae, na, counts, firsts, total, s);
        default:
            return launch_count_t<QPL, kModePlain>(sa, cfg, as, ae, na, counts, firsts, total, s);
    }
}

// The shape of a search when the caller left it open.  Without a model: one
// query per lane, and the largest workgroup that still gives every CU (of a
// given number of workgroups, half of them) one
// (each stages its own copy of the top trees; 1e5 queries by one workgroup of
// 256 threads 1840 us, of 1024 840).  With one: small workgroups,
// which stage nothing and finish apart, and one query per lane (1024 threads
// lowered to what the LDS scratch of two queries per lane allows, before:
// counting 1e4 queries in 1e4 23.6 -> 14.3 us, 1e5 in 5e6 34.0 -> 17.5, 5e7 in
// 5e7 3180 -> 3050), two in large counts against small references, whose two
// searches go in step (1.5e7 in 2e4 455 and 439 us).
static LaunchCfg open_shape(const LaunchCfg& cfg, uint32_t n, uint64_t na) {
    LaunchCfg c = cfg;
    if (!c.open) return c;
    if (c.path == BITS_PATH_LEARNED) {
        c.qpl = n <= kPairedKeys && na >= (1u << 20) ? 2u : 1u;
        c.block = 256u;
    }
    if (c.path != BITS_PATH_TIERED) return c;
    const uint64_t cus = c.grid ? c.grid / 2 : (uint64_t)device_cu_count();
    c.qpl = 1;
    c.block = na >= 1024 * cus ? 1024u : na >= 512 * cus ? 512u : 256u;
    return c;
}

// The same for the shuffles.  A larger workgroup sorts more placements at once,
// which pays when many of them, over items of many shuffles, search a large
// reference (256, 512, 1024 threads: 1e6 x 200 against 5e7 keys 9730, 9480,
// 9140 us, 1e6 x 50 2590, 2550, 2500, 1e6 x 10 798, 844, 925; 1e6 x 400
// against 1e7 16000, 15650, 15270, 1e6 x 40 1729, 1716, 1734, 1e7 x 10 7200,
// 7610, 8050; 1e6 x 160 against 5e6 5830, 5880, 5770, against 2e6 5290, 5400,
// 5375; 1e5 x 100 against 1e6 369, 374, 417).
static LaunchCfg open_shuffle_shape(const LaunchCfg& cfg, uint32_t n, uint64_t na, uint64_t nshuf) {
    LaunchCfg c = open_shape(cfg, n, na * nshuf);
    if (c.open && c.path == BITS_PATH_LEARNED) {
        c.qpl = 1u;
        c.block = n >= (1u << 23) && nshuf >= kMaxChunk / 2 && na * nshuf >= (1u << 25) ? 1024u : 256u;
    }
    return c;
}

hipError_t launch_count(const SearchArgs& sa, const LaunchCfg& cfg0, const uint32_t* as, const uint32_t* ae,
                        uint64_t na, uint32_t* counts, unsigned long long* total, hipStream_t s, uint32_t* firsts) {
    if (!na) return hipSuccess;
    const LaunchCfg cfg = open_shape(cfg0, sa.n, na);
    switch (cfg.qpl) {
        case 1: return launch_count_q<1>(sa, cfg, as, ae, na, counts, firsts, total, s);
        case 4: return launch_count_q<4>(sa, cfg, as, ae, na, counts, firsts, total, s);
        default: return launch_count_q<2>(sa, cfg, as, ae, na, counts, firsts, total, s);
    }
}

static int fill_chrom_tab(const uint32_t* chrom_len, uint32_t n_chrom, ChromTab* ct) {
    if (n_chrom == 0 || n_chrom > BITS_MAX_CHROM) return BITS_E_ARG;
    uint64_t acc = 0;
    ct->n = n_chrom;
    for (uint32_t c = 0; c < n_chrom; ++c) {
        ct->off[c] = (uint32_t)acc;
        acc += chrom_len[c];
        if (acc > 0xFFFFFFFFull) return BITS_E_CHROM;
    }
    ct->off[n_chrom] = (uint32_t)acc;
    for (uint32_t c = n_chrom + 1; c <= BITS_MAX_CHROM; ++c) ct->off[c] = (uint32_t)acc;
    return BITS_OK;
}

hipError_t launch_mc_zero(unsigned long long* totals, uint64_t ns, unsigned long long* observed, const McTable* tab,
                          hipStream_t s) {
    const uint64_t g = (ns + 255) / 256;
    hipLaunchKernelGGL(k_mc_zero, dim3((uint32_t)(g < 1 ? 1 : g > 4096 ? 4096 : g)), dim3(256), 0, s, totals, ns,
                       observed, tab ? tab->hist : nullptr, tab ? tab->cursor : nullptr);
    return hipGetLastError();
}

hipError_t launch_mc_prepare(const uint32_t* as, const uint32_t* ae, uint64_t na, const uint32_t* chrom_len,
                             uint32_t n_chrom, const McTable& tab, void* packed, uint32_t* status, hipStream_t s) {
    ChromTab ct;
    if (fill_chrom_tab(chrom_len, n_chrom, &ct) != BITS_OK) return hipErrorInvalidValue;
    if (!na) return hipSuccess;
    uint64_t g = (na + 1023) / 1024;
    hipLaunchKernelGGL(k_mc_hist, dim3((uint32_t)(g < 256 ? g : 256)), dim3(1024), 0, s, as, na, ct, tab.hist,
                       tab.cursor);
    if (g > 1024) g = 1024;
    hipLaunchKernelGGL(k_mc_prepare, dim3((uint32_t)g), dim3(1024), 0, s, as, ae, na, ct, tab.cursor, tab.off,
                       tab.span, tab.len, tab.idx, (uint2*)packed, status);
    return hipGetLastError();
}

template <int QPL, int MODE>
static hipError_t launch_mc_t(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                              const McTable& tab, uint64_t na, uint64_t seed, uint64_t s0, uint64_t nshuf,
                              unsigned long long* totals, unsigned long long* observed, hipStream_t s) {
    constexpr bool LEARNED = MODE == kModeLearned;
    const size_t lds = search_lds_bytes(LEARNED, sa.depth, QPL, cfg.block);
    const uint64_t tile = (uint64_t)cfg.block * QPL;
    const uint64_t tps = (na + tile - 1) / tile;
    if (observed) {
        const void* ko = (const void*)k_mc<QPL, MODE, true>;
        const uint32_t go = persistent_grid(ko, cfg, lds, tps);
        hipLaunchKernelGGL((k_mc<QPL, MODE, true>), dim3(go), dim3(cfg.block), lds, s, sa, as, ae, tab.off,
                           tab.span, tab.len, tab.idx, na, seed, s0, (uint64_t)1, tps, 1u, observed);
    }
    // the sorted kernel when its LDS (dynamic + ~7 KB static) fits the device's per-workgroup limit
    if (nshuf && LEARNED && BITS_MC_SORTED && sort_lds_bytes(cfg.block) + 8192 <= device_lds_per_block()) {
        const size_t lds1 = sort_lds_bytes(cfg.block);
        const uint64_t tq = (na + sort_tile_q(cfg.block) - 1) / sort_tile_q(cfg.block);
        const void* km = (const void*)k_mc_sorted;
        const uint32_t gm = persistent_grid(km, cfg, lds1, nshuf * tq);
        uint32_t chunk = kMaxChunk;
        while (chunk > 1 && tq * ((nshuf + chunk - 1) / chunk) < 8ull * gm) chunk >>= 1;
        hipLaunchKernelGGL(k_mc_sorted, dim3(gm), dim3(cfg.block), lds1, s, sa, tab.off, tab.span, tab.len, tab.idx,
                           na, seed, s0, nshuf, tq, chunk, totals);
    } else if (nshuf) {
        const void* km = (const void*)k_mc<QPL, MODE, false>;
        const uint32_t gm = persistent_grid(km, cfg, lds, nshuf * tps);
        // shuffles per work item: as many as keep >= 8 items per workgroup
        uint32_t chunk = kMaxChunk;
        while (chunk > 1 && tps * ((nshuf + chunk - 1) / chunk) < 8ull * gm) chunk >>= 1;
        hipLaunchKernelGGL((k_mc<QPL, MODE, false>), dim3(gm), dim3(cfg.block), lds, s, sa, as, ae, tab.off,
                           tab.span, tab.len, tab.idx, na, seed, s0, nshuf, tps, chunk, totals);
    }
    return hipGetLastError();
}

template <int QPL>
static hipError_t launch_mc_q(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                              const McTable& tab, uint64_t na, uint64_t seed, uint64_t s0, uint64_t nshuf,
                              unsigned long long* totals, unsigned long long* observed, hipStream_t s) {
    switch (search_mode(sa, cfg)) {
        case kModeLearned:
            return launch_mc_t<QPL, kModeLearned>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
        case kModeTiered:
            return launch_mc_t<QPL, kModeTiered>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
        case kModeDirect:
            return launch_mc_t<QPL, kModeDirect>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
        default:
            return launch_mc_t<QPL, kModePlain>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
    }
}

hipError_t launch_mc(const SearchArgs& sa, const LaunchCfg& cfg0, const uint32_t* as, const uint32_t* ae,
                     const McTable& tab, uint64_t na, uint64_t seed, uint64_t s0, uint64_t nshuf,
                     unsigned long long* totals, unsigned long long* observed, hipStream_t s) {
    if (!na) return hipSuccess;
    const LaunchCfg cfg = nshuf ? open_shuffle_shape(cfg0, sa.n, na, nshuf) : open_shape(cfg0, sa.n, na);
    switch (cfg.qpl) {
        case 1: return launch_mc_q<1>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
        case 4: return launch_mc_q<4>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
        default: return launch_mc_q<2>(sa, cfg, as, ae, tab, na, seed, s0, nshuf, totals, observed, s);
    }
}

template <int QPL, int MODE>
static hipError_t launch_decide_t(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                                  uint64_t na, uint32_t* found, unsigned long long* witness, hipStream_t s) {
    const size_t lds = search_lds_bytes(learned_mode(MODE), sa.depth, QPL, cfg.block);
    const uint64_t tile = (uint64_t)cfg.block * QPL;
    const void* kern = (const void*)k_decide<QPL, MODE>;
    const uint32_t grid = persistent_grid(kern, cfg, lds, (na + tile - 1) / tile);
    hipLaunchKernelGGL((k_decide<QPL, MODE>), dim3(grid), dim3(cfg.block), lds, s, sa, as, ae, na, found, witness);
    return hipGetLastError();
}

template <int QPL>
static hipError_t launch_decide_q(const SearchArgs& sa, const LaunchCfg& cfg, const uint32_t* as, const uint32_t* ae,
                                  uint64_t na, uint32_t* found, unsigned long long* witness, hipStream_t s) {
    switch (search_mode(sa, cfg, true)) {
        case kModeLearned: return launch_decide_t<QPL, kModeLearned>(sa, cfg, as, ae, na, found, witness, s);
        case kModePaired: return launch_decide_t<QPL, kModePaired>(sa, cfg, as, ae, na, found, witness, s);
        case kModeTiered: return launch_decide_t<QPL, kModeTiered>(sa, cfg, as, ae, na, found, witness, s);
        case kModeDirect: return launch_decide_t<QPL, kModeDirect>(sa, cfg, as, ae, na, found, witness, s);
        default: return launch_decide_t<QPL, kModePlain>(sa, cfg, as, ae, na, found, witness, s);
    }
}

hipError_t launch_decide(const SearchArgs& sa, const LaunchCfg& cfg0, const uint32_t* as, const uint32_t* ae,
                         uint64_t na, uint32_t* found, unsigned long long* witness, hipStream_t s) {
    if (!na) return hipSuccess;
    const LaunchCfg cfg = open_shape(cfg0, sa.n, na);
    switch (cfg.qpl) {
        case 1: return launch_decide_q<1>(sa, cfg, as, ae, na, found, witness, s);
        case 4: return launch_decide_q<4>(sa, cfg, as, ae, na, found, witness, s);
        default: return launch_decide_q<2>(sa, cfg, as, ae, na, found, witness, s);
    }
}

hipError_t launch_select_u64(const unsigned long long* v, uint64_t n, uint64_t k0, uint64_t k1,
                             unsigned long long* out0, unsigned long long* out1, hipStream_t s) {
    hipLaunchKernelGGL(k_select_u64, dim3(1), dim3(1024), 0, s, v, n, k0, k1, out0, out1);
    return hipGetLastError();
}

hipError_t launch_place_rounds(const McTable& tab, const uint32_t* b_start, uint64_t nb, uint64_t stride,
                               uint64_t seed, uint64_t s0, uint32_t rounds, bool identity, uint32_t* S, uint32_t* E,
                               hipStream_t s) {
    const uint64_t total = (uint64_t)rounds * nb;
    if (!total) return hipSuccess;
    uint64_t g = (total + 255) / 256;
    if (g > 16384) g = 16384;
    hipLaunchKernelGGL(k_place_rounds, dim3((uint32_t)g), dim3(256), 0, s, tab.off, tab.span, tab.len, tab.idx,
                       b_start, nb, stride, seed, s0, rounds, identity ? 1u : 0u, S, E);
    return hipGetLastError();
}

hipError_t launch_fill_tails(uint32_t* S, uint32_t* E, uint64_t nb, uint64_t stride, uint32_t rounds, hipStream_t s) {
    const uint32_t words = (uint32_t)(stride - nb) * rounds;   // < 32 * 4096
    if (!words) return hipSuccess;
    hipLaunchKernelGGL(k_fill_tails, dim3((words + 255) / 256), dim3(256), 0, s, S, E, nb, stride, rounds);
    return hipGetLastError();
}

hipError_t launch_count_rounds(const uint32_t* S, const uint32_t* E, uint64_t nb, uint64_t stride, uint32_t rounds,
                               uint32_t* trees, uint32_t* heads, const uint32_t* as, const uint32_t* ae, uint64_t na,
                               unsigned long long* totals, uint32_t* status, hipStream_t s) {
    if (!na || !rounds) return hipSuccess;
    SearchArgs sa{};
    sa.status = status;
    sa.n = (uint32_t)nb;
    sa.bs = S;
    sa.be = E;
    sa.tree = trees;
    sa.hs = heads;
    sa.he = heads + heads_len(nb);
    // both trees of a round fit its segment: 2 * 2^depth <= stride, and depth <= floor(log2 nb)
    while (sa.depth < BITS_MAX_DEPTH && (4ull << sa.depth) <= stride && (2ull << sa.depth) <= nb) ++sa.depth;
    sa.tree_stride = 1u << sa.depth;
    const uint64_t words = (2ull << sa.depth) + (nb > kDirectKeys ? 2 * heads_len(nb) : 0);
    hipLaunchKernelGGL(k_round_index, dim3((uint32_t)((words + 255) / 256 < 256 ? (words + 255) / 256 : 256), rounds),
                       dim3(256), 0, s, S, E, (uint32_t)nb, stride, sa.depth, trees, heads);
    const uint32_t block = 512;
    const uint64_t tiles = (na + block - 1) / block;
    const uint32_t xg = rounds >= kXcds ? kXcds : 1u, turns = (rounds + xg - 1) / xg;
    const uint64_t most = rounds >= kXcds ? kRoundParts : 2ull * device_cu_count() / rounds;
    const uint32_t per = (uint32_t)(tiles < most ? tiles : most);
    const size_t lds = search_lds_bytes(false, sa.depth, 1, block);
    if (nb > kDirectKeys)
        hipLaunchKernelGGL(k_count_rounds<kModeTiered>, dim3(xg * turns * per), dim3(block), lds, s, sa, stride, rounds,
                           per, as, ae, na, totals);
    else
        hipLaunchKernelGGL(k_count_rounds<kModeDirect>, dim3(xg * turns * per), dim3(block), lds, s, sa, stride, rounds,
                           per, as, ae, na, totals);
    return hipGetLastError();
}

hipError_t launch_mc_tail(const unsigned long long* totals, uint64_t nshuf, const unsigned long long* observed,
                          unsigned long long* n_ge, unsigned long long* n_le, hipStream_t s) {
    hipLaunchKernelGGL(k_mc_tail, dim3(1), dim3(1024), 0, s, totals, nshuf, observed, n_ge, n_le);
    return hipGetLastError();
}

hipError_t launch_project(const uint32_t* chrom_len, uint32_t n_chrom, const uint32_t* chrom, const uint32_t* ls,
                          const uint32_t* le, uint64_t n, uint32_t* gs, uint32_t* ge, uint32_t* status,
                          hipStream_t s) {
    ChromTab ct;
    if (fill_chrom_tab(chrom_len, n_chrom, &ct) != BITS_OK) return hipErrorInvalidValue;
    if (!n) return hipSuccess;
    uint64_t g = (n + 255) / 256;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(k_project, dim3((uint32_t)g), dim3(256), 0, s, ct, chrom, ls, le, n, gs, ge, status);
    return hipGetLastError();
}

template <int QPL>
static const void* batch_kernel_q(uint32_t path) {
    switch (path) {
        case BITS_PATH_LEARNED: return (const void*)k_batch<QPL, kModeLearned>;
        case BITS_PATH_TIERED: return (const void*)k_batch<QPL, kModeTiered>;
        default: return (const void*)k_batch<QPL, kModePlain>;
    }
}

static const void* batch_kernel(uint32_t qpl, uint32_t path) {
    switch (qpl) {
        case 1: return batch_kernel_q<1>(path);
        case 4: return batch_kernel_q<4>(path);
        default: return batch_kernel_q<2>(path);
    }
}

static size_t batch_lds(const LaunchCfg& cfg, uint32_t max_depth) {
    return search_lds_bytes(cfg.path == BITS_PATH_LEARNED, max_depth, (int)cfg.qpl, cfg.block);
}

hipError_t launch_batch(const BatchRef* refs, const BatchQuery* qs, const BatchItem* items, const uint32_t* wg_begin,
                        uint32_t n_wg, uint32_t n_ref, uint32_t max_depth, const LaunchCfg& cfg,
                        unsigned long long* pair_totals, uint32_t* status, hipStream_t s) {
    const size_t lds = batch_lds(cfg, max_depth);
    const void* k = batch_kernel(cfg.qpl, cfg.path);
    void* args[] = {(void*)&refs, (void*)&qs, (void*)&items, (void*)&wg_begin, (void*)&n_wg, (void*)&n_ref,
                    (void*)&max_depth, (void*)&pair_totals, (void*)&status};
    return hipLaunchKernel(k, dim3(n_wg), dim3(cfg.block), args, lds, s);
}

int batch_blocks_per_cu(const LaunchCfg& cfg, uint32_t max_depth) {
    return blocks_per_cu(batch_kernel(cfg.qpl, cfg.path), (int)cfg.block,
                         batch_lds(cfg, max_depth));
}

}  // namespace bits
