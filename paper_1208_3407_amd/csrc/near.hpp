// The step rule of the search for a query's second rank next to its first one
// (search.hip, icount_near): plain arithmetic on line counts, compiled for the
// kernels and for the host.
#ifndef BITS_NEAR_HPP
#define BITS_NEAR_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bits {

constexpr uint32_t kNoLine = 0xFFFFFFFFu;
// Expected hits up to which a line is looked at: with more the line is missed
// too often and the look comes on top of the full search.  1e7 queries against
// 5e6 keys through the model with 30, 50, 80, 130, 180 hits each: at 64 in
// every lane of the wave 624, 650, 649, 648, 648 us; at 160 622, 686, 758, 649, 649;
// at 64 lane by lane 620, 717, 712, 650, 647; both searches in full 648.
constexpr float kNearCount = 64.0f;

// One step towards r = #{K < x}: cnt = #{keys < x} of the line at w.  On
// return either r is known (true), or w is the neighbouring line to look at
// and r the line boundary between the two, which the step has bounded r by
// from one side; the neighbour bounding it from the other side decides it.
// Before the first step r is kNoLine.
__host__ __device__ inline bool near_step(uint32_t n, uint32_t cnt, uint32_t& w, uint32_t& r) {
    if (cnt == 0u) {                       // rank <= w
        if (w == 0u) r = 0u;
        if (w == 0u || r == w) return true;   // r == w: the line to the left is full
        r = w;
        w -= 32u;
        return false;
    }
    const uint32_t end = w + cnt;
    if (cnt < 32u || end >= n || r == end) {  // r == end: the line to the right counts 0
        r = end;
        return true;
    }
    r = w += 32u;                          // rank >= w
    return false;
}

// first, the starts' density and the query -> the first line to look at, or
// kNoLine for the full search; `done` when #{B_E < s} is 0 without a look.
__host__ __device__ inline uint32_t near_line(uint32_t n, uint32_t first, float dens, float mean, uint32_t s, uint32_t e,
                                              bool& done) {
    done = s == 0u;
    const float est = dens * ((float)(e - s) + mean);
    if (done || e == 0xFFFFFFFFu || !(est <= kNearCount)) return kNoLine;
    const uint32_t back = 1u + (uint32_t)est;
    const uint32_t at = first > back ? first - back : 0u;
    return (at < n - 1u ? at : n - 1u) & ~31u;
}

}  // namespace bits

#endif
