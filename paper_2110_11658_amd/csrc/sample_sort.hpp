// sample_sort.hpp -- sizes and sample places of the sample sort (sort.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbh {

constexpr int kSsCap = 8192;        // keys one workgroup sorts in LDS
constexpr int kSsOver = 8;          // samples a bucket
constexpr int kSsMaxS = 2048;
constexpr int64_t kSsMaxN = (int64_t)kSsMaxS * 2048;

// Buckets of n keys (n > kSsCap): 1024 to 2048 keys each on average.
inline int ss_buckets(int64_t n) {
    int s = 4;
    while (s < kSsMaxS && (int64_t)s * 2048 < n) s <<= 1;
    return s;
}

// Place of sample j of m: a pseudo-random one of the j-th of m equal stretches of the
// n keys (j < m <= n <= kSsMaxN; places rise with j). The first of each stretch would
// show one phase of an order with a period: at a power of two the stretches are 256
// keys, of which a lattice in row order, or particles in pairs, have the like. One
// bucket then held up to half of the keys, and its workgroup sorted it through global
// memory. Builds in ms, first of each stretch / drawn: lattice of 64^3 points 0.80 /
// 0.17, of 128 x 64 x 128 6.06 / 0.31, 2^20 particles with every second one in a clump
// 8.40 / 0.51, in random order 0.43 / 0.42.
__host__ __device__ inline int64_t ss_sample_at(int64_t j, int64_t n, int64_t m) {
    const int64_t a = j * n / m, len = (j + 1) * n / m - a;
    constexpr uint64_t kOdd = 0x9e3779b97f4a7c15ull;   // 2^64 / golden ratio
    uint64_t h = (uint64_t)(j + 1) * kOdd;
    h = (h ^ (h >> 32)) * kOdd;
    return a + (int64_t)(((h >> 32) * (uint64_t)len) >> 32);
}

}  // namespace pbh
