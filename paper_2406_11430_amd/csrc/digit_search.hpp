// Search for the k-th smallest of many 32-bit keys by the 1024 lanes of a workgroup: histograms of digits in
// LDS, and the digit that holds the k-th key.
#pragma once
#include "l2kv_device.hpp"

namespace l2kv {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWaveSize;   // 16

// Digits of a search over whole keys, from the top.
constexpr int kTopBits = 12, kMidBits = 10, kLowBits = 10;
static_assert(kTopBits + kMidBits + kLowBits == 32, "digits cover the key");
constexpr int kTopBins = 1 << kTopBits, kMidBins = 1 << kMidBits, kLowBins = 1 << kLowBits;

// LDS histogram of kCopies interleaved counters per digit; lane l counts in copy l % kCopies.  LDS
// atomics on one address are served one lane at a time, so the copies bound what tied or padded
// rows (all keys in one digit) cost: 32k equal keys per head took 35 us with 4 copies, 94 us with
// one, when three digits were counted, and ordinary norms the same either way.
constexpr int kCopies = 4;
__device__ __forceinline__ void count_digit(uint32_t* hist, uint32_t digit) {
    atomicAdd(&hist[digit * kCopies + threadIdx.x % kCopies], 1u);
}
__device__ __forceinline__ uint32_t digit_count(const uint32_t* hist, uint32_t digit) {
    const uint4 c = reinterpret_cast<const uint4*>(hist)[digit];
    static_assert(kCopies == 4, "one 16-byte read per digit");
    return c.x + c.y + c.z + c.w;
}
// Clears `words` counters, a multiple of 4 * 1024.
__device__ __forceinline__ void clear_counts(uint32_t* hist, int words) {
    for (int i = threadIdx.x; i < words / 4; i += kSelThreads) reinterpret_cast<uint4*>(hist)[i] = make_uint4(0, 0, 0, 0);
}

// Where the k-th key lies in a histogram: its digit and the number of keys in lower digits.
struct Found { uint32_t digit, below, count; };

struct FindShared {
    uint32_t wave_total[kSelWaves];
    Found found;
};

// Sum of the entries [0, wave) of a table with one entry per wave: lane i of each DPP row reads entry i.  (All entries in
// every lane take 16 registers, which kernels that hold rows in flight meanwhile do not have.)
__device__ __forceinline__ uint32_t sum_before(const uint32_t* per_wave, int wave) {
    static_assert(kSelWaves == kRowLanes, "one entry per lane of a row");
    const int i = threadIdx.x % kRowLanes;
    const uint32_t v = per_wave[i];
    return __builtin_amdgcn_readfirstlane(row16_sum(i < wave ? v : 0u));
}

// Called by all 1024 lanes, hist complete (the caller's barrier); ends with a barrier.  `want`
// is 1-based and at most the sum of the histogram.
template <int BINS>
__device__ __forceinline__ Found find_digit(const uint32_t* hist, uint32_t want, FindShared& sh) {
    constexpr int kPer = BINS / kSelThreads;
    static_assert(kPer >= 1 && BINS % kSelThreads == 0, "whole bins per lane");
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    uint32_t c[kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        c[i] = digit_count(hist, threadIdx.x * kPer + i);
        sum += c[i];
        if (i % 2 == 1) __builtin_amdgcn_sched_barrier(0);            // 8 registers for the copies, not 16, as in sum_before
    }
    const uint32_t incl = wave_inclusive_sum(sum);
    if (lane == kWaveSize - 1) sh.wave_total[wave] = incl;
    __syncthreads();
    uint32_t before = incl - sum + sum_before(sh.wave_total, wave);
    if (before < want && want <= before + sum) {          // exactly one lane
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (before < want && want <= before + c[i]) {
                sh.found.digit = (uint32_t)(threadIdx.x * kPer + i);
                sh.found.below = before;
                sh.found.count = c[i];
            }
            before += c[i];
        }
    }
    __syncthreads();
    return sh.found;
}

}  // namespace l2kv
