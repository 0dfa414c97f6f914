// Into how many shares the ranking of a head is cut, and what a share may hold (alr.hip).
#pragma once
#include <stdint.h>

namespace l2kv {

constexpr int kSortLanes = 1024;
constexpr int kListPer = 20;                         // 4-byte words of the LDS list per lane
constexpr int kListWords = kListPer * kSortLanes;    // 80 KB
constexpr int kListAhead = 4;                        // words read past the last element of a share
constexpr uint32_t kMaxBin = 1024;                   // elements of one bin of a head that is cut along bins
// What a share may be given, so that the list holds it with what its last bin may bring with it: logits, and norms with their positions.
constexpr uint32_t kLongestShare = kListWords - kListAhead - kMaxBin, kLongestRankedShare = kListWords / 2 - kListAhead - kMaxBin;

// How many workgroups share a head; 0: one workgroup per head and the counting passes.  `longest` = elements
// a share may be given.
//  - as many as that needs;
//  - more while the launch has fewer workgroups than compute units, down to 2048 elements each;
//  - every share goes over all keys of its head, one head by the passes is one workgroup's, so many long heads
//    are the passes'.  Norms, ms by shares (distinct norms, 30 % zero) and by the passes: 16 heads of 1M 5.2, 6.4
//    and 8.4, 7.6; 32 of 1M 9.7, 11.9 and 11.5, 10.0; 64 of 1M 18.2, 23.2 and 16.4, 13.2; 64 of 400k 1.5, 3.9 and 5.9, 4.6;
//    512 of 131k 1.6, 4.1 and 6.4, 4.7.  Scores: 32 heads of 1M 5.0, 5.9 and 6.0, 6.5; 64 of 1M 10.2, 11.8 and 9.1, 8.7.
//    Heads of more than kCrowded elements cannot do without the sort of their shares, shorter ones mostly can.
inline int64_t share_plan(int64_t n_heads, int64_t T, int64_t longest) {
    constexpr int64_t kLongest = int64_t{1} << 23;     // the records of all shares of a head fit the LDS list
    constexpr int64_t kCrowded = 3 << 18;
    if (T > kLongest) return 0;
    int64_t shares = (T + longest - 1) / longest;
    if (T > kCrowded ? n_heads * shares > 2048 : shares > 64 && n_heads * shares > 4096) return 0;
    const int64_t fill = (256 + n_heads - 1) / n_heads, most = (T + 2047) / 2048;
    const int64_t want = fill < most ? fill : most;
    if (want > shares) shares = want;
    return n_heads * shares <= 0x7fffffffLL ? shares : 0;      // ceil(T / shares) <= longest
}

// Keys per lane of the kernel for a head's scores, 0: they do not stay in registers.  Every one costs the same whether it is there or not
// (12000 tokens at 32: 41.3 us, at 16: 36.6).
inline int score_keys_per_lane(int64_t T) {
    for (const int per : {8, 16, 20, 24, 32}) {
        if (T <= per * kSortLanes) return per;
    }
    return 0;
}
// Most blocks of 1024 positions of a share there: all, or half of them where a head of more than kListPer blocks has two shares.
__host__ __device__ constexpr uint32_t position_slots(int per) { return per <= kListPer ? per : (per + 1) / 2; }
static_assert(kListPer * kSortLanes >= kLongestShare, "heads of more blocks have two shares");

}  // namespace l2kv
