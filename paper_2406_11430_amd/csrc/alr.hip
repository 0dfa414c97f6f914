// Attention-loss analysis of Sec. 3 on the GPU: for every query head, the
// attention mass lost by dropping m pairs by key norm (Eq. 5), the loss of the
// ideal rule that drops the m lowest attention scores (reference of Eq. 6) and
// the sum over m = 1..T of their gap (Eq. 7).
//
// Sum over m in closed form.  With r(p) = number of pairs the norm rule discards
// before p, pair p is inside the dropped set for T - r(p) values of m, so
//     sum_m L^m     = sum_p a_p (T - r(p)),
//     sum_m L^m,ref = sum_j a_(j) (T - j)       (a_(0) <= a_(1) <= ... ascending),
//     Y             = sum_j a_(j) j - sum_p a_p r(p).
// r depends only on the key norms: it is the rank of (norm bits, position) in its KV head
// (norm_ranks_kernel) and is shared by all queries.  The second term is then a dot product; the
// first needs the scores of one query in ascending order.
//
// Both need the rank of every element among the n of its head, not the sorted array.
// A head is shared by several workgroups (share_plan has the rule), each of which ranks a
// range of VALUES holding about n / shares elements: it counts all keys of the head in
// 4096 bins of equal width between the smallest and the largest key (the few hundred KB of
// a head come from the L2), takes the bins whose first element falls into its range of
// ranks, and ranks those few thousand elements in LDS: counted again in 8192 finer bins,
// put into bin order, each then compared with the one or two others of its bin.  The scores of heads of more than 8192 tokens whose keys
// stay in registers are counted once, in 20480 bins, and sorted in runs of 32 (order_share).
// What bounds it is the passes of every workgroup over all keys of its head (fetch, LDS counting,
// gathering: two thirds of the time) and the LDS round trips of the comparisons, so the
// shares are as few as the LDS list allows until they fill the chip.  (One workgroup per
// head and four counting passes of 8 bits over global memory, which this replaces, took
// 196 us for 32 heads of 32k norms and 221 us for 128 heads of scores; now 21 and 28 us.
// 131k norms of 8 heads: 671 -> 52 us.)
// Where the bins do not separate the keys -- more than kMaxBin elements in a bin of the head, more than
// kMaxFine in a finer one, more than kMaxOfBin in one of the single count: tied or clustered rows, one outlier that stretches the bins of a long head, heads
// of a million elements -- a share finds the elements of its ranks exactly and sorts them (sorted_range).
// Short heads are sorted whole, one small workgroup each (is_short, sort_head).  The counting passes, one workgroup per
// head, remain for many long heads (share_plan).
//
// The counting passes are a least-significant-digit radix sort (4 passes of 8 bits) by
// one 1024-lane workgroup.  Each wavefront owns a contiguous chunk of
// the input; a pass counts digits per wavefront in LDS, turns the 16 x 256 counts
// into start offsets (digit-major, wavefront-minor, which keeps the pass stable)
// and scatters in input order, ranking the 64 keys of a step against each other
// with wave ballots.  Data ping-pongs between two global buffers that stay in
// L2; all waves of a workgroup share one vector L1, so a workgroup barrier is all
// the ordering the passes need.
//
// Unnormalised scores e_p = 2^(s_p - max) are ranked by their logits and summed (double
// accumulators, fixed order), and the three results are divided by sum_p e_p at
// the end.
#include "digit_search.hpp"
#include "l2kv_device.hpp"
#include "l2kv_host.hpp"
#include "position_blocks.hpp"
#include "rank_shares.hpp"

#include <cstddef>
#include <type_traits>

namespace l2kv {
namespace {

constexpr int kSortWaves = kSortLanes / kWaveSize;
constexpr int kRadixBits = 8;
constexpr int kBins = 1 << kRadixBits;
constexpr int kBatch = 8;            // keys per lane fetched together

struct SortShared {
    uint32_t hist[kSortWaves][kBins];   // per-wave digit counts, then running output offsets
    uint32_t digit_base[kBins];         // first output position of each digit
};

// What a pass reads as payload and what it writes.
enum PassKind {
    kKeysOnly,      // keys in, keys out
    kIotaIn,        // payload in = position; (key, payload) out
    kPairs,         // (key, payload) in and out
    kRankOut        // (key, payload) in; writes out_val[payload] = n - 1 - output position
};

// One stable counting pass on digit (key >> shift) & 255 over n keys.  Called by
// all 1024 lanes of the workgroup; leaves a barrier behind it.
template <PassKind KIND>
__device__ void radix_pass(const uint32_t* in_key, const uint32_t* in_val, uint32_t* out_key,
                           uint32_t* out_val, int64_t n, int shift, SortShared& sh) {
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    // contiguous chunk of this wavefront, a multiple of 64 keys
    const int64_t chunk = ((n + kSortWaves - 1) / kSortWaves + kWaveSize - 1) / kWaveSize * kWaveSize;
    const int64_t lo = wave * chunk < n ? wave * chunk : n;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;

    for (int i = threadIdx.x; i < kSortWaves * kBins; i += kSortLanes) (&sh.hist[0][0])[i] = 0u;
    __syncthreads();
    // kBatch independent loads are issued before their first use, so a wavefront
    // pays the L2 latency once per kBatch x 64 keys
    for (int64_t base = lo; base < hi; base += kBatch * kWaveSize) {
        uint32_t key[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t i = base + u * kWaveSize + lane;
            key[u] = i < hi ? in_key[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (base + u * kWaveSize + lane < hi) atomicAdd(&sh.hist[wave][(key[u] >> shift) & (kBins - 1)], 1u);
    }
    __syncthreads();

    // counts -> start offsets: within a digit the wavefronts follow each other in
    // input order; digits follow each other in value order
    if (threadIdx.x < kBins) {
        uint32_t run = 0;
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t c = sh.hist[w][threadIdx.x];
            sh.hist[w][threadIdx.x] = run;
            run += c;
        }
        sh.digit_base[threadIdx.x] = run;
    }
    __syncthreads();
    if (wave == 0) {
        uint32_t t[kBins / kWaveSize];
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < kBins / kWaveSize; ++i) {
            t[i] = sh.digit_base[lane * (kBins / kWaveSize) + i];
            sum += t[i];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < kWaveSize; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        uint32_t run = incl - sum;
#pragma unroll
        for (int i = 0; i < kBins / kWaveSize; ++i) {
            sh.digit_base[lane * (kBins / kWaveSize) + i] = run;
            run += t[i];
        }
    }
    __syncthreads();

    // scatter in input order; hist[wave][d] is private to this wavefront from here on
    volatile uint32_t* my_off = sh.hist[wave];
    for (int64_t base = lo; base < hi; base += kBatch * kWaveSize) {
        uint32_t keys[kBatch], vals[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t i = base + u * kWaveSize + lane;
            const bool valid = i < hi;
            keys[u] = valid ? in_key[i] : 0u;
            vals[u] = 0u;
            if constexpr (KIND == kIotaIn) vals[u] = (uint32_t)i;
            if constexpr (KIND == kPairs || KIND == kRankOut) vals[u] = valid ? in_val[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (base + u * kWaveSize >= hi) break;              // same for all lanes of the wavefront
            const bool valid = base + u * kWaveSize + lane < hi;
            const uint32_t key = keys[u], val = vals[u];
            const uint32_t d = (key >> shift) & (kBins - 1);
            uint64_t same = __ballot(valid);                    // lanes holding my digit
#pragma unroll
            for (int b = 0; b < kRadixBits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t has = __ballot(bit);
                same &= bit ? has : ~has;
            }
            const uint32_t before = lanes_below(same);          // same-digit lanes ahead of me
            const uint32_t count = (uint32_t)__popcll(same);
            const uint32_t off = my_off[d];
            const uint32_t pos = sh.digit_base[d] + off + before;
            if (valid && pos < n && val < n) {                  // counts add up to n, so this always holds
                if constexpr (KIND == kRankOut) {
                    out_val[val] = (uint32_t)(n - 1) - pos;
                } else {
                    out_key[pos] = key;
                    if constexpr (KIND != kKeysOnly) out_val[pos] = val;
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (valid && before + 1 == count) my_off[d] = off + count;   // last lane of the digit advances it
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
}

// ---- ranking by value ranges ------------------------------------------------------------------
constexpr int kBinBits = 12;
constexpr int kRankBins = 1 << kBinBits;             // 4 per lane
static_assert(kRankBins == 4 * kSortLanes, "prefix sums take four bins per lane");
constexpr uint32_t kLongHead = 1 << 17;              // keys from which the counters of the bins have copies
constexpr int kDppWaveShl1 = 0x130;                  // lane i <- lane i + 1; the last lane keeps its own
constexpr uint32_t kMaxFine = 64;                    // elements of a finer bin that are compared with each other

constexpr int kFinePer = 8;                          // finer bins per lane
constexpr int kFineBins = kFinePer * kSortLanes;

struct __attribute__((aligned(16))) BinShared {
    uint32_t bin[kRankBins + 4];                     // of the head; one word more than bins
    uint32_t fine[kFineBins];                        // of the share
    uint32_t wave[2][kSortWaves];
    uint32_t first, end, base, stop, crowded;
};

// A workgroup's part of a head: `share` of `shares`.
struct Part { int64_t head; int share; };

// Workgroups go to the 8 compute dies round-robin.  With a multiple of 8 heads, the shares of a
// head are 8 apart, so that the keys of a head are read through one die's L2 and the ranks, which
// are scattered over the whole head, meet in it.  Otherwise head and share in plain order.
__device__ __forceinline__ Part part_of_block(uint32_t block, uint32_t n_heads, uint32_t shares) {
    if (n_heads % 8 == 0) {
        const uint32_t y = block / 8;
        return Part{(int64_t)(y / shares) * 8 + block % 8, (int)(y % shares)};
    }
    return Part{block / shares, (int)(block % shares)};
}

// How n elements are cut into shares: the first `rest` of them take one more than n / shares.
struct Cut {
    uint32_t shares, quotient, rest;
    __host__ __device__ Cut(uint32_t n, uint32_t count) : shares(count), quotient(n / count), rest(n % count) {}
    __device__ __forceinline__ uint32_t start(uint32_t s) const { return s * quotient + (s < rest ? s : rest); }
};

// Bins of a range of keys, monotone in the key.  Norms spread over octaves: equal widths in their bit
// patterns (about the logarithm).  Logits lie on both sides of zero: equal widths in the value.  (One fused
// multiply-add is monotone whatever its rounding, and the clamp keeps every input inside; NaN goes to bin 0.)
struct BitBins {
    using Key = uint32_t;
    static constexpr uint32_t kLowest = 0u, kHighest = 0xffffffffu;
    uint32_t lo;
    int shift;
    static __device__ __forceinline__ uint32_t key(uint32_t bits) { return bits; }
    static __device__ __forceinline__ uint32_t lower(uint32_t a, uint32_t b) { return a < b ? a : b; }
    static __device__ __forceinline__ uint32_t higher(uint32_t a, uint32_t b) { return a > b ? a : b; }
    static __device__ __forceinline__ int width_shift(uint32_t span) {
        const int bits = span == 0 ? 0 : 32 - __builtin_clz(span);
        return bits > kBinBits ? bits - kBinBits : 0;
    }
    static __device__ __forceinline__ BitBins over(uint32_t kmin, uint32_t kmax) { return BitBins{kmin, width_shift(kmax - kmin)}; }
    __device__ __forceinline__ uint32_t operator()(uint32_t key) const { return (key - lo) >> shift; }
    // how far into its bin `b` a key lies, 0 .. 1
    __device__ __forceinline__ float within(uint32_t key, uint32_t b) const {
        return __builtin_ldexpf((float)(key - lo - (b << shift)), -shift);
    }
};
struct ValueBins {
    using Key = float;
    static constexpr float kLowest = -INFINITY, kHighest = INFINITY;
    float offset, scale;
    static __device__ __forceinline__ float key(uint32_t bits) { return __builtin_bit_cast(float, bits); }
    static __device__ __forceinline__ float lower(float a, float b) { return fminf(a, b); }
    static __device__ __forceinline__ float higher(float a, float b) { return fmaxf(a, b); }
    static __device__ __forceinline__ ValueBins over(float kmin, float kmax) {
        const float scale = (float)kRankBins / (kmax - kmin);
        return ValueBins{-kmin * scale, scale};
    }
    static constexpr float kTop = (float)kRankBins - 0x1p-12f;       // the largest below the number of bins
    __device__ __forceinline__ float position(float key) const { return __builtin_amdgcn_fmed3f(fmaf(key, scale, offset), 0.f, kTop); }
    __device__ __forceinline__ uint32_t operator()(float key) const { return (uint32_t)position(key); }
    __device__ __forceinline__ float within(float key, uint32_t) const { return __builtin_amdgcn_fractf(position(key)); }
};
// Bit patterns that order like the floats (other than NaN) they are made from, for the counting passes.
__device__ __forceinline__ uint32_t ordered_bits(uint32_t bits) { return bits ^ ((int32_t)bits < 0 ? 0xffffffffu : 0x80000000u); }
__device__ __forceinline__ float float_of_ordered(uint32_t v) {
    return __builtin_bit_cast(float, v ^ ((int32_t)v < 0 ? 0x80000000u : 0xffffffffu));
}

// The keys of a head: E > 0: at most 1024 * E, kept in registers; E == 0: re-read in every pass.
template <int E, typename B> struct HeadKeys {
    using Bins = B;
    using Key = typename B::Key;
    static constexpr bool kReread = E == 0;
    const uint32_t* src;
    uint32_t n;
    Key reg[E > 0 ? E : 1];
    __device__ __forceinline__ HeadKeys(const uint32_t* s, uint32_t count) : src(s), n(count) {
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t t = e * kSortLanes + threadIdx.x;
                reg[e] = B::key(src[t < n ? t : n - 1]);
            }
        }
    }
    // body(keys, position(u), valid(u)) for batches of keys, called by all lanes of the workgroup alike
    template <typename F> __device__ __forceinline__ void each_batch(F&& body) const {
        if constexpr (E > 0) {
            uint32_t left = n - threadIdx.x;
            asm volatile("" : "+v"(left));
            body(reg, [](int u) { return (uint32_t)(u * kSortLanes) + threadIdx.x; }, [&](int u) { return (int32_t)left > u * kSortLanes; });
        } else {
            for (uint32_t base = 0; base < n; base += kBatch * kSortLanes) {
                Key key[kBatch];
                load_batch(key, base);
                body(key, [&](int u) { return base + u * kSortLanes + threadIdx.x; },
                     [&](int u) { return base + u * kSortLanes + threadIdx.x < n; });
            }
        }
    }
    __device__ __forceinline__ void load_batch(Key (&key)[kBatch], uint32_t base) const {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t t = base + u * kSortLanes + threadIdx.x;
            key[u] = B::key(src[t < n ? t : n - 1]);
        }
    }
    // body(key, position) for every key of the head once
    template <typename F> __device__ __forceinline__ void each(F&& body) const {
        if constexpr (E > 0) {
            uint32_t left = n - threadIdx.x;                          // negative past the end
            asm volatile("" : "+v"(left));                            // the lane masks are not worth keeping between passes
#pragma unroll
            for (int e = 0; e < E; ++e)
                if ((int32_t)left > e * kSortLanes) body(reg[e], (uint32_t)(e * kSortLanes) + threadIdx.x);
        } else {
            for (uint32_t base = 0; base < n; base += kBatch * kSortLanes) {
                Key key[kBatch];
                load_batch(key, base);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const uint32_t t = base + u * kSortLanes + threadIdx.x;
                    if (t < n) body(key[u], t);
                }
            }
        }
    }
};

// Turns kPer counters per lane into the sums of all lower ones, written to `starts`.  One
// barrier inside; the caller's barriers order the counting before and the use after.
template <int kPer> struct Counts {
    uint32_t v[kPer], before;
    __device__ __forceinline__ void load(const uint32_t* counters) {
        const uint4* const mine = reinterpret_cast<const uint4*>(counters) + threadIdx.x * (kPer / 4);
#pragma unroll
        for (int i = 0; i < kPer / 4; ++i) {
            const uint4 q = mine[i];
            v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
        }
    }
};
template <int kPer>
__device__ __forceinline__ void counts_to_starts(Counts<kPer>& c, uint32_t* starts, uint32_t* wave_total) {
    static_assert(kPer % 4 == 0, "16-byte accesses");
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum += c.v[i];
    const uint32_t incl = wave_inclusive_sum(sum);
    if (lane == kWaveSize - 1) wave_total[wave] = incl;
    __syncthreads();
    uint32_t before = incl - sum;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) before += w < wave ? wave_total[w] : 0u;
    c.before = before;
    uint4* const mine = reinterpret_cast<uint4*>(starts) + threadIdx.x * (kPer / 4);
#pragma unroll
    for (int i = 0; i < kPer / 4; ++i) {
        uint4 v;
        v.x = before; before += c.v[4 * i];
        v.y = before; before += c.v[4 * i + 1];
        v.z = before; before += c.v[4 * i + 2];
        v.w = before; before += c.v[4 * i + 3];
        mine[i] = v;
    }
}

template <typename Bins> struct Share {
    typename Bins::Key kmin, kmax;      // over the head
    Bins bins;                          // of the head
    uint32_t first, end;                // bins of this share
    uint32_t base, count;               // rank of its first element, number of elements
    bool crowded;                       // some bin of the head holds more than kMaxBin elements
};

// `work`: room for the counters of the bins, the list's.  Called by all lanes; ends with a barrier.  All shares of a head see the same bins, so they agree
// on kmin, kmax and crowded, and every bin belongs to exactly one of them.  count is at most
// ceil(n / shares) + kMaxBin - 1 unless the head is crowded.  sh.bin then holds the rank of the first
// element of every bin.
template <typename Keys>
__device__ __forceinline__ Share<typename Keys::Bins> find_share(const Keys& keys, uint32_t n, uint32_t s, const Cut& cut,
                                                                 uint32_t* work, BinShared& sh) {
    using Bins = typename Keys::Bins;
    using Key = typename Bins::Key;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    Share<Bins> r;
    Key lo = Bins::kHighest, hi = Bins::kLowest;
    keys.each([&](Key key, uint32_t) {
        lo = Bins::lower(lo, key);
        hi = Bins::higher(hi, key);
    });
#pragma unroll
    for (int off = kWaveSize / 2; off > 0; off >>= 1) {
        lo = Bins::lower(lo, __shfl_xor(lo, off));
        hi = Bins::higher(hi, __shfl_xor(hi, off));
    }
    if (lane == 0) {
        sh.wave[0][wave] = __builtin_bit_cast(uint32_t, lo);
        sh.wave[1][wave] = __builtin_bit_cast(uint32_t, hi);
    }
    // long heads: interleaved counters, which equal keys share (64 heads of 400k norms, 30 % zero: 3.95 ms instead of 4.59);
    // short ones would notice the clearing (8 heads of 4k: 10.3 us instead of 9.4)
    const bool copies = Keys::kReread && n > kLongHead;
    if (copies) clear_counts(work, kRankBins * kCopies);
    else reinterpret_cast<uint4*>(sh.bin)[threadIdx.x] = make_uint4(0, 0, 0, 0);
    if (threadIdx.x == 0) {
        sh.first = sh.base = 0;               // what share 0 starts with
        sh.crowded = 0;
        sh.bin[kRankBins] = n;                // where a bin behind the last would start
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        lo = Bins::lower(lo, __builtin_bit_cast(Key, sh.wave[0][w]));
        hi = Bins::higher(hi, __builtin_bit_cast(Key, sh.wave[1][w]));
    }
    r.kmin = lo;
    r.kmax = hi;
    r.bins = Bins::over(lo, hi);
    if (copies) keys.each([&](Key key, uint32_t) { count_digit(work, r.bins(key)); });
    else keys.each([&](Key key, uint32_t) { atomicAdd(&sh.bin[r.bins(key)], 1u); });
    __syncthreads();
    Counts<4> c;
    if (copies) {
#pragma unroll
        for (int i = 0; i < 4; ++i) c.v[i] = digit_count(work, 4 * threadIdx.x + i);
    } else {
        c.load(sh.bin);
    }
    counts_to_starts(c, sh.bin, sh.wave[0]);
    uint32_t before = c.before;
    // The share starts with the first bin that starts at or past its first rank, i.e. behind the
    // bin that holds the rank before; it stops behind the bin that holds its last rank.
    const uint32_t r0 = cut.start(s), r1 = cut.start(s + 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t after = before + c.v[i];
        if (r0 > 0 && before <= r0 - 1 && r0 - 1 < after) {
            sh.first = 4 * threadIdx.x + i + 1;
            sh.base = after;
        }
        if (r1 > 0 && before <= r1 - 1 && r1 - 1 < after) {
            sh.end = 4 * threadIdx.x + i + 1;
            sh.stop = after;
        }
        if (c.v[i] > kMaxBin) sh.crowded = 1;
        before = after;
    }
    if (r1 == 0 && threadIdx.x == 0) sh.end = sh.stop = 0;       // no rank falls to it
    __syncthreads();
    r.first = sh.first;
    r.end = sh.end;
    r.base = sh.base;
    r.count = sh.stop - sh.base;
    r.crowded = sh.crowded != 0;
    return r;
}

// The elements of a share (at most kPer per lane), each with its rank inside the share: key[u], pos[u]
// and rank[u] where u * 1024 + lane < count.  One pass over the head gathers them into the list.  They are then
// counted in finer bins, put into the order of those, and every element compares itself with the others
// of its bin.  A finer bin is a range of expected ranks: the rank of the first element of the head's bin
// plus the way into that bin times its elements, so that dense and sparse stretches of values
// fill the finer bins alike (8192 bins for up to 20k elements).  With finer bins of equal width the
// tails of the logits left a few hundred elements in each of the others: 140 us for 128 heads in two shares
// against 46.  Hits are gathered with one counter update per wave and batch (a ballot and an update per key:
// 16k cycles of the 48k of a share, now 7k).  Keys and positions lie side by side in the list, so that one LDS access moves both: its
// issue bounds the gather (32 heads of 32k norms 20.7 -> 20.5 us, 20 equal norms each 29.0 -> 28.0; with the lanes that store named by
// ballots 0.7 more).  Equal keys rank by position (kWithPos), else in any order.  Called by all lanes; the
// list is free again after the caller's barrier.
template <typename Bins> struct FineBins {
    const Share<Bins>& s;
    const BinShared& sh;
    const float per_rank;
    __device__ __forceinline__ FineBins(const Share<Bins>& share, const BinShared& shared)
        : s(share), sh(shared), per_rank((float)kFineBins / (float)(share.count > 0 ? share.count : 1)) {}
    __device__ __forceinline__ uint32_t operator()(typename Bins::Key key) const {
        const uint32_t b = s.bins(key);
        const uint32_t start = sh.bin[b], next = sh.bin[b + 1];
        const float expected = fmaf(s.bins.within(key, b), (float)(next - start), (float)(start - s.base));
        return (uint32_t)fminf(expected * per_rank, (float)(kFineBins - 1));
    }
};
template <int kPer, typename Bins> struct Ranked {
    typename Bins::Key key[kPer];
    uint32_t pos[kPer], rank[kPer];
};
template <bool kWithPos, int kPer, typename Keys>
__device__ __forceinline__ bool rank_share(const Keys& keys, const Share<typename Keys::Bins>& s, BinShared& sh,
                                           typename Keys::Key* list,
                                           Ranked<kPer, typename Keys::Bins>& out) {
    using Key = typename Keys::Key;
    const auto put = [&](uint32_t at, Key key, uint32_t pos) {
        if constexpr (kWithPos) reinterpret_cast<uint2*>(list)[at] = make_uint2(key, pos);
        else list[at] = key;
    };
    const auto get = [&](uint32_t at, Key& key, uint32_t& pos) {
        if constexpr (kWithPos) {
            const uint2 both = reinterpret_cast<const uint2*>(list)[at];
            key = both.x;
            pos = both.y;
        } else {
            key = list[at];
            pos = at;                                                 // ties in the order of the list
        }
    };
    const uint32_t bins = s.end - s.first;
    typename Keys::Bins coarse = s.bins;
    if constexpr (std::is_same_v<Key, float>) asm volatile("" : "+v"(coarse.scale));   // computed afresh: the bins of
    else asm volatile("" : "+v"(coarse.lo));                                           // the count would not stay in registers
    if (threadIdx.x == 0) sh.wave[1][0] = 0;                          // elements gathered
    for (int i = 0; i < kFinePer / 4; ++i) reinterpret_cast<uint4*>(sh.fine)[i * kSortLanes + threadIdx.x] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    keys.each_batch([&](const auto& key, auto pos, auto valid) {
        constexpr int kN = sizeof(key) / sizeof(key[0]);
        // this lane's hits as a bit mask, one counter update per wave
        uint32_t hits = 0;
#pragma unroll
        for (int u = 0; u < kN; ++u) hits |= valid(u) && coarse(key[u]) - s.first < bins ? 1u << u : 0u;
        const uint32_t incl = wave_inclusive_sum(__popc(hits));
        uint32_t at = 0;
        if (threadIdx.x % kWaveSize == kWaveSize - 1) at = atomicAdd(&sh.wave[1][0], incl) + incl;
        at = __shfl(at, kWaveSize - 1) - __shfl(incl, kWaveSize - 1) + incl - __popc(hits);
#pragma unroll
        for (int u = 0; u < kN; ++u) {
            if (hits >> u & 1u) {
                put(at++, key[u], pos(u));
            }
        }
    });
    __syncthreads();
    const FineBins<typename Keys::Bins> fine_bin(s, sh);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t i = u * kSortLanes + threadIdx.x;
        if (i < s.count) {
            get(i, out.key[u], out.pos[u]);
            out.rank[u] = fine_bin(out.key[u]);
            atomicAdd(&sh.fine[out.rank[u]], 1u);
        }
    }
    __syncthreads();
    Counts<kFinePer> c;
    c.load(sh.fine);
    counts_to_starts(c, sh.fine, sh.wave[0]);
#pragma unroll
    for (int i = 0; i < kFinePer; ++i)
        if (c.v[i] > kMaxFine) sh.crowded = 1;                        // 0 so far: the head is not crowded
    __syncthreads();
    if (sh.crowded != 0) return false;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (u * kSortLanes + threadIdx.x < s.count) {
            put(atomicAdd(&sh.fine[out.rank[u]], 1u), out.key[u], out.pos[u]);
        }
    }
    __syncthreads();
    // A bin now ends at its counter and starts where the bin before it ends.  The lanes take the elements
    // in the order of the bins, so that a large bin keeps few waves busy, four at a time and the
    // first kListAhead elements of their bins at once, so that the LDS round trips overlap; longer
    // bins go on in steps of as many.  (The list has room for kListAhead words behind any share.)
    constexpr int kTogether = 4;
    uint32_t lane_of_all = threadIdx.x;
    asm volatile("" : "+v"(lane_of_all));                             // the positions of the passes above are not worth registers
#pragma unroll
    for (int u0 = 0; u0 < kPer; u0 += kTogether) {
        if (u0 * kSortLanes >= (int)s.count) break;
        uint32_t start[kTogether], end[kTogether];
#pragma unroll
        for (int v = 0; v < kTogether && u0 + v < kPer; ++v) {
            const uint32_t i = (u0 + v) * kSortLanes + lane_of_all;
            const uint32_t at = i < s.count ? i : 0u;
            get(at, out.key[u0 + v], out.pos[u0 + v]);
        }
#pragma unroll
        for (int v = 0; v < kTogether && u0 + v < kPer; ++v) {
            const uint32_t f = fine_bin(out.key[u0 + v]);
            start[v] = f > 0 ? sh.fine[f - 1] : 0u;
            end[v] = sh.fine[f];
        }
        Key other[kTogether][kListAhead];
        uint32_t order[kTogether][kListAhead];
#pragma unroll
        for (int v = 0; v < kTogether && u0 + v < kPer; ++v) {
#pragma unroll
            for (int j = 0; j < kListAhead; ++j) get(start[v] + j, other[v][j], order[v][j]);
        }
#pragma unroll
        for (int v = 0; v < kTogether && u0 + v < kPer; ++v) {
            const Key key = out.key[u0 + v];
            const uint32_t pos = out.pos[u0 + v];
            uint32_t r = start[v];
#pragma unroll
            for (int j = 0; j < kListAhead; ++j)
                r += start[v] + j < end[v] && (other[v][j] < key || (other[v][j] == key && order[v][j] < pos)) ? 1u : 0u;
            for (uint32_t j0 = start[v] + kListAhead; j0 < end[v]; j0 += kListAhead) {
                Key o[kListAhead];
                uint32_t p[kListAhead];
#pragma unroll
                for (int j = 0; j < kListAhead; ++j) get(j0 + j, o[j], p[j]);
#pragma unroll
                for (int j = 0; j < kListAhead; ++j) r += j0 + j < end[v] && (o[j] < key || (o[j] == key && p[j] < pos)) ? 1u : 0u;
            }
            out.rank[u0 + v] = r;
        }
    }
    return true;
}

// ---- the elements of a share in order, straight from registers ----------------------------------
// For logits, whose positions do not matter, while the keys of the head stay in registers.  All keys of the head are counted once, in bins
// so fine that a few share one (ScoreBins); the number the counter returns is a key's place in its bin, so that, once the bins have their
// starts, one more store puts the keys of the share in order of the bins, and nothing is gathered or read again.  What is then left
// to do is order inside the bins: a lane sorts 32 neighbours in registers, which does every bin that does not reach over their end, and
// merges the upper half of them with the lower half of the next lane's, which does the others, as long as
// no bin has more than 17 (fuller ones are put in order by themselves, sort_full_bins).  The lane then holds 32 elements of consecutive
// ranks and adds them up.
// What bounds it: a key costs 0.2 us per vector instruction and CU (32 keys a lane, four waves a SIMD), and each of its LDS
// accesses 10 to 20 cycles a wave with its bank conflicts; so a key's way takes a dozen and a half instructions, one atomic and two
// accesses, all lanes doing the same.  128 heads of 32k logits in two shares each, us by stamps in the kernel, without its launch: fetch and range 6.9, position sums 1.2, bins 4.7,
// starts 2.1, scatter 3.4, sort 1.4, merge and sums 3.5, records 2.6: 26 in place of 30.5 with the keys counted in 4096 bins of equal width
// (5.7) and again in 8192 of the share (7.4 with their starts).  Both launches, with the logits, 74.9 -> 71.7, 32 heads of 9000 23.4 -> 21.5.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kTogetherKeys = 4;                     // keys whose LDS round trips overlap (8: the same time)
constexpr int kRun = 32;                             // elements a lane sorts
constexpr uint32_t kMaxRun = kRun / 2 + 1;           // of one bin
constexpr uint32_t kListFront = kRun / 2;            // words of the list in front of the first element

template <int kN, int kSpan, int kStep> __device__ __forceinline__ void merge_step(float (&x)[kN]) {
#pragma unroll
    for (int j = kStep % kSpan; j + kStep < kN; j += 2 * kStep) {
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
            const int a = i + j, b = a + kStep;
            if (b < kN && a / (2 * kSpan) == b / (2 * kSpan)) {
                const float lo = fminf(x[a], x[b]), hi = fmaxf(x[a], x[b]);
                x[a] = lo;
                x[b] = hi;
            }
        }
    }
    if constexpr (kStep > 1) merge_step<kN, kSpan, kStep / 2>(x);
}
// Sorted runs of kSpan become one of kN: Batcher's odd-even merge sort.
template <int kN, int kSpan> __device__ __forceinline__ void merge_runs(float (&x)[kN]) {
    merge_step<kN, kSpan, kSpan>(x);
    if constexpr (2 * kSpan < kN) merge_runs<kN, 2 * kSpan>(x);
}

// Word of the list for an element: 16-byte pieces of the 32 words of a lane in an order that depends on the lane, so
// that lanes reading the same piece of theirs hit different banks.
__device__ __forceinline__ uint32_t run_word(uint32_t at) { return at ^ ((at >> 5 & 7u) << 2); }

__device__ __forceinline__ float read_lane(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Bins with more elements than the runs take care of: every element finds its place by comparing itself with all others of the bin, a
// wave to a bin, four from 129 elements on (one bin of 200 among 9000 logits 33 us by one wave).  Bins of equal elements, as copies of a row
// make them, are left as they are.
constexpr uint32_t kMaxOfBin = 512;                  // fuller ones: exact cut
struct FullBin {                                     // in one word
    uint32_t word;
    static __device__ __forceinline__ FullBin of(uint32_t start, uint32_t count) { return FullBin{start | count << 16}; }
    __device__ __forceinline__ uint32_t start() const { return word & 0xffffu; }
    __device__ __forceinline__ uint32_t count() const { return word >> 16; }
};
// A lane's elements lane + 64 * (part + kWaves * k) of a bin, and their places in it; without elements: nothing.
template <uint32_t kWaves, uint32_t kPer> struct PlacedElements {
    float x[kPer];
    uint32_t first, place[kPer];
    FullBin bin;
    __device__ __forceinline__ PlacedElements(FullBin b, uint32_t part, const float* list) : first(part * kWaveSize + threadIdx.x % kWaveSize), bin(b) {
        const uint32_t n = bin.count(), lane = threadIdx.x % kWaveSize;
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) {
            const uint32_t i = first + k * kWaves * kWaveSize;
            x[k] = list[run_word(bin.start() + (i < n ? i : 0u))];
            place[k] = 0;
        }
        for (uint32_t base = 0; base < n; base += kWaveSize) {
            const float others = list[run_word(bin.start() + (base + lane < n ? base + lane : 0u))];
            const uint32_t end = n - base < kWaveSize ? n - base : kWaveSize;
            constexpr uint32_t kTogether = 8;
            for (uint32_t j0 = 0; j0 < end; j0 += kTogether) {
#pragma unroll
                for (uint32_t u = 0; u < kTogether; ++u) {
                    const uint32_t j = j0 + u;                        // below 64
                    const float other = read_lane(others, (int)j);    // equal ones in the order in which they stand; no branches
#pragma unroll
                    for (uint32_t k = 0; k < kPer; ++k)
                        place[k] += (((other < x[k]) | ((other == x[k]) & (base + j < first + k * kWaves * kWaveSize))) & (j < end)) ? 1u : 0u;
                }
            }
        }
    }
    __device__ __forceinline__ void store(float* list) const {
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k)
            if (first + k * kWaves * kWaveSize < bin.count()) list[run_word(bin.start() + place[k])] = x[k];
    }
};
struct FullBins { uint32_t listed, few, many; };     // bins in the list; of them, bins whose elements differ, up to 128 and more of them
// `list_end` words in all: the listed bins, behind them those of few differing elements, from the end downwards those of many.
__device__ __forceinline__ void sort_full_bins(uint32_t* bins, uint32_t list_end, FullBins& found, float* list) {
    constexpr uint32_t kAtOnce = kWaveSize / kRowLanes;               // bins that a wave looks over together
    constexpr uint32_t kWavesOfMany = 4;
    const uint32_t lane = threadIdx.x % kWaveSize, c = lane % kRowLanes, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const uint32_t count = __builtin_amdgcn_readfirstlane(found.listed);
    for (uint32_t i0 = wave * kAtOnce; i0 < count; i0 += kSortWaves * kAtOnce) {
        const uint32_t i = i0 + lane / kRowLanes;
        const FullBin bin{bins[i < count ? i : count - 1]};
        const float first = list[run_word(bin.start())];
        bool differ = false;
        for (uint32_t j = c; j < bin.count(); j += kRowLanes) differ |= list[run_word(bin.start() + j)] != first;
        const uint64_t group = 0xffffull << (lane / kRowLanes * kRowLanes);
        if ((__ballot(differ) & group) != 0 && c == 0 && i < count) {
            if (bin.count() <= 2 * kWaveSize) bins[count + atomicAdd(&found.few, 1u)] = bin.word;
            else bins[list_end - 1 - atomicAdd(&found.many, 1u)] = bin.word;
        }
    }
    __syncthreads();
    auto record = [&](uint32_t at) { return FullBin{(uint32_t)__builtin_amdgcn_readfirstlane((int)bins[at])}; };
    const uint32_t few = __builtin_amdgcn_readfirstlane(found.few), many = __builtin_amdgcn_readfirstlane(found.many);
    for (uint32_t i = wave; i < few; i += kSortWaves) {
        const FullBin bin = record(count + i);
        if (bin.count() <= kWaveSize) PlacedElements<1, 1>(bin, 0, list).store(list);
        else PlacedElements<1, 2>(bin, 0, list).store(list);
    }
    for (uint32_t i0 = 0; i0 < many; i0 += kSortWaves / kWavesOfMany) {
        const uint32_t i = i0 + wave / kWavesOfMany;
        const FullBin bin = i < many ? record(list_end - 1 - i) : FullBin{0};
        const PlacedElements<kWavesOfMany, kMaxOfBin / kWaveSize / kWavesOfMany> mine(bin, wave % kWavesOfMany, list);
        __syncthreads();                                              // all waves of a bin have read it
        mine.store(list);
    }
    __syncthreads();
}

// Bins of the logits of a head, monotone in the logit: equal widths in the bit pattern of the distance from the mean plus an
// offset, below the mean and above it alike; 2048 bins to an octave for the first four octaves, 1024 for the fifth and 256 from there on.
// So they are of one width near the mean, where the logits lie densely, and grow with the distance where they thin out: 32k logits
// of normal or log-normally scaled rows put 3 elements into a bin on average over the elements and 15 into the fullest, where as many
// bins of equal width hold 200 of the latter.  (Sums and shifts of rounded floats are monotone whatever their rounding.)
struct ScoreRange { float lo, hi, mean, deviation; };
struct ScoreBins {
    static constexpr uint32_t kHalf = 4u * 10240u;                    // bytes of the counters on one side of the mean
    static constexpr uint32_t kFourth = 4u * 8192u, kFifth = 4u * (8u * 9216u - 10240u);     // where the lines of 1024 and 256 to an octave meet zero
    float mean, offset;
    uint32_t origin;
    // The offset: a 56th of the largest distance, which is 5 octaves and a bit; where a few logits lie so far out that this is wide for
    // the others, 0.3 standard deviations, but no less than the nine octaves that there is room for reach.
    __device__ __forceinline__ explicit ScoreBins(const ScoreRange& r) : mean(r.mean) {
        const float far = fmaxf(r.hi - r.mean, r.mean - r.lo);
        offset = fminf(far * (1.f / 56.f), fmaxf(far * (1.f / 511.f), 0.3f * r.deviation));
        origin = __builtin_bit_cast(uint32_t, offset);
    }
    // byte offset of the counter of a logit
    __device__ __forceinline__ uint32_t operator()(float logit) const {
        const float x = logit - mean;
        const uint32_t d = (__builtin_bit_cast(uint32_t, fabsf(x) + offset) - origin) >> 10;
        const uint32_t away = min(min(min(d, (d + kFourth) >> 1), (d + kFifth) >> 3), kHalf - 1);    // the last for what is not a number
        const uint32_t side = (uint32_t)(__builtin_bit_cast(int32_t, x) >> 31);
        return ((away ^ side) + kHalf) & ~3u;                         // below the mean: kHalf - 1 - away
    }
};
constexpr int kScoreBinsPer = 20;                    // per lane
constexpr uint32_t kScoreBins = kScoreBinsPer * kSortLanes;
static_assert(ScoreBins::kHalf * 2 == kScoreBins * 4, "a counter per bin");
constexpr uint32_t kRunWords = (kListFront + kLongestShare + kMaxOfBin + 31) / 32 * 32;      // a share, and what its last bin brings with it
static_assert(kRunWords >= kListFront + kLongestShare + kMaxOfBin && kLongestShare + kMaxOfBin <= kRun * kSortLanes - kRun, "room for the scatter, lanes for the runs");
struct RunBins {
    uint32_t bin[kScoreBins + 4];                    // one word more than bins
    uint32_t aside[kWaveSize];                       // a word per lane for positions past the end
};
struct RunShared {
    float lo[kSortWaves], hi[kSortWaves], sum[kSortWaves], squares[kSortWaves];
    uint32_t wave[kSortWaves];
    uint32_t base, stop, crowded, full;
    FullBins bins;
};

template <typename Op> __device__ __forceinline__ float row16_all(float v, Op op) {
    v = op(v, dpp_read<kDppXor1>(v));
    v = op(v, dpp_read<kDppXor2>(v));
    v = op(v, dpp_read<kDppHalfMirror>(v));
    return op(v, dpp_read<kDppMirror>(v));
}
template <typename Op> __device__ __forceinline__ float wave_all(float v, Op op) {
    v = row16_all(v, op);
    return op(op(read_lane(v, 0), read_lane(v, 16)), op(read_lane(v, 32), read_lane(v, 48)));
}

// Least and largest logit of the head, their mean and standard deviation, the same in all lanes and shares.  Called by all lanes; one barrier.
template <int E>
__device__ __forceinline__ ScoreRange score_range(const HeadKeys<E, ValueBins>& keys, RunShared& sh) {
    auto least = [](float a, float b) { return fminf(a, b); };
    auto most = [](float a, float b) { return fmaxf(a, b); };
    auto plus = [](float a, float b) { return a + b; };
    float lo = INFINITY, hi = -INFINITY, sum = 0.f, squares = 0.f;
    keys.each([&](float key, uint32_t) {
        lo = least(lo, key);
        hi = most(hi, key);
        sum += key;
        squares = fmaf(key, key, squares);
    });
    lo = wave_all(lo, least);
    hi = wave_all(hi, most);
    sum = wave_all(sum, plus);
    squares = wave_all(squares, plus);
    const uint32_t wave = threadIdx.x / kWaveSize;
    if (threadIdx.x % kWaveSize == 0) {
        sh.lo[wave] = lo;
        sh.hi[wave] = hi;
        sh.sum[wave] = sum;
        sh.squares[wave] = squares;
    }
    if (threadIdx.x == 0) {
        sh.crowded = sh.full = sh.base = sh.stop = 0;
        sh.bins = FullBins{0, 0, 0};
    }
    __syncthreads();
    static_assert(kSortWaves == kRowLanes, "a wave's value per lane of a DPP row");
    const uint32_t i = threadIdx.x % kRowLanes;
    auto uniform = [](float v) { return read_lane(v, 0); };
    const float mean = uniform(row16_all(sh.sum[i], plus)) / (float)keys.n, square = uniform(row16_all(sh.squares[i], plus)) / (float)keys.n;
    return ScoreRange{uniform(row16_all(sh.lo[i], least)), uniform(row16_all(sh.hi[i], most)), mean,
                      sqrtf(fmaxf(square - mean * mean, 0.f))};
}

// True: run[] holds the elements of ranks base + kRun * threadIdx.x .., as far as they are among the `count` of the share: the bins
// that start inside its range of ranks.  False, where some bin of the head holds more than kMaxOfBin elements: nothing (all shares alike).
// The bins are cleared.  Called by all lanes; the list is free again after the caller's barrier.
template <int E>
__device__ __forceinline__ bool order_share(const HeadKeys<E, ValueBins>& keys, const ScoreRange& range, uint32_t share, const Cut& cut,
                                            RunBins& rb, RunShared& sh, float* list, float (&run)[kRun], uint32_t& base, uint32_t& count) {
    const uint32_t lane = threadIdx.x % kWaveSize;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const ScoreBins bin_of(range);
    // One pass for all: the number that the counter returns is the key's place in its bin.
    uint32_t place[E];
    uint32_t left = keys.n - threadIdx.x;                             // negative past the end
    asm volatile("" : "+v"(left));
    constexpr uint32_t kAsideAt = (kScoreBins + 4) * 4, kPlaceShift = 17;
    static_assert(kAsideAt + 4 * kWaveSize <= 1 << kPlaceShift && E * kSortLanes <= 1 << (32 - kPlaceShift), "counter and place in one word");
#pragma unroll
    for (int e0 = 0; e0 < E; e0 += kTogetherKeys) {
#pragma unroll
        for (int u = 0; u < kTogetherKeys; ++u) {
            const uint32_t b = bin_of(keys.reg[e0 + u]);
            place[e0 + u] = (int32_t)left > (e0 + u) * kSortLanes ? b : kAsideAt + 4 * lane;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kTogetherKeys; ++u) {
            uint32_t* const counter = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(rb.bin) + place[e0 + u]);
            place[e0 + u] |= atomicAdd(counter, 1u) << kPlaceShift;
        }
#pragma unroll
        for (int u = 0; u < kTogetherKeys; ++u) asm volatile("" : "+v"(place[e0 + u]));       // one register each, not two
    }
    __syncthreads();
    {
        Counts<kScoreBinsPer> c;
        c.load(rb.bin);
        counts_to_starts(c, rb.bin, sh.wave);
        if (threadIdx.x < kWaveSize) rb.aside[threadIdx.x] = 1u << 31;         // in no share
        if (threadIdx.x == 0) rb.bin[kScoreBins] = keys.n;
        // The share starts behind the bin that holds the rank before its first, and stops behind the bin that holds its last.
        const uint32_t r0 = cut.start(share), r1 = cut.start(share + 1);
        uint32_t before = c.before, sum = 0, fullest = 0;
#pragma unroll
        for (int i = 0; i < kScoreBinsPer; ++i) {
            sum += c.v[i];
            fullest = c.v[i] > fullest ? c.v[i] : fullest;
        }
        if (r0 - 1 - before < sum || r1 - 1 - before < sum) {         // r0 == 0: no bin
#pragma unroll
            for (int i = 0; i < kScoreBinsPer; ++i) {
                const uint32_t after = before + c.v[i];
                if (r0 - 1 - before < c.v[i]) sh.base = after;
                if (r1 - 1 - before < c.v[i]) sh.stop = after;
                before = after;
            }
        }
        if (fullest > kMaxRun) {
            sh.full = 1;
            if (fullest > kMaxOfBin) sh.crowded = 1;
        }
    }
    __syncthreads();
    if (sh.crowded != 0) return false;
    base = __builtin_amdgcn_readfirstlane(sh.base);
    count = __builtin_amdgcn_readfirstlane(sh.stop) - base;
    const uint32_t full = __builtin_amdgcn_readfirstlane(sh.full);
    constexpr uint32_t kAside = kRunWords;                            // behind the longest share
#pragma unroll
    for (int e = 0; e < E; ++e) {
        constexpr uint32_t kCounter = (1u << kPlaceShift) - 1;
        const uint32_t start = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(rb.bin) + (place[e] & kCounter));
        const uint32_t at = start + (place[e] >> kPlaceShift) - base;
        list[at < count ? run_word(at + kListFront) : kAside + lane] = keys.reg[e];
    }
    if (threadIdx.x < kListFront) list[run_word(threadIdx.x)] = -INFINITY;
    __syncthreads();
    if (__builtin_expect(full != 0, false)) {
        // the starts are not needed any longer: the full bins' records take their place
        static_assert(kRunWords < 1 << 16 && kRunWords / kMaxRun * 2 <= kScoreBins, "a word each, or two, in place of the bins");
        Counts<kScoreBinsPer> starts;
        starts.load(rb.bin);
        const uint32_t behind = rb.bin[(threadIdx.x + 1) * kScoreBinsPer];
        auto elements = [&](int i) {
            const uint32_t n = (i + 1 < kScoreBinsPer ? starts.v[i + 1 < kScoreBinsPer ? i + 1 : 0] : behind) - starts.v[i];
            return n > kMaxRun && starts.v[i] - base < count ? n : 0u;
        };
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < kScoreBinsPer; ++i) mine += elements(i) > 0 ? 1u : 0u;
        const uint32_t incl = wave_inclusive_sum(mine);
        uint32_t slot = 0;
        if (lane == kWaveSize - 1) slot = atomicAdd(&sh.bins.listed, incl);
        slot = (uint32_t)__builtin_amdgcn_readlane((int)slot, kWaveSize - 1) + incl - mine;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kScoreBinsPer; ++i) {
            const uint32_t n = elements(i);
            if (n > 0) rb.bin[slot++] = FullBin::of(starts.v[i] - base + kListFront, n).word;
        }
        __syncthreads();
        sort_full_bins(rb.bin, kScoreBins, sh.bins, list);
    }
    // Lane i: the words 32 i .. 32 i + 31, elements from 16 before its ranks on.
    const uint32_t words = count + kListFront;
    float x[kRun];
    if (wave * (kWaveSize * kRun) < words) {
#pragma unroll
        for (uint32_t q = 0; q < kRun / 4; ++q) {
            const uint32_t at = threadIdx.x * kRun + 4 * q;
            f32x4 v = {INFINITY, INFINITY, INFINITY, INFINITY};
            if (at < words) v = *reinterpret_cast<const f32x4*>(list + run_word(at));
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) x[4 * q + i] = at + i < words ? v[i] : INFINITY;
        }
        merge_runs<kRun, 1>(x);
    } else {
#pragma unroll
        for (int i = 0; i < kRun; ++i) x[i] = INFINITY;
    }
    // the lower half of the next lane's; of the next wave's first lane through LDS
    float* const edge = reinterpret_cast<float*>(rb.bin);
    if (lane == 0) {
#pragma unroll
        for (uint32_t i = 0; i < kRun / 2; ++i) edge[wave * (kRun / 2) + i] = x[i];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kRun / 2; ++i) {
        const float next = wave + 1 < (uint32_t)kSortWaves ? edge[(wave + 1) * (kRun / 2) + i] : INFINITY;
        run[kRun / 2 + i] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, next),
                                                                                 __builtin_bit_cast(int, x[i]), kDppWaveShl1, 0xf, 0xf, false));
        run[i] = x[kRun / 2 + i];
    }
    merge_step<kRun, kRun / 2, kRun / 2>(run);
    return true;
}

// ---- ranking by an exact cut and a sort ---------------------------------------------------------
// For the keys that bins do not separate: tied or clustered ones, and long heads.  The elements of ranks
// [r0, r1) in the order of (key, position), whatever the keys are.  The cuts are found as in the selection, by
// three digits for both at once; the elements between them are gathered in the order of their positions
// and sorted in the list by 8-bit digits of what their keys differ in, every wave a stretch of the list with
// its elements in registers.  Five passes over the head (re-read from the L2) and up to four over the list:
//   32 heads of 32k norms, 30 % zero       174 us by one workgroup's counting passes, 63 here
//   128 heads of 8k norms, 9 values        60 us, 507 by comparing inside the bins, 36 here
//   128 heads of 32k scores, 36 values     266 us, 1500 by comparing inside the bins, 157 here (with the logits)
//   4 heads of 1M norms                    7.4 ms, 1.4 here
struct NormKey {
    static __device__ __forceinline__ uint32_t of(uint32_t bits) { return bits; }
};
struct LogitKey {
    static __device__ __forceinline__ uint32_t of(uint32_t bits) { return ordered_bits(bits); }
};

// The first r elements of a head: the keys below tau and the first `need` keys equal to it.
struct Bound { uint32_t tau, need; };

// Elements x0 .. x0 + count - 1 that lie in [from, to).
__device__ __forceinline__ uint32_t overlap(uint32_t x0, uint32_t count, uint32_t from, uint32_t to) {
    const uint32_t a = x0 > from ? x0 : from, b = x0 + count < to ? x0 + count : to;
    return a < b ? b - a : 0u;
}

struct CutShared {
    FindShared find;
    uint32_t inside[kSortWaves], at_lo[kSortWaves], at_hi[kSortWaves];
};

// Four consecutive keys of a head, which starts at any word.
typedef uint32_t KeyQuad __attribute__((ext_vector_type(4), aligned(4)));

// The elements of ranks [r0, r1) into the list, in the order of their positions; returns the keys they lie between.
// `work`: 16384 words, may be the list's.  Called by all lanes; ends with a barrier.
struct KeyRange { uint32_t least, most; };
template <typename KeyOf, bool kWithPos>
__device__ __forceinline__ KeyRange gather_range(const uint32_t* src, uint32_t n, uint32_t r0, uint32_t r1, uint32_t* work,
                                                 uint32_t* list_key, uint32_t* list_pos, CutShared& cs) {
    const uint32_t lane = threadIdx.x % kWaveSize;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const uint32_t count = r1 - r0;
    // Every wave takes a stretch of consecutive positions, a lane four at a time in one 16-byte load (four of which in
    // flight; single words leave the L2's latency exposed: 64 heads of 262k norms, 30 % zero, 2.71 ms
    // in place of 2.17).
    // body(four keys, position of the first, is_real(j)), by all lanes, in the order of the positions.
    constexpr uint32_t kLoads = 4, kStep = 4 * kWaveSize;
    const uint32_t stretch = (n + kSortWaves * kLoads * kStep - 1) / (kSortWaves * kLoads * kStep) * (kLoads * kStep);
    auto each = [&](auto&& body) {
        const uint32_t first = wave * stretch;
        const uint32_t end = first + stretch < n ? first + stretch : n;
        uint32_t base = first;
        for (; base < end && base + kLoads * kStep <= n; base += kLoads * kStep) {
            uint32_t key[kLoads][4];
#pragma unroll
            for (uint32_t u = 0; u < kLoads; ++u) {
                const KeyQuad q = *reinterpret_cast<const KeyQuad*>(src + base + u * kStep + lane * 4);
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) key[u][j] = q[j];
            }
#pragma unroll
            for (uint32_t u = 0; u < kLoads; ++u) {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) key[u][j] = KeyOf::of(key[u][j]);
                body(key[u], base + u * kStep + lane * 4, [](uint32_t) { return true; });
            }
        }
        for (; base < end; base += kStep) {                           // the last steps of the head
            const uint32_t t = base + lane * 4;
            uint32_t key[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) key[j] = KeyOf::of(src[t + j < n ? t + j : n - 1]);
            body(key, t, [&](uint32_t j) { return t + j < n; });
        }
    };

    // the key of rank r0, and that of rank r1 (or the largest, all of which then are inside)
    uint32_t want_lo = r0 + 1, want_hi = r1 < n ? r1 + 1 : n;
    clear_counts(work, kTopBins * kCopies);
    __syncthreads();
    each([&](const uint32_t (&key)[4], uint32_t, auto is_real) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            if (is_real(j)) count_digit(work, key[j] >> (32 - kTopBits));
    });
    __syncthreads();
    Found a = find_digit<kTopBins>(work, want_lo, cs.find);
    Found b = find_digit<kTopBins>(work, want_hi, cs.find);
    Bound lo{a.digit, want_lo - a.below}, hi{b.digit, want_hi - b.below};
    static_assert(kMidBits == kLowBits, "two digits of one size");
    uint32_t* const count_lo = work;
    uint32_t* const count_hi = work + kMidBins * kCopies;
#pragma unroll
    for (int shift = kLowBits; shift >= 0; shift -= kLowBits) {
        clear_counts(work, 2 * kMidBins * kCopies);
        __syncthreads();
        each([&](const uint32_t (&key)[4], uint32_t, auto is_real) {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t in_lo = (key[j] >> shift) - (lo.tau << kMidBits), in_hi = (key[j] >> shift) - (hi.tau << kMidBits);
                if (is_real(j) && in_lo < kMidBins) count_digit(count_lo, in_lo);
                if (is_real(j) && in_hi < kMidBins) count_digit(count_hi, in_hi);
            }
        });
        __syncthreads();
        a = find_digit<kMidBins>(count_lo, lo.need, cs.find);
        b = find_digit<kMidBins>(count_hi, hi.need, cs.find);
        lo = Bound{lo.tau << kMidBits | a.digit, lo.need - a.below};
        hi = Bound{hi.tau << kMidBits | b.digit, hi.need - b.below};
    }
    [[maybe_unused]] const uint32_t lo_count = a.count, hi_count = b.count;      // keys equal to the bounds
    lo.need -= 1;                                                     // the element of rank r0 itself is inside
    hi.need = r1 < n ? hi.need - 1 : 0xffffffffu;

    // of the keys equal to a bound, those inside: positions [lo.need, lo_end) and [0, hi_end) among their equals
    const bool one_key = lo.tau == hi.tau;
    [[maybe_unused]] const uint32_t lo_end = one_key ? hi.need : 0xffffffffu, hi_end = one_key ? 0u : hi.need;
    const uint32_t between = one_key ? 0u : hi.tau - lo.tau - 1;
    auto is_inside = [&](uint32_t key) { return key - (lo.tau + 1) < between; };
    if constexpr (!kWithPos) {
        // equal keys are alike: copies of the bounds, and what lies between them in any order
        const uint32_t equal_lo = one_key ? count : (lo_count - lo.need < count ? lo_count - lo.need : count);
        const uint32_t equal_hi = one_key ? 0u : (r1 < n ? hi.need : hi_count);
        for (uint32_t i = threadIdx.x; i < equal_lo; i += kSortLanes) list_key[i] = lo.tau;
        for (uint32_t i = threadIdx.x; i < equal_hi; i += kSortLanes) list_key[count - 1 - i] = hi.tau;
        if (threadIdx.x == 0) cs.inside[0] = equal_lo;
        __syncthreads();
        each([&](const uint32_t (&key)[4], uint32_t, auto is_real) {
            uint32_t take = 0;
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) take |= is_real(j) && is_inside(key[j]) ? 1u << j : 0u;
            if (__ballot(take != 0) == 0) return;                     // the same for all lanes
            const uint32_t incl = wave_inclusive_sum(__popc(take));
            uint32_t at = 0;
            if (lane == kWaveSize - 1) at = atomicAdd(&cs.inside[0], incl);
            at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWaveSize - 1) + incl - __popc(take);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                if ((take >> j & 1u) && at < count) list_key[at++] = key[j];      // counts add up, so `at` always is
            }
        });
        __syncthreads();
        return KeyRange{lo.tau, hi.tau};
    }
    uint32_t inside = 0, at_lo = 0, at_hi = 0;
    each([&](const uint32_t (&key)[4], uint32_t, auto is_real) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            inside += is_real(j) && is_inside(key[j]) ? 1u : 0u;
            at_lo += is_real(j) && key[j] == lo.tau ? 1u : 0u;
            at_hi += is_real(j) && key[j] == hi.tau ? 1u : 0u;
        }
    });
    inside = wave_inclusive_sum(inside);
    at_lo = wave_inclusive_sum(at_lo);
    at_hi = wave_inclusive_sum(at_hi);
    if (lane == kWaveSize - 1) {
        cs.inside[wave] = inside;
        cs.at_lo[wave] = at_lo;
        cs.at_hi[wave] = at_hi;
    }
    __syncthreads();
    uint32_t out = 0;
    at_lo = at_hi = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)kSortWaves; ++w) {
        if (w < wave) {
            out += cs.inside[w] + overlap(at_lo, cs.at_lo[w], lo.need, lo_end) + overlap(at_hi, cs.at_hi[w], 0u, hi_end);
            at_lo += cs.at_lo[w];
            at_hi += cs.at_hi[w];
        }
    }
    // numbers the set bits of all lanes in order, from `from` on; `from` moves behind the last
    auto numbered = [&](uint32_t bits, uint32_t& from) {
        const uint32_t incl = wave_inclusive_sum(__popc(bits));
        const uint32_t mine = from + incl - __popc(bits);
        from += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWaveSize - 1);
        return mine;
    };
    each([&](const uint32_t (&key)[4], uint32_t t, auto is_real) {
        uint32_t take = 0, is_lo = 0, is_hi = 0;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            take |= is_real(j) && is_inside(key[j]) ? 1u << j : 0u;
            is_lo |= is_real(j) && key[j] == lo.tau ? 1u << j : 0u;
            is_hi |= is_real(j) && key[j] == hi.tau ? 1u << j : 0u;
        }
        if (__ballot((is_lo | is_hi) != 0) != 0) {                    // the same for all lanes
            uint32_t lo_at = numbered(is_lo, at_lo), hi_at = numbered(is_hi, at_hi);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                if (is_lo >> j & 1u) take |= lo_at >= lo.need && lo_at < lo_end ? 1u << j : 0u, ++lo_at;
                if (is_hi >> j & 1u) take |= hi_at < hi_end ? 1u << j : 0u, ++hi_at;
            }
        }
        if (__ballot(take != 0) != 0) {
            uint32_t at = numbered(take, out);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                if ((take >> j & 1u) && at < count) {                 // counts add up, so `at` always is
                    list_key[at] = key[j];
                    if constexpr (kWithPos) list_pos[at] = t + j;
                    ++at;
                }
            }
        }
    });
    __syncthreads();
    return KeyRange{lo.tau, hi.tau};
}

// Sorts the list by key, equal keys in the order in which they stand.  Eight of the bits in which the keys may differ at
// a time.  count <= kPer * 1024.  Called by all lanes; ends with a barrier.
template <bool kWithPos, int kPer, typename Sh>
__device__ __forceinline__ void sort_list(uint32_t* list_key, uint32_t* list_pos, uint32_t count, KeyRange range, Sh& sh) {
    const uint32_t lane = threadIdx.x % kWaveSize;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const uint32_t span = range.most - range.least;
    const int bits = span == 0 ? 0 : 32 - __builtin_clz(span);
    const uint32_t chunk = ((count + kSortWaves - 1) / kSortWaves + kWaveSize - 1) / kWaveSize * kWaveSize;
    const uint32_t first = wave * chunk;                              // of this wave; chunk <= kPer * 64
    const uint32_t mine = first >= count ? 0u : (count - first < chunk ? count - first : chunk);
    static_assert(kSortWaves * kBins <= kFineBins && kBins <= kRankBins && kBins % kWaveSize == 0, "counters fit the bins");
    // of this wave: its elements of every digit so far, read and written for the other lanes to see
    uint32_t* const counts = sh.fine + wave * kBins;
    auto count_of = [&](uint32_t d) { return __hip_atomic_load(counts + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
    auto set_count = [&](uint32_t d, uint32_t v) { __hip_atomic_store(counts + d, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
    for (int shift = 0; shift < bits; shift += kRadixBits) {
        uint32_t key[kPer], pos[kPer], place[(kPer + 1) / 2];          // places below 2^16, two to a word
        for (uint32_t i = lane; i < kBins; i += kWaveSize) set_count(i, 0u);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t i = u * kWaveSize + lane;
            key[u] = list_key[first + (i < mine ? i : 0u)];
            pos[u] = kWithPos ? list_pos[first + (i < mine ? i : 0u)] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if ((uint32_t)(u * kWaveSize) >= mine) break;             // same for all lanes of the wave
            const bool valid = u * kWaveSize + lane < mine;
            const uint32_t d = (key[u] - range.least) >> shift & (kBins - 1);
            uint64_t same = __ballot(valid);                          // lanes holding my digit
#pragma unroll
            for (int bit = 0; bit < kRadixBits; ++bit) {
                const bool set = d >> bit & 1u;
                const uint64_t has = __ballot(set);
                same &= set ? has : ~has;
            }
            const uint32_t before = lanes_below(same), together = (uint32_t)__popcll(same);
            const uint32_t so_far = count_of(d);
            if (u % 2 == 0) place[u / 2] = so_far + before;
            else place[u / 2] |= (so_far + before) << 16;
            __builtin_amdgcn_wave_barrier();
            if (valid && before + 1 == together) set_count(d, so_far + together);    // last lane of the digit
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // digits follow each other in value order, the waves of a digit in the order of the list
        if (threadIdx.x < kBins) {
            uint32_t run = 0;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = sh.fine[w * kBins + threadIdx.x];
                sh.fine[w * kBins + threadIdx.x] = run;
                run += c;
            }
            const uint32_t incl = wave_inclusive_sum(run);
            sh.bin[threadIdx.x] = incl - run;
            if (lane == kWaveSize - 1) sh.wave[0][wave] = incl;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (u % 4 == 0) __builtin_amdgcn_sched_barrier(0);        // not the reads of all steps at once: the registers are full
            if (u * kWaveSize + lane < mine) {
                const uint32_t d = (key[u] - range.least) >> shift & (kBins - 1);
                uint32_t at = sh.bin[d] + count_of(d) + (place[u / 2] >> (u % 2 * 16) & 0xffffu);
#pragma unroll
                for (uint32_t w = 0; w + 1 < (uint32_t)(kBins / kWaveSize); ++w) at += w < d / kWaveSize ? sh.wave[0][w] : 0u;
                if (at < count) {
                    list_key[at] = key[u];
                    if constexpr (kWithPos) list_pos[at] = pos[u];
                }
            }
        }
        __syncthreads();
    }
}

// All elements of a head that fits the list, in order (8 heads of 4k, 30 % zero: 24 us, 28 by the cuts).
template <typename KeyOf, bool kWithPos, int kPer, typename Sh>
__device__ __forceinline__ void sort_head(const uint32_t* src, uint32_t n, uint32_t* list_key, uint32_t* list_pos, Sh& sh) {
    uint32_t least = 0xffffffffu, most = 0u;
    uint32_t lane_of_all = threadIdx.x;
    asm volatile("" : "+v"(lane_of_all));                             // positions of earlier passes are not worth registers until here
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t t = u * kSortLanes + lane_of_all;
        if (t < n) {
            const uint32_t key = KeyOf::of(src[t]);
            list_key[t] = key;
            if constexpr (kWithPos) list_pos[t] = t;
            least = key < least ? key : least;
            most = key > most ? key : most;
        }
    }
    least = wave_min(least);
    most = ~wave_min(~most);
    if (threadIdx.x % kWaveSize == 0) {
        sh.wave[0][threadIdx.x / kWaveSize] = least;
        sh.wave[1][threadIdx.x / kWaveSize] = most;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        least = sh.wave[0][w] < least ? sh.wave[0][w] : least;
        most = sh.wave[1][w] > most ? sh.wave[1][w] : most;
    }
    sort_list<kWithPos, kPer>(list_key, list_pos, n, KeyRange{least, most}, sh);
}

// The elements of ranks [r0, r1) in order; returns where in the list they start.  Two shares and more would each sort the
// whole head, which costs less than the cuts while it is short.
template <typename KeyOf, bool kWithPos, int kPer>
__device__ __forceinline__ uint32_t sorted_range(const uint32_t* src, uint32_t n, uint32_t r0, uint32_t r1, uint32_t* list_key,
                                                 uint32_t* list_pos, BinShared& sh, CutShared& cs) {
    __syncthreads();                                                  // the list is free
    if (n <= (uint32_t)(kPer * kSortLanes / 2) || (r0 == 0 && r1 == n && n <= (uint32_t)(kPer * kSortLanes))) {
        sort_head<KeyOf, kWithPos, kPer>(src, n, list_key, list_pos, sh);
        return r0;
    }
    if (r0 == r1) return 0;                                           // the same for all lanes
    const KeyRange range = gather_range<KeyOf, kWithPos>(src, n, r0, r1, list_key, list_key, list_pos, cs);
    sort_list<kWithPos, kPer>(list_key, list_pos, r1 - r0, range, sh);
    return 0;
}

// drop_rank[h][t] = T - 1 - (rank of (norm bits, t) in ascending order).
template <int E>
__global__ __launch_bounds__(kSortLanes)
void norm_ranks_kernel(const float* __restrict__ norms, int64_t T, uint32_t n_heads, Cut cut, int32_t* __restrict__ drop_rank) {
    __shared__ BinShared sh;
    __shared__ CutShared s_cut;
    __shared__ __attribute__((aligned(16))) uint32_t s_list[kListWords];
    const Part part = part_of_block(blockIdx.x, n_heads, cut.shares);
    const uint32_t n = (uint32_t)T;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(norms) + part.head * T;
    uint32_t* rank = reinterpret_cast<uint32_t*>(drop_rank) + part.head * T;
    const HeadKeys<E, BitBins> keys(src, n);
    const auto s = find_share(keys, n, part.share, cut, s_list, sh);
    if (s.kmin == s.kmax) {                                          // equal norms: the order of the positions
        const uint32_t end = cut.start(part.share + 1);
        for (uint32_t t = cut.start(part.share) + threadIdx.x; t < end; t += kSortLanes) rank[t] = n - 1 - t;
        return;
    }
    constexpr int kPer = kListPer / 2;                               // keys and positions share the list
    uint32_t* const list_pos = s_list + kPer * kSortLanes;
    if (!s.crowded) {
        Ranked<kPer, BitBins> mine;
        if (rank_share<true, kPer>(keys, s, sh, s_list, mine)) {
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (u * kSortLanes + threadIdx.x < s.count) rank[mine.pos[u]] = n - 1 - (s.base + mine.rank[u]);
            return;
        }
    }
    const uint32_t r0 = s.crowded ? cut.start(part.share) : s.base;
    const uint32_t r1 = s.crowded ? cut.start(part.share + 1) : s.base + s.count;
    const uint32_t at = sorted_range<NormKey, true, kPer>(src, n, r0, r1, s_list, list_pos, sh, s_cut);
    for (uint32_t i = threadIdx.x; i < r1 - r0; i += kSortLanes) rank[list_pos[at + i]] = n - 1 - (r0 + i);
}

// Short heads: sorted whole by one workgroup each, in so little LDS that two run on a compute unit.
struct ShortShared {
    uint32_t fine[kSortWaves * kBins];
    uint32_t bin[kBins];
    uint32_t wave[2][kSortWaves];
};
template <int kPer>
__global__ __launch_bounds__(kSortLanes)
void norm_ranks_short_kernel(const float* __restrict__ norms, int64_t T, int32_t* __restrict__ drop_rank) {
    __shared__ ShortShared sh;
    __shared__ uint32_t s_key[kPer * kSortLanes], s_pos[kPer * kSortLanes];
    const uint32_t n = (uint32_t)T;
    uint32_t* rank = reinterpret_cast<uint32_t*>(drop_rank) + blockIdx.x * T;
    sort_head<NormKey, true, kPer>(reinterpret_cast<const uint32_t*>(norms) + blockIdx.x * T, n, s_key, s_pos, sh);
    __syncthreads();                                                  // one key: no pass, no barrier
    for (uint32_t i = threadIdx.x; i < n; i += kSortLanes) rank[s_pos[i]] = n - 1 - i;
}

// The same by the counting passes, one workgroup per head (share_plan has the line).
__global__ __launch_bounds__(kSortLanes)
void norm_ranks_passes_kernel(const float* __restrict__ norms, int64_t T, uint32_t* __restrict__ scratch,
                              int32_t* __restrict__ drop_rank) {
    __shared__ SortShared sort;
    const int64_t head = blockIdx.x;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(norms) + head * T;
    uint32_t* a_key = scratch + head * 4 * T;
    uint32_t* a_val = a_key + T;
    uint32_t* b_key = a_val + T;
    uint32_t* b_val = b_key + T;
    radix_pass<kIotaIn>(src, nullptr, a_key, a_val, T, 0, sort);
    radix_pass<kPairs>(a_key, a_val, b_key, b_val, T, 8, sort);
    radix_pass<kPairs>(b_key, b_val, a_key, a_val, T, 16, sort);
    radix_pass<kRankOut>(a_key, a_val, nullptr, reinterpret_cast<uint32_t*>(drop_rank) + head * T, T, 24, sort);
}

// Where the shares of a query head leave their sums: at the start of the head's second scratch array,
// which only the counting passes use otherwise.  One counter, then a record per share.
constexpr int kRecordHeader = 4;                     // words in front of the records
constexpr int kRecordSums = 5;                       // sum e, sum e * rank, dropped sum, sum e_(j) * j, sum of the m lowest
constexpr int kRecordWords = 2 * kRecordSums;        // doubles
__device__ __forceinline__ uint32_t* record_base(uint32_t* second, int64_t head, int64_t T) {
    return reinterpret_cast<uint32_t*>((reinterpret_cast<uintptr_t>(second + head * T) + 15) & ~(uintptr_t)15);
}

// Scaled logits of all G query heads of one KV head over a block of rows:
// scores[b*Hq + hkv*G + g][t] = (q_g . K_t) * scale * log2(e).
constexpr int kScoreWaves = 4;
// 4 loads in flight per lane: 43.5 us for 32 heads of 32k rows and 4 query heads each (6.2 TB/s); 8 loads 44.8, 2 loads
// 47.5.  Scores stored straight from the row loop, 16 bytes per row group, instead of one run per wave
// and head: 46.7 (8 loads).
constexpr int kScoreLoads = 4;                                        // row loads in flight per lane
constexpr int kScoreRowsPerWave = kScoreLoads * kRowsPerWaveLoad;     // 16
constexpr int kScoreRowsPerBlock = kScoreWaves * kScoreRowsPerWave;   // 64

template <typename E, int D, int G>
__global__ __launch_bounds__(kScoreWaves * kWaveSize)
void alr_scores_kernel(const void* __restrict__ Q, const void* __restrict__ K, int64_t T,
                       int64_t k_head_stride, float scale_log2e, float* __restrict__ scores,
                       uint32_t* __restrict__ records, bool through) {
    using S = Slice<E, D>;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    const int c = lane % kRowLanes;
    const int r = lane / kRowLanes;
    const int64_t head = blockIdx.y;                                   // b * Hkv + hkv
    const int64_t q_head0 = head * G;                                  // b * Hq + hkv * G
    // the arrival counters of the ranking launch that follows
    if (records != nullptr && blockIdx.x == 0 && threadIdx.x < G) *record_base(records, q_head0 + threadIdx.x, T) = 0u;
    // q and K rows are shared among the 16 lanes in the same 16-byte pieces (the dot product
    // does not care which lane holds which element)
    using P = Pieces<S::kWords>;
    const char* kbase = static_cast<const char*>(K) + head * k_head_stride * E::kBytes + c * P::kBytes;
    const char* qbase = static_cast<const char*>(Q) + q_head0 * S::kRowBytes + c * P::kBytes;

    float q[G][S::kElems];
#pragma unroll
    for (int g = 0; g < G; ++g) widen<E, D>(load_words<S::kWords, P::kStride>(qbase + (size_t)g * S::kRowBytes), q[g]);

    __shared__ float s_scores[kScoreWaves][G][kScoreRowsPerWave];      // every wave uses its own part
    const int64_t row0 = (int64_t)blockIdx.x * kScoreRowsPerBlock + wave * kScoreRowsPerWave + r;
    Words<S::kWords> tile[kScoreLoads];
#pragma unroll
    for (int u = 0; u < kScoreLoads; ++u) {
        int64_t t = row0 + u * kRowsPerWaveLoad;
        t = t < T ? t : T - 1;                                         // clamped, never stored
        tile[u] = load_words_stream<S::kWords, P::kStride>(kbase + (size_t)t * S::kRowBytes);
    }
#pragma unroll
    for (int u = 0; u < kScoreLoads; ++u) {
        float x[S::kElems];
        widen<E, D>(tile[u], x);
        float mine = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < S::kElems; ++i) p = fmaf(q[g][i], x[i], p);
            p = row16_tree_sum(p);
            mine = c == g ? p : mine;
        }
        if (c < G) s_scores[wave][c][u * kRowsPerWaveLoad + r] = mine * scale_log2e;
    }
    // the wave's scores of consecutive rows leave as one run per head; other lanes wrote them, so the
    // compiler must not move the reads past the writes (the wave's LDS accesses themselves stay in order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int64_t first = (int64_t)blockIdx.x * kScoreRowsPerBlock + wave * kScoreRowsPerWave;
    constexpr int kHeadsPerStore = kWaveSize / kScoreRowsPerWave;
    const int row = lane % kScoreRowsPerWave;
#pragma unroll
    for (int g0 = 0; g0 < G; g0 += kHeadsPerStore) {
        const int g = g0 + lane / kScoreRowsPerWave;
        if (g < G && first + row < T) {
            float* const out = scores + (q_head0 + g) * T + first + row;
            const float score = s_scores[wave][g][row];
            if (through) __hip_atomic_store(out, score, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *out = score;
        }
    }
}

// Sum of one double per lane over the wave, in a fixed order; the same in all lanes.
template <int CTRL> __device__ __forceinline__ double dpp_read(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double read_lane(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_read<kDppXor1>(v);
    v += dpp_read<kDppXor2>(v);
    v += dpp_read<kDppHalfMirror>(v);
    v += dpp_read<kDppMirror>(v);
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Fixed-order sums of doubles over the workgroup, in two steps: every wave leaves its sums of v in stage[wave][kFrom ..]; once all
// are there, the first wave adds them up (results valid in thread 0; ends with a barrier).
template <int kFrom, int N, int kAll>
__device__ __forceinline__ void stage_sums(const double (&v)[N], double (*stage)[kAll]) {
    static_assert(kFrom + N <= kAll, "columns");
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double s = wave_sum(v[i]);
        if (threadIdx.x % kWaveSize == 0) stage[threadIdx.x / kWaveSize][kFrom + i] = s;
    }
}
template <int N>
__device__ __forceinline__ void sum_staged(double (&v)[N], double (*stage)[N]) {
    __syncthreads();
    if (threadIdx.x < kWaveSize) {        // the 16 lanes of a row hold the waves' sums of a column, four columns at a time
        static_assert(kSortWaves == kRowLanes, "a lane per wave");
        const int row = threadIdx.x / kRowLanes;
#pragma unroll
        for (int i = 0; i < N; i += 4) {
            double s = stage[threadIdx.x % kRowLanes][i + row < N ? i + row : 0];
            s += dpp_read<kDppXor1>(s);
            s += dpp_read<kDppXor2>(s);
            s += dpp_read<kDppHalfMirror>(s);
            s += dpp_read<kDppMirror>(s);
#pragma unroll
            for (int j = i; j < N && j < i + 4; ++j) v[j] = read_lane(s, (j - i) * kRowLanes);
        }
    }
    __syncthreads();
}
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double (*stage)[N]) {
    stage_sums<0>(v, stage);
    sum_staged(v, stage);
}

__device__ __forceinline__ double score(float logit, float mx) { return (double)__builtin_amdgcn_exp2f(logit - mx); }

// What the element of rank j in ascending order of the scores adds to the reference of Eq. 6 and 7.
struct RankedSums { double weighted = 0.0, lowest = 0.0; };
__device__ __forceinline__ void add_ranked(RankedSums& sums, double e, uint32_t j, int64_t m) {
    sums.weighted += e * (double)j;
    sums.lowest += (int64_t)j < m ? e : 0.0;
}

// e_p = 2^(logit - mx) of positions [p0, p1): their sum, the rank-weighted sum and the mass of the m pairs dropped by
// norm.  equal: all scores are, so that positions do for ranks.  kToBits: the logits are replaced by their ordered bits.
struct PositionSums { double all = 0.0, weighted = 0.0, dropped = 0.0; };
template <bool kToBits>
__device__ __forceinline__ PositionSums position_sums(uint32_t* logits, const int32_t* __restrict__ rank, uint32_t p0, uint32_t p1,
                                                      int64_t m, float mx, bool equal, RankedSums& ranked) {
    PositionSums sums;
    for (uint32_t base = p0; base < p1; base += kBatch * kSortLanes) {
        uint32_t bits[kBatch];
        int32_t rk[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t t = base + u * kSortLanes + threadIdx.x;
            bits[u] = logits[t < p1 ? t : p1 - 1];
            rk[u] = rank[t < p1 ? t : p1 - 1];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t t = base + u * kSortLanes + threadIdx.x;
            const double e = t < p1 ? score(__builtin_bit_cast(float, bits[u]), mx) : 0.0;
            sums.all += e;
            sums.weighted += e * (double)rk[u];
            sums.dropped += rk[u] < m ? e : 0.0;
            if (equal) add_ranked(ranked, e, t, m);
            if (kToBits && t < p1) logits[t] = ordered_bits(bits[u]);
        }
    }
    return sums;
}

// The same for heads whose logits are in registers, where a share takes whole blocks of 1024 positions: nothing but the ranks is
// fetched, and those are on their way while the range of the logits is found.
template <int E> struct RegisterSums {
    static constexpr uint32_t kSlots = position_slots(E);
    __amdgpu_buffer_rsrc_t rank;                                      // reads zero past the end
    uint32_t n;
    PositionBlocks<kSlots> blocks;
    int32_t rk[kSlots];
    __device__ __forceinline__ RegisterSums(const int32_t* r, uint32_t count, uint32_t share, uint32_t shares)
        : n(count), blocks((count + kSortLanes - 1) / kSortLanes, share, shares) {
        rank = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(r), 0, (int)(n * sizeof(int32_t)), kRawBufferWord3);
        // all of the offset per lane: that is what is checked against the end of the head
#pragma unroll
        for (uint32_t j = 0; j < kSlots; ++j)
            rk[j] = __builtin_amdgcn_raw_buffer_load_b32(rank, (blocks.in_slot(j) * kSortLanes + threadIdx.x) * sizeof(int32_t), 0, kBufferPolicyPlain);
    }
    template <typename Keys>
    __device__ __forceinline__ PositionSums add_up(const Keys& keys, int64_t m, float mx, bool equal, RankedSums& ranked) {
        PositionSums sums;
        uint32_t left = n - threadIdx.x;
        asm volatile("" : "+v"(left));
        const int32_t dropped = m < INT32_MAX ? (int32_t)m : INT32_MAX;
#pragma unroll
        for (uint32_t e = 0; e < (uint32_t)E; ++e) {
            if (blocks.has(e)) {                                      // the same for all lanes
                const double x = (int32_t)left > (int32_t)(e * kSortLanes) ? score(keys.reg[e], mx) : 0.0;
                const int32_t r = rk[e % kSlots];
                sums.all += x;
                sums.weighted += x * (double)r;
                sums.dropped += r < dropped ? x : 0.0;
            }
        }
        if (equal) {
            for (uint32_t t = blocks.first * kSortLanes + threadIdx.x; t < blocks.end * kSortLanes && t < n; t += kSortLanes) add_ranked(ranked, score(mx, mx), t, m);
        }
        return sums;
    }
};

// The elements of ranks r0 .. r0 + kRun - 1, `count` of which are there.
__device__ __forceinline__ void add_run(RankedSums& sums, const float (&run)[kRun], float mx, uint32_t r0, uint32_t count, int64_t m) {
    double all = 0.0, above = 0.0;                                    // sum e, sum e * (rank - r0)
#pragma unroll
    for (int i = kRun - 1; i >= 0; --i) {
        if (i < kRun - 1) above += all;
        all += (uint32_t)i < count ? score(run[i], mx) : 0.0;
    }
    sums.weighted += all * (double)r0 + above;
    if ((int64_t)r0 + kRun <= m) {
        sums.lowest += all;
    } else if ((int64_t)r0 < m) {
#pragma unroll
        for (int i = 0; i < kRun; ++i) sums.lowest += (uint32_t)i < count && (int64_t)(r0 + i) < m ? score(run[i], mx) : 0.0;
    }
}

__device__ __forceinline__ void write_losses(const double (&acc)[kRecordSums], int64_t head, double* __restrict__ alr,
                                             double* __restrict__ loss, double* __restrict__ loss_ref) {
    alr[head] = (acc[3] - acc[1]) / acc[0];
    if (loss != nullptr) loss[head] = acc[2] / acc[0];
    if (loss_ref != nullptr) loss_ref[head] = acc[4] / acc[0];
}

// What the ranking of a head's scores keeps in LDS: with runs 163712 of the 163840 bytes that a compute unit has.
template <bool kRuns> struct HeadShared {
    union {
        BinShared sh;
        std::conditional_t<kRuns, RunBins, uint32_t> bins;
    };
    CutShared cut;
    __attribute__((aligned(16))) uint32_t list[kRuns ? kRunWords + kWaveSize : (uint32_t)kListWords];
    double stage[kSortWaves][kRecordSums];
    RunShared runs;
    uint32_t ticket;
};

// The sums in order of rank of one share, ranks [r0, r1), by an exact cut and a sort, wherever its elements lie.
typedef const uint32_t __attribute__((address_space(1)))* GlobalWords;     // of a plain pointer it would not know that it is not LDS
template <bool kRuns>
__device__ __forceinline__ RankedSums sorted_sums(GlobalWords logits, uint32_t n, uint32_t r0, uint32_t r1, float mx, int64_t m, HeadShared<kRuns>& lds) {
    RankedSums ranked;
    const uint32_t at = sorted_range<LogitKey, false, kListPer>((const uint32_t*)logits, n, r0, r1, lds.list, nullptr, lds.sh, lds.cut);
    for (uint32_t i = threadIdx.x; i < r1 - r0; i += kSortLanes)
        add_ranked(ranked, score(float_of_ordered(lds.list[at + i]), mx), r0 + i, m);
    return ranked;
}
// The same by comparing inside the finer bins, as long as these do not hold too many; else false.
template <typename Keys>
__device__ __forceinline__ bool compared_sums(const Keys& keys, const Share<ValueBins>& s, int64_t m, RankedSums& ranked, HeadShared<false>& lds) {
    float* const list = reinterpret_cast<float*>(lds.list);
    Ranked<kListPer, ValueBins> mine;
    if (!rank_share<false, kListPer>(keys, s, lds.sh, list, mine)) return false;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kListPer; ++u)
        if (u * kSortLanes + threadIdx.x < s.count) list[mine.rank[u]] = mine.key[u];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < s.count; i += kSortLanes) add_ranked(ranked, score(list[i], s.kmax), s.base + i, m);
    return true;
}

// Heads of more than 8192 tokens whose keys stay in registers: in runs.  us for the losses, compared in the list / in runs: 128 heads of 9000
// 34.1, 30.7; 16384 47.3, 43.3; 32768 85.3, 74.4; 256 heads of 18000 72.6, 62.7; 32 heads of 9000 23.4, 22.4, of 32768 38.3, 35.3.  Up to
// 8192 tokens a share is so small that runs of 32 leave most lanes idle: 32 heads of 3000 18.4, 19.7; 128 of 3000 20.9, 22.2.
// Equal logits, counted twice in bins of a share with at most 64 in a bin, and the exact cut beyond / here: 20 equal each, 128 heads of 32768
// 95, 93, of 12000 48, 43, 32 of 9000 30.5, 27.3; 40 equal 142, 90, 68, 47, 31.0, 31.7; 100 equal 141, 116, 68, 57, 54, 44; half of all equal
// (exact cut) 128 of 12000 70.4, 70.7.  One key row 200 times as long as the others: 135, 78.
template <int E> constexpr bool kInRuns = E > 8;

// Softmax statistics, rank-weighted sums, ranks of the scores by value ranges, and the three
// outputs.  Every share adds up its stretch of positions and its range of ranks; with several
// shares the sums meet in the head's records and the share that finishes last (arrival counter)
// adds them in order of the shares, so the result does not depend on timing.  Records and counter
// travel with device scope; a share waits until its record has been acknowledged before it
// takes its ticket, and nobody waits for anybody.
template <int E>
__global__ __launch_bounds__(kSortLanes)
void alr_head_kernel(uint32_t* __restrict__ scratch, const int32_t* __restrict__ drop_rank, int64_t T,
                     uint32_t n_heads, int32_t G, Cut cut, int64_t m, double* __restrict__ alr,
                     double* __restrict__ loss, double* __restrict__ loss_ref) {
    constexpr bool kRuns = kInRuns<E>;
    __shared__ HeadShared<kRuns> lds;
    uint32_t* const s_list = lds.list;
    double (&stage)[kSortWaves][kRecordSums] = lds.stage;
    const Part part = part_of_block(blockIdx.x, n_heads, cut.shares);     // head = b * Hq + hq
    const int64_t head = part.head;
    const uint32_t n = (uint32_t)T;
    // scratch: two arrays [n_heads][T]; the first holds the logits
    uint32_t* logits = scratch + head * T;
    uint32_t* second = scratch + (int64_t)n_heads * T;
    const int32_t* rank = drop_rank + (head / G) * T;

    const uint32_t p0 = cut.start(part.share), p1 = cut.start(part.share + 1);
    const HeadKeys<E, ValueBins> keys(logits, n);
    std::conditional_t<(E > 0), RegisterSums<E>, std::nullptr_t> by_position = [&] {
        if constexpr (E > 0) return RegisterSums<E>(rank, n, part.share, cut.shares);
        else return nullptr;
    }();
    // equal scores: any order.  mx: the largest.
    auto sum_positions = [&](float mx, bool equal, RankedSums& ranked) {
        PositionSums sums;
        if constexpr (E > 0) sums = by_position.add_up(keys, m, mx, equal, ranked);
        else sums = position_sums<false>(logits, rank, p0, p1, m, mx, equal, ranked);
        stage_sums<0>({sums.all, sums.weighted, sums.dropped}, stage);        // not in registers any longer
    };
    RankedSums ranked;
    float mx;
    uint32_t r0 = p0, r1 = p1;                                            // ranks that an exact cut takes
    bool done = true;
    if constexpr (kRuns) {
        for (uint32_t i = threadIdx.x; i < kScoreBins / 4; i += kSortLanes) reinterpret_cast<uint4*>(lds.bins.bin)[i] = make_uint4(0, 0, 0, 0);
        const ScoreRange range = score_range(keys, lds.runs);
        mx = range.hi;
        sum_positions(mx, range.lo == range.hi, ranked);
        if (range.lo != range.hi) {
            float run[kRun];
            uint32_t base, count;
            done = order_share<E>(keys, range, part.share, cut, lds.bins, lds.runs, reinterpret_cast<float*>(s_list), run, base, count);
            const uint32_t at = threadIdx.x * kRun;
            if (done && at < count) add_run(ranked, run, mx, base + at, count - at, m);
        }
    } else {
        const auto s = find_share(keys, n, part.share, cut, s_list, lds.sh);
        mx = s.kmax;
        sum_positions(mx, s.kmin == s.kmax, ranked);
        if (s.kmin != s.kmax) {
            done = !s.crowded && compared_sums(keys, s, m, ranked, lds);
            if (!s.crowded) r0 = s.base, r1 = s.base + s.count;
        }
    }
    // Seldom, as the compiler has to know, and with nothing left in registers for it, not even what would only be loaded again:
    // otherwise the path that nearly all heads take spills (42 us in place of 33 for 128 heads of 32k).
    if (__builtin_expect(!done, false)) {
        GlobalWords again = (GlobalWords)logits;
        uint32_t count = n;
        asm volatile("" : "+s"(again), "+s"(count));
        ranked = sorted_sums(again, count, r0, r1, mx, m, lds);
    }
    stage_sums<3>({ranked.weighted, ranked.lowest}, stage);
    double acc[kRecordSums];
    sum_staged(acc, stage);                                           // valid in thread 0

    if (cut.shares > 1) {
        uint32_t* counter = record_base(second, head, T);
        uint32_t* records = counter + kRecordHeader;
        if (threadIdx.x == 0) {
            auto* out = reinterpret_cast<unsigned long long*>(records + part.share * kRecordWords);
#pragma unroll
            for (int i = 0; i < kRecordSums; ++i)
                __hip_atomic_store(out + i, __builtin_bit_cast(unsigned long long, acc[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            lds.ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (lds.ticket != cut.shares - 1) return;
        // the records into LDS with independent loads, then added in order
        uint32_t* copy = s_list;
        for (uint32_t i = threadIdx.x; i < cut.shares * kRecordWords; i += kSortLanes)
            copy[i] = __hip_atomic_load(records + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int i = 0; i < kRecordSums; ++i) acc[i] = 0.0;
            for (uint32_t w = 0; w < cut.shares; ++w) {
#pragma unroll
                for (int i = 0; i < kRecordSums; ++i) acc[i] += reinterpret_cast<const double*>(copy + w * kRecordWords)[i];
            }
        }
    }
    if (threadIdx.x == 0) write_losses(acc, head, alr, loss, loss_ref);
}

// The same for short heads, sorted whole by one workgroup each.
template <int kPer>
__global__ __launch_bounds__(kSortLanes)
void alr_head_short_kernel(uint32_t* __restrict__ scratch, const int32_t* __restrict__ drop_rank, int64_t T, int32_t G, int64_t m,
                           double* __restrict__ alr, double* __restrict__ loss, double* __restrict__ loss_ref) {
    __shared__ ShortShared sh;
    __shared__ uint32_t s_key[kPer * kSortLanes];
    __shared__ double stage[kSortWaves][kRecordSums];
    const int64_t head = blockIdx.x;
    const uint32_t n = (uint32_t)T;
    uint32_t* logits = scratch + head * T;
    sort_head<LogitKey, false, kPer>(logits, n, s_key, nullptr, sh);
    __syncthreads();
    const float mx = float_of_ordered(s_key[n - 1]);
    RankedSums ranked;
    for (uint32_t j = threadIdx.x; j < n; j += kSortLanes) add_ranked(ranked, score(float_of_ordered(s_key[j]), mx), j, m);
    const PositionSums sums = position_sums<false>(logits, drop_rank + (head / G) * T, 0, n, m, mx, false, ranked);
    double acc[kRecordSums] = {sums.all, sums.weighted, sums.dropped, ranked.weighted, ranked.lowest};
    block_sum<kRecordSums>(acc, stage);
    if (threadIdx.x == 0) write_losses(acc, head, alr, loss, loss_ref);
}

// The same by the counting passes, one workgroup per head.  Both scratch arrays are the passes'.
__global__ __launch_bounds__(kSortLanes)
void alr_head_passes_kernel(uint32_t* __restrict__ scratch, const int32_t* __restrict__ drop_rank, int64_t T, int32_t G, int64_t m,
                            double* __restrict__ alr, double* __restrict__ loss, double* __restrict__ loss_ref) {
    __shared__ SortShared sort;
    __shared__ double stage[kSortWaves][kRecordSums];
    __shared__ float s_max[kSortWaves];
    const int64_t head = blockIdx.x;
    const uint32_t n = (uint32_t)T;
    uint32_t* buf0 = scratch + head * T;
    uint32_t* buf1 = scratch + ((int64_t)gridDim.x + head) * T;
    const int32_t* rank = drop_rank + (head / G) * T;

    float mx = -INFINITY;
    for (uint32_t t = threadIdx.x; t < n; t += kSortLanes) mx = fmaxf(mx, __builtin_bit_cast(float, buf0[t]));
#pragma unroll
    for (int off = kWaveSize / 2; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (threadIdx.x % kWaveSize == 0) s_max[threadIdx.x / kWaveSize] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) mx = fmaxf(mx, s_max[w]);

    RankedSums ranked;
    const PositionSums sums = position_sums<true>(buf0, rank, 0, n, m, mx, false, ranked);
    __syncthreads();                                                  // the stores before the sort
    radix_pass<kKeysOnly>(buf0, nullptr, buf1, nullptr, T, 0, sort);
    radix_pass<kKeysOnly>(buf1, nullptr, buf0, nullptr, T, 8, sort);
    radix_pass<kKeysOnly>(buf0, nullptr, buf1, nullptr, T, 16, sort);
    radix_pass<kKeysOnly>(buf1, nullptr, buf0, nullptr, T, 24, sort);
    for (uint32_t j = threadIdx.x; j < n; j += kSortLanes) add_ranked(ranked, score(float_of_ordered(buf0[j]), mx), j, m);
    double acc[kRecordSums] = {sums.all, sums.weighted, sums.dropped, ranked.weighted, ranked.lowest};
    block_sum<kRecordSums>(acc, stage);
    if (threadIdx.x == 0) write_losses(acc, head, alr, loss, loss_ref);
}

// Heads that are sorted whole in a small workgroup.  Binning takes 100 KB more of LDS, so that half as many run at once, and
// does not gain on a sort of one or two keys per lane.  Norms, us, by bins / by the counting passes / whole: 16 heads of 300
// 8.3, 11.0, 6.3 (30 % zero 34.8, 11.1, 6.3); 4096 heads of 300 117, 94, 52; 4096 of 1000 122, 152, 81; 1024 of 2000 37.5,
// 70.9, 38.7 (30 % zero 77, 64, 37); the bins are the better 16 heads of 2000 9.0, 18.3, 12.1 and 1024 of 4096 50, 137, 71.
bool is_short(int64_t n_heads, int64_t T) { return T <= kSortLanes || (T <= 2 * kSortLanes && n_heads >= 512); }

template <typename E, int D>
l2kv_status launch_scores(const void* Q, const void* K, int32_t B, int32_t Hkv, int32_t G, int64_t T,
                          int64_t k_head_stride, float scale_log2e, float* scores, uint32_t* records, hipStream_t stream) {
    const dim3 grid((unsigned)((T + kScoreRowsPerBlock - 1) / kScoreRowsPerBlock), (unsigned)(B * Hkv));
    const dim3 block(kScoreWaves * kWaveSize);
    // Scores stored past the L2 as they come leave nothing to be written back between the two launches, and the workgroups that rank
    // them, on other dies than those that wrote them, wait less for theirs.  Both launches, us, ordinary stores / through: 128 heads
    // of 32k (16 MB) 75.1 / 73.7, 256 of 32k 145.1 / 141.2, 256 of 9500 (9.3 MB) 41.4 / 40.3, 1024 of 2500 76.8 / 76.5; less than
    // 8 MB stay in the L2s: 32 of 32k (4 MB) 35.2 / 35.7, 128 of 3000 20.65 / 20.81.
    const bool through = (int64_t)B * Hkv * G * T * (int64_t)sizeof(float) >= 9 << 20;
#define L2KV_SCORES(GG)                                                                             \
    case GG:                                                                                        \
        hipLaunchKernelGGL((alr_scores_kernel<E, D, GG>), grid, block, 0, stream, Q, K, T,          \
                           k_head_stride, scale_log2e, scores, records, through);                   \
        break;
    switch (G) {
        L2KV_SCORES(1) L2KV_SCORES(2) L2KV_SCORES(3) L2KV_SCORES(4)
        L2KV_SCORES(5) L2KV_SCORES(6) L2KV_SCORES(7) L2KV_SCORES(8)
        default: return L2KV_ERR_SHAPE;
    }
#undef L2KV_SCORES
    return launch_status();
}

}  // namespace

size_t norm_ranks_workspace_bytes(int64_t n_heads, int64_t T) {
    const size_t raw = (size_t)n_heads * (size_t)T * 4 * sizeof(uint32_t);
    return (raw + 255) / 256 * 256;
}

size_t alr_workspace_bytes(int32_t B, int32_t Hq, int64_t T) {
    const size_t raw = (size_t)B * (size_t)Hq * (size_t)T * 2 * sizeof(uint32_t);
    return (raw + 255) / 256 * 256;
}

l2kv_status norm_ranks_dispatch(const float* norms, int64_t n_heads, int64_t T, int32_t* drop_rank,
                                void* workspace, hipStream_t stream) {
    if (is_short(n_heads, T)) {
        auto kernel = T <= kSortLanes ? norm_ranks_short_kernel<1> : norm_ranks_short_kernel<2>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_heads), dim3(kSortLanes), 0, stream, norms, T, drop_rank);
        return launch_status();
    }
    const int64_t shares = share_plan(n_heads, T, kLongestRankedShare);
    if (shares == 0) {
        hipLaunchKernelGGL(norm_ranks_passes_kernel, dim3((unsigned)n_heads), dim3(kSortLanes), 0, stream, norms, T,
                           static_cast<uint32_t*>(workspace), drop_rank);
        return launch_status();
    }
    // keys per lane: 32 heads of 16384 norms 17.5 us at 32, 14.5 at 16, 8 of 9000 15.3 and 12.4, 8 of 20001 16.2 and, at 24, 14.6
    auto kernel = T <= 8 * kSortLanes    ? norm_ranks_kernel<8>
                  : T <= 16 * kSortLanes ? norm_ranks_kernel<16>
                  : T <= 24 * kSortLanes ? norm_ranks_kernel<24>
                  : T <= 32 * kSortLanes ? norm_ranks_kernel<32>
                                         : norm_ranks_kernel<0>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_heads * shares)), dim3(kSortLanes), 0, stream, norms, T,
                       (uint32_t)n_heads, Cut((uint32_t)T, (uint32_t)shares), drop_rank);
    return launch_status();
}

l2kv_status alr_dispatch(const void* Q, const void* K, l2kv_dtype dt, const int32_t* drop_rank, int32_t B,
                         int32_t Hq, int32_t Hkv, int64_t T, int32_t D, int64_t k_head_stride, float scale,
                         int64_t m, double* alr, double* loss, double* loss_ref, void* workspace,
                         hipStream_t stream) {
    const int32_t G = Hq / Hkv;
    const float s = scale > 0.f ? scale : 1.0f / sqrtf((float)D);
    const float scale_log2e = s * 1.44269504088896340736f;
    float* scores = static_cast<float*>(workspace);
    const int64_t n_heads = (int64_t)B * Hq;
    const int64_t shares = is_short(n_heads, T) ? 1 : share_plan(n_heads, T, kLongestShare);
    uint32_t* records = shares > 1 ? static_cast<uint32_t*>(workspace) + n_heads * T : nullptr;
    l2kv_status st;
    if (dt == L2KV_BF16 && D == 256)
        st = launch_scores<BF16, 256>(Q, K, B, Hkv, G, T, k_head_stride, scale_log2e, scores, records, stream);
    else if (dt == L2KV_BF16)
        st = D == 128 ? launch_scores<BF16, 128>(Q, K, B, Hkv, G, T, k_head_stride, scale_log2e, scores, records, stream)
                      : launch_scores<BF16, 64>(Q, K, B, Hkv, G, T, k_head_stride, scale_log2e, scores, records, stream);
    else
        st = D == 128 ? launch_scores<F32, 128>(Q, K, B, Hkv, G, T, k_head_stride, scale_log2e, scores, records, stream)
                      : launch_scores<F32, 64>(Q, K, B, Hkv, G, T, k_head_stride, scale_log2e, scores, records, stream);
    if (st != L2KV_OK) return st;
    if (is_short(n_heads, T)) {
        auto kernel = T <= kSortLanes ? alr_head_short_kernel<1> : alr_head_short_kernel<2>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_heads), dim3(kSortLanes), 0, stream,
                           static_cast<uint32_t*>(workspace), drop_rank, T, G, m, alr, loss, loss_ref);
        return launch_status();
    }
    if (shares == 0) {
        hipLaunchKernelGGL(alr_head_passes_kernel, dim3((unsigned)n_heads), dim3(kSortLanes), 0, stream,
                           static_cast<uint32_t*>(workspace), drop_rank, T, G, m, alr, loss, loss_ref);
        return launch_status();
    }
    const int per = score_keys_per_lane(T);
    auto kernel = per == 8    ? alr_head_kernel<8>
                  : per == 16 ? alr_head_kernel<16>
                  : per == 20 ? alr_head_kernel<20>
                  : per == 24 ? alr_head_kernel<24>
                  : per == 32 ? alr_head_kernel<32>
                              : alr_head_kernel<0>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_heads * shares)), dim3(kSortLanes), 0, stream,
                       static_cast<uint32_t*>(workspace), drop_rank, T, (uint32_t)n_heads, G, Cut((uint32_t)T, (uint32_t)shares), m,
                       alr, loss, loss_ref);
    return launch_status();
}

}  // namespace l2kv
