// l2kv_select: per head, the k positions that come first in the total order
// (bit pattern of the fp32 squared norm, token index), written in ascending
// token order.  This is the eviction rule of arXiv 2406.11430 (Sec. 1: keep
// the lowest-norm keys; Eq. 5: exactly m pairs dropped per layer and head)
// with ties resolved towards the lower token index.
//
// The k-th smallest key tau (key = norm bits, complemented for the keep-highest
// control) is found exactly: the keys are counted in 4096 LDS bins (2048 for heads of at most 2048 tokens) of equal width between the
// smallest and the largest of the head, and the prefix sums lead to the bin that holds the k-th.  The bin's
// keys, a few dozen as a rule, are listed and compared with each other; a fuller bin (tied or
// clustered norms) is divided into as many again, at most twice, until its keys are few or equal.
// Bound by the LDS round trips and barriers of that chain, not by its arithmetic: 512 heads
// of 4k take 8.8 us, 256 of 32k 15.9, 1024 of 32k 65 (three digits of 12, 10 and 10 bits with a prefix sum for
// each, in 80 KB of LDS and so one workgroup per compute unit: 11.6, 17.3 and 72; heads with an infinite and a
// zero norm, whose bins are divided once more, 8.2 against 6.8 for 256 of 4k).
// (A binary search over the 32 bits, one barrier and one compare per key
// and bit, took 40 us for 256 heads of 32k tokens.)  The emit is ordered: every wave owns a contiguous token
// range, so a prefix over the wave totals plus a running ballot prefix gives
// each kept token its output slot; keys equal to tau are admitted in token order
// until the budget k is met.
//
// Four launch shapes:
//  - one workgroup of 1024 lanes per head, its keys in registers (up to 32 per
//    lane) or, for longer heads, re-read from the L2 in every step;
//  - few heads, or long ones: each head is cut into chunks and three kernels
//    with one workgroup per chunk share the work through the caller's workspace
//    (select_plan below has the rule);
//  - short heads on their way to compaction: several workgroups per head repeat the search and each copies a
//    share of the rows (select_compact_kernel);
//  - the shortest: they compute the norms as well (compress_short_kernel).
#include "digit_search.hpp"
#include "l2kv_device.hpp"
#include "l2kv_host.hpp"
#include "row_norm.hpp"

#include <type_traits>

namespace l2kv {

constexpr int kSelMaxRegKeys = 32;                   // keys per lane held in registers
constexpr int kSelBatch = 8;                         // keys per lane fetched together when they are re-read

// Ordered emit shared by both launch shapes.  Every wave of the workgroup owns `iters` * 64
// consecutive positions of [t0, ...); fetch(e) is this lane's key of iteration e (positions past
// the end read as the largest key and come after every real one).  lt_before / eq_before: keys
// below / equal to tau ahead of this workgroup's range.  put(i, t): token t is the i-th kept one.  A wave whose tokens
// would go beyond `limit` of them emits none (kLimited: the counts come from the caller's memory).
struct EmitShared { uint32_t lt[kSelWaves], eq[kSelWaves]; };

template <int kUnroll, bool kLimited, typename Fetch, typename Put>
__device__ __forceinline__ void emit_ordered(Fetch fetch, int64_t iters, uint32_t t0, uint32_t tau, uint32_t need_eq,
                                             uint32_t lt_before, uint32_t eq_before, Put put, uint32_t limit, EmitShared& sh) {
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    uint32_t lt_w = 0, eq_w = 0;
    for (int64_t e0 = 0; e0 < iters; e0 += kUnroll) {
        uint32_t key[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) key[u] = fetch(e0 + u);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            lt_w += __popcll(__ballot(key[u] < tau));
            eq_w += __popcll(__ballot(key[u] == tau));
        }
    }
    if (lane == 0) {
        sh.lt[wave] = lt_w;
        sh.eq[wave] = eq_w;
    }
    __syncthreads();
    lt_before += sum_before(sh.lt, wave);
    eq_before += sum_before(sh.eq, wave);
    uint32_t out_base = lt_before + (eq_before < need_eq ? eq_before : need_eq);
    auto for_iters = [&](auto&& body) {
        for (int64_t e0 = 0; e0 < iters; e0 += kUnroll) {
            uint32_t key[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) key[u] = fetch(e0 + u);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) body(key[u], (int32_t)(t0 + (uint32_t)(e0 + u) * kWaveSize + lane));
        }
    };
    const bool all_eq = eq_w != 0 && eq_before + eq_w <= need_eq;         // every tie of this wave's range is kept
    if constexpr (kLimited) {
        const uint32_t left = eq_before < need_eq ? need_eq - eq_before : 0u;
        if ((uint64_t)out_base + lt_w + (eq_w < left ? eq_w : left) > limit) return;
    }
    if (all_eq || eq_w == 0 || eq_before >= need_eq) {
        // ... or none is: one comparison per key.  (Padding equals tau only if tau is the largest
        // key; a range with padding then never has all its ties kept, need_eq counts real keys.)
        if (lt_w == 0 && !all_eq) return;
        uint32_t highest = all_eq ? tau : tau - 1;       // tau > 0 where some key is below it
        asm volatile("" : "+v"(highest));                  // compare afresh: the masks of the tally would not stay in registers
        for_iters([&](uint32_t key, int32_t t) {
            const bool keep = key <= highest;
            const uint64_t keep_mask = __ballot(keep);
            if (keep) put(out_base + lanes_below(keep_mask), t);
            out_base += __popcll(keep_mask);
        });
    } else {
        // the wave in whose range the last kept tie lies
        uint32_t eq_base = eq_before;
        for_iters([&](uint32_t key, int32_t t) {
            const bool is_eq = key == tau;
            const uint64_t eq_mask = __ballot(is_eq);
            const bool keep = key < tau || (is_eq && (eq_base + lanes_below(eq_mask)) < need_eq);
            const uint64_t keep_mask = __ballot(keep);
            if (keep) put(out_base + lanes_below(keep_mask), t);
            out_base += __popcll(keep_mask);
            eq_base += __popcll(eq_mask);
        });
    }
}

// ---- one workgroup per head ---------------------------------------------------------------
// E > 0 : keys of the head fit E per lane and are cached in registers.
// E == 0: streaming variant, keys are re-read from memory (L2) in every pass.
template <int E> struct HeadKeys {
    const uint32_t* src;
    uint32_t T, flip, t0;                 // t0: first token of the wave's range
    int64_t iters;
    uint32_t regs[E > 0 ? E : 1];
    // Wave w owns tokens [w*span, (w+1)*span), span a multiple of 64; iteration
    // e of lane l looks at token w*span + e*64 + l.
    __device__ __forceinline__ HeadKeys(const uint32_t* s, int64_t count, uint32_t f) : src(s), T((uint32_t)count), flip(f) {
        iters = E > 0 ? E : ((count + (int64_t)kSelThreads * kSelBatch - 1) / ((int64_t)kSelThreads * kSelBatch) * kSelBatch);
        t0 = (uint32_t)(threadIdx.x / kWaveSize * iters * kWaveSize);     // T < 2^31 and the padded range ends below T + 2^14
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) regs[e] = fetch_mem(e);
        }
    }
    __device__ __forceinline__ uint32_t token(int64_t e) const { return t0 + (uint32_t)e * kWaveSize + threadIdx.x % kWaveSize; }
    // Branch-free: positions past the end re-read the last key (in bounds) and
    // are replaced by the largest key, which is never "below" anything.  Such
    // padding sits after every real token, so in the ordered emit it is reached
    // only after all real keys equal to tau, when the budget is already met.
    __device__ __forceinline__ uint32_t fetch_mem(int64_t e) const {
        const uint32_t t = token(e);
        const uint32_t v = src[t < T ? t : T - 1] ^ flip;
        return t < T ? v : 0xffffffffu;
    }
    __device__ __forceinline__ uint32_t fetch(int64_t e) const {
        if constexpr (E > 0) return regs[e];
        else return fetch_mem(e);
    }
    // body(key, real) for every key once, in batches whose loads are issued together
    template <typename F> __device__ __forceinline__ void each(F&& body) const {
        if constexpr (E > 0) {
            uint32_t left = T - token(0);                     // negative past the end; fresh masks in every pass
            asm volatile("" : "+v"(left));
#pragma unroll
            for (int e = 0; e < E; ++e) body(regs[e], (int32_t)left > e * kWaveSize);
        } else {
            for (int64_t e0 = 0; e0 < iters; e0 += kSelBatch) {
                uint32_t key[kSelBatch];
#pragma unroll
                for (int u = 0; u < kSelBatch; ++u) key[u] = fetch_mem(e0 + u);
#pragma unroll
                for (int u = 0; u < kSelBatch; ++u) body(key[u], token(e0 + u) < T);
            }
        }
    }
};

constexpr uint32_t kListedKeys = 256;                 // keys of a bin that are compared with each other
constexpr uint32_t kFewListed = 8;                    // by every wave for itself (35 so: 2 us more than through LDS)
// Heads of at most 2048 tokens are counted in half as many bins: 32 KB to clear and to sum up, and a bin holds a few keys all the same.  One-launch
// compressions of 512 tokens 6.85 -> 6.27 us, of 128 5.88 -> 5.25, of 8 heads of 2048 in two launches 9.15 -> 8.80, together with the comparison by
// every wave.  (In 1024 bins a zero row, which makes the bins wide, costs heads of 1000 more than that gains: 7.74 -> 8.06, here 7.35;
// for the same reason not up to 4096 tokens: 512 heads 8.2 -> 7.5, with a zero row each 10.0 -> 11.8.)
constexpr int kFewBits = 11;
struct SearchShared {
    uint32_t hist[kTopBins * kCopies];                // 64 KB: two workgroups per compute unit
    uint32_t list[kListedKeys];
    uint32_t lo[kSelWaves], hi[kSelWaves];
    FindShared find;
    uint32_t listed, tau, need_eq;
};
struct Threshold { uint32_t tau, need_eq; };          // need_eq >= 1 keys equal to tau are kept, lowest tokens first

// The k-th smallest of a head's keys, 1 <= k <= their number.  Called by all 1024 lanes.
template <int E>
__device__ __forceinline__ Threshold find_threshold(const HeadKeys<E>& keys, uint32_t k, SearchShared& sh) {
    constexpr int kBits = E == 1 || E == 2 ? kFewBits : kTopBits;
    constexpr uint32_t kBins = 1u << kBits;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    uint32_t lo = 0xffffffffu, hi = 0u;
    keys.each([&](uint32_t key, bool real) {
        lo = key < lo ? key : lo;                     // the padding is the largest key
        hi = real && key > hi ? key : hi;
    });
    lo = wave_min(lo);
    hi = ~wave_min(~hi);
    if (lane == 0) {
        sh.lo[wave] = lo;
        sh.hi[wave] = hi;
    }
    if (threadIdx.x == 0) sh.listed = 0;
    clear_counts(sh.hist, kBins * kCopies);
    __syncthreads();
    lo = __builtin_amdgcn_readfirstlane(row16_min(sh.lo[lane % kRowLanes]));
    hi = ~__builtin_amdgcn_readfirstlane(row16_min(~sh.hi[lane % kRowLanes]));
    // every pass computes the bins afresh: kept from one pass to the next they would not fit the registers
    auto origin = [&] { uint32_t v = lo; asm volatile("" : "+s"(v)); return v; };
    const int bits = hi == lo ? 0 : 32 - __builtin_clz(hi - lo);
    int shift = bits > kBits ? bits - kBits : 0;
    // (the padding falls into the last bin: it comes after all real keys and k is at most their number)
    uint32_t o = origin();
    keys.each([&](uint32_t key, bool) {
        const uint32_t b = (key - o) >> shift;
        count_digit(sh.hist, b < kBins ? b : kBins - 1);
    });
    __syncthreads();
    Found f = find_digit<kBins>(sh.hist, k, sh.find);
    uint32_t want = k - f.below;
    uint32_t bin = __builtin_amdgcn_readfirstlane(f.digit);           // (key - lo) >> shift of the wanted key
    uint32_t count = __builtin_amdgcn_readfirstlane(f.count);
    while (shift > 0 && count > kListedKeys) {
        const int finer = shift > kBits ? shift - kBits : 0;
        clear_counts(sh.hist, kBins * kCopies);
        __syncthreads();
        o = origin();
        keys.each([&](uint32_t key, bool) {
            if ((key - o) >> shift == bin) count_digit(sh.hist, ((key - o) >> finer) - (bin << (shift - finer)));
        });
        __syncthreads();
        f = find_digit<kBins>(sh.hist, want, sh.find);
        want -= f.below;
        bin = (bin << (shift - finer)) + __builtin_amdgcn_readfirstlane(f.digit);
        count = __builtin_amdgcn_readfirstlane(f.count);
        shift = finer;
    }
    if (shift == 0) return Threshold{lo + bin, want};                 // one key per bin
    o = origin();
    keys.each([&](uint32_t key, bool) {
        if ((key - o) >> shift == bin) sh.list[atomicAdd(&sh.listed, 1u)] = key;
    });
    __syncthreads();
    count = __builtin_amdgcn_readfirstlane(sh.listed);                // without padding that was counted with the last bin
    if (count <= kFewListed) {
        // every wave by itself, lane i with the i-th of them: no barrier, and nothing through LDS
        const uint32_t key = sh.list[(uint32_t)lane < count ? lane : 0];
        uint32_t less = 0, equal = 0;
        for (uint32_t j = 0; j < count; ++j) {
            const uint32_t other = __builtin_amdgcn_readlane((int)key, (int)j);
            less += other < key ? 1u : 0u;
            equal += other == key ? 1u : 0u;
        }
        const uint64_t wanted = __ballot((uint32_t)lane < count && less < want && want <= less + equal);      // and its equals
        const int at = (int)__builtin_ctzll(wanted | 1ull << (kWaveSize - 1));
        return Threshold{(uint32_t)__builtin_amdgcn_readlane((int)key, at), want - (uint32_t)__builtin_amdgcn_readlane((int)less, at)};
    }
    // four lanes to a key, each for a quarter of the others
    static_assert(kListedKeys * 4 == kSelThreads, "all of them at once");
    if (threadIdx.x / 4 < count) {
        const uint32_t key = sh.list[threadIdx.x / 4];
        uint32_t less = 0, equal = 0;
        constexpr uint32_t kTogether = 4;                             // reads on their way at a time: one by one a full list takes 1.2 us more
        const uint32_t whole = count - count % (4 * kTogether);
        for (uint32_t j0 = threadIdx.x % 4; j0 < whole; j0 += 4 * kTogether) {
            uint32_t other[kTogether];
#pragma unroll
            for (uint32_t u = 0; u < kTogether; ++u) other[u] = sh.list[j0 + 4 * u];
#pragma unroll
            for (uint32_t u = 0; u < kTogether; ++u) {
                less += other[u] < key ? 1u : 0u;
                equal += other[u] == key ? 1u : 0u;
            }
        }
        for (uint32_t j = whole + threadIdx.x % 4; j < count; j += 4) {
            const uint32_t other = sh.list[j];
            less += other < key ? 1u : 0u;
            equal += other == key ? 1u : 0u;
        }
        less = dpp_add<kDppXor2>(dpp_add<kDppXor1>(less));           // the lanes of a quad are here together
        equal = dpp_add<kDppXor2>(dpp_add<kDppXor1>(equal));
        if (less < want && want <= less + equal) {                    // the wanted key, and its equals alike
            sh.tau = key;
            sh.need_eq = want - less;
        }
    }
    __syncthreads();
    return Threshold{sh.tau, sh.need_eq};
}

// Ragged batches: [n_planes][total_in] norms, sequence s at in_off[s]..in_off[s+1];
// its kept positions (relative to the sequence start) go to
// [n_planes][total_out] at out_off[s]..out_off[s+1].  in_off == NULL: uniform.
struct RaggedSelect {
    const int64_t* in_off;
    const int64_t* out_off;
    int64_t n_seq, total_in, total_out;
};

template <int E>
__global__ __launch_bounds__(kSelThreads)
void select_kernel(const uint32_t* __restrict__ norm_bits, int64_t T, uint32_t k, uint32_t flip,
                   int32_t* __restrict__ kept_idx, int32_t* __restrict__ kept_count,
                   RaggedSelect rag) {
    __shared__ __attribute__((aligned(16))) SearchShared s_search;
    __shared__ EmitShared s_emit;

    const int64_t head = blockIdx.x;
    const uint32_t* src = norm_bits + head * T;
    int32_t* out = kept_idx + head * (int64_t)k;
    if (rag.in_off != nullptr) {
        // ragged batch: block = (plane, sequence); sizes and places come from the offset arrays
        const int64_t plane = (uint32_t)head / (uint32_t)rag.n_seq;
        const int64_t seq = (uint32_t)head % (uint32_t)rag.n_seq;
        const Range in = clamped_range(rag.in_off, seq, rag.total_in);
        const Range outr = clamped_range(rag.out_off, seq, rag.total_out);
        T = in.count;
        // the register variants see the first 1024 * E tokens (the caller's bound on the lengths)
        if (E > 0 && T > (int64_t)E * kSelThreads) T = (int64_t)E * kSelThreads;
        const int64_t kk = outr.count;
        if (T <= 0 || kk <= 0) return;                       // whole workgroup: nothing to select
        k = (uint32_t)(kk < T ? kk : T);                     // never more than there are
        src = norm_bits + plane * rag.total_in + in.first;
        out = kept_idx + plane * rag.total_out + outr.first;
    }
    const HeadKeys<E> keys(src, T, flip);
    const Threshold th = find_threshold(keys, k, s_search);
    emit_ordered<E == 0 ? kSelBatch : E, false>([&](int64_t e) { return keys.fetch(e); }, E == 0 ? keys.iters : E, keys.t0, th.tau,
                                         th.need_eq, 0u, 0u, [&](uint32_t i, int32_t t) { out[i] = t; }, k, s_emit);
    if (kept_count != nullptr && threadIdx.x == 0) kept_count[head] = (int32_t)k;
}

// ---- selection and compaction of short heads in one launch ------------------------------------
// The rows of a head are shared by gridDim.x workgroups.  Each finds the threshold by itself (the keys of a
// short head are a few per lane, so repeating the search costs less than the launch and the round trip
// through memory that a search of its own takes), writes its share of the indices and copies
// its share of the rows.
// The search (about 6 us with two workgroups on a compute unit) is a chain of LDS round trips during which the memory is idle.
// So a share is a stretch of tokens where that can be: the rows of V it may need are requested ahead of the search and wait in
// registers, kept or not, and only the kept rows of K, which the norm pass has just read, are left to fetch.  With the norm
// pass, other inputs in every call, us, three kernels / shares of kept rows / of tokens: half of 8 heads of 2k 14.1, 12.4,
// 9.8, of 32 heads of 4k 26.0, 25.3, 21.7 (0.9 of them 34.4 in three kernels, 27.5), of 8 heads of 8k 18.6, 17.4, 16.4, of 100 heads of
// 1k of 64 elements -, 15.9, 13.4.  Kept tokens all in one stretch, and so all rows of some shares and none of others, 32 heads of 4k: 24.9, 21.2.
constexpr int kFuseMaxTokens = 8 * kSelThreads;
constexpr int kFuseMaxHeads = 256;
constexpr int kDies = 8;                               // compute dies, 32 compute units each
constexpr int64_t kFuseMaxBytes = int64_t{20} << 20, kShortHeadBytes = int64_t{128} << 10, kShortHeadBytesF32 = int64_t{192} << 10;
constexpr int kShortManyHeads = 4;
constexpr int kFuseRows = 4096;                       // most rows of a share: indices in LDS as 16-bit numbers
static_assert(kFuseMaxTokens <= 65536, "token indices fit 16 bits");

struct FuseShared {
    SearchShared search;
    EmitShared emit;
    uint16_t row[kFuseRows];
};

// Rows [r0, r0 + rows) of the kept rows of a head: selection by all lanes, indices, copy of K and V.  K, V, out, Kc,
// Vc point at the head.
template <int E, int kRowBytes>
__device__ __forceinline__ void select_and_copy(const HeadKeys<E>& keys, uint32_t k, uint32_t r0, uint32_t rows,
                                                const char* __restrict__ K, const char* __restrict__ V, int32_t* __restrict__ out,
                                                char* __restrict__ Kc, char* __restrict__ Vc, FuseShared& sh) {
    const Threshold th = find_threshold(keys, k, sh.search);
    emit_ordered<E, false>([&](int64_t e) { return keys.fetch(e); }, E, keys.t0, th.tau, th.need_eq, 0u, 0u,
                    [&](uint32_t i, int32_t t) {
                        if (i - r0 < rows) {
                            sh.row[i - r0] = (uint16_t)t;
                            out[i] = t;
                        }
                    }, k, sh.emit);
    __syncthreads();
    using P = RowCopy<kRowBytes>;
    constexpr uint32_t kRowsPerStep = kSelThreads / P::kLanes;
    constexpr int kUnroll = 2;
    const uint32_t c = threadIdx.x % P::kLanes, rg = threadIdx.x / P::kLanes;
    for (uint32_t base = 0; base < rows; base += kRowsPerStep * kUnroll) {
        Words<P::kWords> a[kUnroll], b[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t r = base + u * kRowsPerStep + rg;
            const int64_t from = sh.row[r < rows ? r : rows - 1] * (int64_t)kRowBytes + c * 16;
            a[u] = load_words_stream<P::kWords, P::kStride>(K + from);
            b[u] = load_words_stream<P::kWords, P::kStride>(V + from);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t r = base + u * kRowsPerStep + rg;
            const int64_t to = (r0 + (int64_t)r) * kRowBytes + c * 16;
            if (r < rows) {
                store_words_stream<P::kWords, P::kStride>(Kc + to, a[u]);
                store_words_stream<P::kWords, P::kStride>(Vc + to, b[u]);
            }
        }
    }
}

// Rows of V on their way to registers while the search runs.  16 registers: with the keys and what the search takes, 60 of the 64
// that two workgroups on a compute unit leave a lane.  (Spilled, they are waited for before the search: 28.8 us in place of 21.7.)
template <int kRowBytes> struct RowsAhead {
    using P = RowCopy<kRowBytes>;
    static constexpr uint32_t kRowsPerStep = kSelThreads / P::kLanes;
    static constexpr int kSteps = kRowBytes > 256 ? 2 : 4;                          // 16 registers
    static constexpr uint32_t kTokens = kRowsPerStep * kSteps;                      // most tokens of a share
    Words<P::kWords> row[kSteps];
    // V points at the first token of the share
    __device__ __forceinline__ void load(const char* __restrict__ V, uint32_t tokens) {
        const uint32_t c = threadIdx.x % P::kLanes, rg = threadIdx.x / P::kLanes;
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const uint32_t r = u * kRowsPerStep + rg;
            row[u] = load_words_stream<P::kWords, P::kStride>(V + (r < tokens ? r : tokens - 1) * (int64_t)kRowBytes + c * 16);
        }
    }
};

constexpr uint16_t kDropped = 0xffff;
static_assert(kFuseMaxTokens < kDropped && RowsAhead<128>::kTokens <= kSelThreads && RowsAhead<128>::kTokens <= kFuseRows, "places of a share");
// Tokens [t0, t0 + tokens) of a head, whose rows of V are in `ahead`.  K, out, Kc, Vc point at the head.
template <int E, int kRowBytes>
__device__ __forceinline__ void select_and_copy_ahead(const HeadKeys<E>& keys, uint32_t k, uint32_t t0, uint32_t tokens,
                                                      const RowsAhead<kRowBytes>& ahead, const char* __restrict__ K,
                                                      int32_t* __restrict__ out, char* __restrict__ Kc, char* __restrict__ Vc,
                                                      FuseShared& sh) {
    using A = RowsAhead<kRowBytes>;
    using P = typename A::P;
    if (threadIdx.x < A::kTokens) sh.row[threadIdx.x] = kDropped;
    const Threshold th = find_threshold(keys, k, sh.search);
    emit_ordered<E, false>([&](int64_t e) { return keys.fetch(e); }, E, keys.t0, th.tau, th.need_eq, 0u, 0u,
                    [&](uint32_t i, int32_t t) {
                        if ((uint32_t)t - t0 < tokens) {
                            sh.row[(uint32_t)t - t0] = (uint16_t)i;
                            out[i] = t;
                        }
                    }, k, sh.emit);
    __syncthreads();
    uint32_t at_lane = threadIdx.x;
    asm volatile("" : "+v"(at_lane));                                // afresh: places kept from the loads on would not fit the registers
    const uint32_t c = at_lane % P::kLanes, rg = at_lane / P::kLanes;
    Words<P::kWords> key_row[A::kSteps];
    uint32_t to[A::kSteps];
#pragma unroll
    for (int u = 0; u < A::kSteps; ++u) {
        if (kRowBytes == 128 && u * A::kRowsPerStep >= tokens) break;                 // four steps of 128 tokens are seldom full
        const uint32_t r = u * A::kRowsPerStep + rg;
        to[u] = sh.row[r];                                            // past the share: dropped
        if (to[u] != kDropped) key_row[u] = load_words_stream<P::kWords, P::kStride>(K + (t0 + r) * (int64_t)kRowBytes + c * 16);
    }
#pragma unroll
    for (int u = 0; u < A::kSteps; ++u) {
        if (kRowBytes == 128 && u * A::kRowsPerStep >= tokens) break;                 // four steps of 128 tokens are seldom full
        if (to[u] != kDropped) {
            const int64_t at = to[u] * (int64_t)kRowBytes + c * 16;
            store_words_stream<P::kWords, P::kStride>(Vc + at, ahead.row[u]);
            store_words_stream<P::kWords, P::kStride>(Kc + at, key_row[u]);
        }
    }
}

// kAhead: share = `per_share` tokens of a head, else as many of its kept rows.
template <int E, int kRowBytes, bool kAhead>
__global__ __launch_bounds__(kSelThreads, kAhead && E <= 4 ? 8 : 4)
void select_compact_kernel(const uint32_t* __restrict__ norm_bits, int64_t T, uint32_t k, uint32_t per_share,
                           const char* __restrict__ K, const char* __restrict__ V, int64_t head_stride_bytes,
                           int32_t* __restrict__ kept_idx, char* __restrict__ Kc, char* __restrict__ Vc) {
    __shared__ __attribute__((aligned(16))) FuseShared sh;
    const int64_t head = blockIdx.y;
    const uint32_t all = kAhead ? (uint32_t)T : k, first = blockIdx.x * per_share;
    if (first >= all) return;
    const uint32_t count = all - first < per_share ? all - first : per_share;
    const HeadKeys<E> keys(norm_bits + head * T, T, 0u);
    const int64_t dense = head * (int64_t)k;
    K += head * head_stride_bytes;
    V += head * head_stride_bytes;
    kept_idx += dense;
    Kc += dense * kRowBytes;
    Vc += dense * kRowBytes;
    if constexpr (kAhead) {
        RowsAhead<kRowBytes> ahead;
        ahead.load(V + first * (int64_t)kRowBytes, count);
        __builtin_amdgcn_sched_barrier(0);                            // not next to their use
        select_and_copy_ahead<E, kRowBytes>(keys, k, first, count, ahead, K, kept_idx, Kc, Vc, sh);
    } else {
        select_and_copy<E, kRowBytes>(keys, k, first, count, K, V, kept_idx, Kc, Vc, sh);
    }
}

// The whole compression of heads of at most 1024 tokens and 128 KB (fp32, four heads and more: 192 KB) in one launch: every
// share also computes all norms of its head (out of the L2 for all but the first reader), the first share writes them.  Bound by the chain of load, sums, search
// and copy of one workgroup.  us, two launches / one: half of 4 heads of 512 tokens 8.2, 7.3, of 64 of 256 9.5, 7.3, of 128 of
// 512 (16 MB) 13.9, 12.4; of 500 tokens of 17 heads 9.0, 7.7, with the shares of a head on all compute dies 9.6.  Not beyond 128 KB of a head,
// which one workgroup goes through before anything else: 16 heads of 1024 tokens 9.5, 10.0, one of them 8.0, 9.1, rows of 512 bytes
// 8.5, 13.8.  Fp32 has half the elements in a byte to go through: 8 heads of 552 tokens of 64 8.5, 7.8, of 374 of 128 9.5, 8.5, 64 of 365
// 13.0, 10.3, but 2 of 689 7.7, 7.6, one of 756 6.9, 7.4, and beyond 192 KB 4 of 418 8.0, 8.9.  However little is kept, although all rows of
// V are loaded: against shares of kept rows in one or two launches, 0.05 kept, 64 heads of 256 8.8, 6.7, 128 of 512 12.7, 12.1; 448
// calls of 1 to 256 heads of 128 to 1000 tokens, 0.05 to all kept, none slower.
template <typename E, int D>
__global__ __launch_bounds__(kSelThreads)
void compress_short_kernel(const char* __restrict__ K, const char* __restrict__ V, uint32_t n_heads, uint32_t shares, int64_t T,
                           uint32_t k, uint32_t tokens_per_share, int64_t head_stride_bytes, float* __restrict__ norms,
                           int32_t* __restrict__ kept_idx, char* __restrict__ Kc, char* __restrict__ Vc) {
    using S = Slice<E, D>;
    __shared__ __attribute__((aligned(16))) FuseShared sh;
    __shared__ uint32_t s_norm[kSelThreads];                          // bit patterns
    // Workgroups go to the compute dies round-robin: the shares of a head, which all read the whole of it, to the same one.
    const uint32_t slot = blockIdx.x / kDies, share = slot % shares;
    const int64_t head = slot / shares * kDies + blockIdx.x % kDies;
    const uint32_t n = (uint32_t)T, first = share * tokens_per_share;
    if (head >= n_heads || first >= n) return;
    const char* Kh = K + head * head_stride_bytes;
    const int c = threadIdx.x % kRowLanes;
    constexpr uint32_t kGroups = kSelThreads / kRowLanes;            // 64 row groups
    // kRows rows (pairs of the short ones, 8 lanes each) per row group, all requested before the first is summed
    auto sums = [&](auto batch) {
        constexpr int kRows = decltype(batch)::value;
        using P = Pieces<S::kWords>;
        constexpr bool kPairs = S::kRowBytes == 128;
        constexpr uint32_t kStep = kPairs ? 2 * kGroups : kGroups;
        const uint32_t mine = kPairs ? 2 * (threadIdx.x / kRowLanes) + c / 8 : threadIdx.x / kRowLanes;
        for (uint32_t base = 0; base < n; base += kStep * kRows) {
            Words<kPairs ? 4 : S::kWords> raw[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const uint32_t row = base + u * kStep + mine;
                const char* const from = Kh + (row < n ? row : n - 1) * (int64_t)S::kRowBytes;
                if constexpr (kPairs) raw[u] = load_words<4>(from + (c % 8) * 16);
                else raw[u] = load_words<S::kWords, P::kStride>(from + c * P::kBytes);
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const uint32_t row = base + u * kStep + mine;
                float v;
                if constexpr (kPairs) {
                    v = row_pair_sum_of_squares(raw[u]);
                } else {
                    float x[S::kElems];
                    widen<E, D>(raw[u], x);
                    v = chunked_sum_of_squares<E, D>(x);
                }
                if ((kPairs ? c % 8 : c) == 0 && row < n) s_norm[row] = __builtin_bit_cast(uint32_t, v);
            }
        }
    };
    // twice the rows where that saves a round trip, not where it only adds sums of rows that are not there: 512 rows of
    // 256 bytes 7.6 us, not 8.0, but 80 rows 7.6, not 6.9 (fp32 rows slower throughout: 512 of 256 bytes 7.9, not 7.6)
    constexpr int kBatch = S::kWords > 4 ? 2 : 4;
    constexpr uint32_t kBatchRows = kBatch * (S::kRowBytes == 128 ? 2 * kGroups : kGroups);
    if (E::kBytes == 2 && n > kBatchRows) sums(std::integral_constant<int, 2 * kBatch>());
    else sums(std::integral_constant<int, kBatch>());
    const uint32_t count = n - first < tokens_per_share ? n - first : tokens_per_share;
    RowsAhead<S::kRowBytes> ahead;
    ahead.load(V + head * head_stride_bytes + first * (int64_t)S::kRowBytes, count);
    __builtin_amdgcn_sched_barrier(0);                                // not next to their use
    __syncthreads();
    if (share == 0 && threadIdx.x < n) norms[head * T + threadIdx.x] = __builtin_bit_cast(float, s_norm[threadIdx.x]);
    const HeadKeys<1> keys(s_norm, T, 0u);
    const int64_t dense = head * (int64_t)k;
    select_and_copy_ahead<1, S::kRowBytes>(keys, k, first, count, ahead, Kh, kept_idx + dense, Kc + dense * S::kRowBytes,
                                           Vc + dense * S::kRowBytes, sh);
}

// ---- several workgroups per head -------------------------------------------------------------
// chunk c of a head = tokens [c * chunk, (c+1) * chunk).  Three kernels, ordered by the stream:
//   select_count_kernel   histogram of the top digit per chunk (64 coarse counts beside the 4096)
//   select_gather_kernel  the digit of tau; keys of that digit go to the candidate list of the
//                         head, in chunk order; per chunk the counts below it and in it
//   select_emit_kernel    every workgroup finishes the search over the candidates by itself (3 % of log-normal
//                         norms, a third of the norms of rows without a scale of their own; all of them in the
//                         worst case), counts what lies ahead of its chunk and emits its kept tokens
// Counts and lists pass from kernel to kernel through the caller's memory (SelectScratch).  No access is bounded by what is read there
// alone: if two calls overlap on one workspace, against the contract, they select wrong rows and nothing worse.
constexpr int kCoarse = 64;                          // coarse counts per chunk, of kTopBins / 64 digits each
constexpr int kFinePerCoarse = kTopBins / kCoarse;   // 64
constexpr int kChunkUnit = kSelThreads * 4;          // chunks are multiples of 4096 tokens
constexpr int64_t kChunk16 = 8 * kChunkUnit;         // up to here the counts of a chunk are 16-bit numbers

struct SelectSplit {
    void* fine;           // [heads][chunks][kTopBins], 16-bit numbers while the chunks are short, else 32-bit ones
    uint32_t* coarse;     // [heads][chunks][kCoarse]
    uint2* info;          // [heads][chunks]: keys below the digit of tau, keys in it
    uint32_t* head_info;  // [heads][2]: digit of tau, keys below it in the head
    uint32_t* cand;       // [heads][T]
    int64_t chunk;        // tokens per chunk
    int32_t chunks;       // per head
};

struct SelectPlan {
    int64_t chunk = 0;    // 0: one workgroup per head
    int32_t chunks = 0;
    size_t counts = 256, list = 0;    // bytes of scratch memory
};

static size_t round256(size_t n) { return (n + 255) / 256 * 256; }
static size_t count_bytes(int64_t chunk) { return chunk <= kChunk16 ? sizeof(uint16_t) : sizeof(uint32_t); }

// Heads that fit the registers of one workgroup (32k tokens) are never split: 8 heads of 32k take
// 15.5 us either way, more heads are faster whole.  Longer ones are split while the heads alone
// leave most of the chip idle, into as many chunks as run at once in all: every one goes over the candidates of the
// whole head, which are all keys where all are equal, so that their number must not grow with the length
// (with chunks of at most 32k keys 64 heads of 4M took 1.8 ms, 58 for equal keys).  us, one workgroup per head / split:
//                  log-normal norms   normal, no scale   30 % zero, 30 % kept   all equal
//   8 of 131k           59 / 17           59 / 22             87 / 38            64 / 92
//   64 of 131k          65 / 39           64 / 51             90 / 72            68 / 177
//   64 of 262k         158 / 68          156 / 91            183 / 132          136 / 344
//   8 of 1M            549 / 54          546 / 108           674 / 339          488 / 1102
//   64 of 1M           654 / 267         656 / 354           722 / 500          551 / 1352
//   4 of 4M           2396 / 126        2438 / 331          2790 / 796         2095 / 4206
//   64 of 4M          3285 / 1117       3296 / 1483         3450 / 2054        2562 / 5447
// and log-normal 8 of 40k 22.9 / 16.1, 64 of 40k 23.9 / 28.6, 128 of 131k 80 / 69 (not split: 112 / 199 for equal keys).
static SelectPlan select_plan(int64_t n_heads, int64_t T) {
    SelectPlan p;
    constexpr int64_t kWorkgroups = 512;             // two per compute unit
    if (T <= (int64_t)kSelThreads * kSelMaxRegKeys || T > (int64_t{1} << 22)) return p;
    if (n_heads > 64 || n_heads > T / 2048) return p;
    const int64_t want = (kWorkgroups + n_heads - 1) / n_heads;
    const int64_t chunk = ((T + want - 1) / want + kChunkUnit - 1) / kChunkUnit * kChunkUnit;
    p.chunk = chunk;
    p.chunks = (int32_t)((T + chunk - 1) / chunk);
    const size_t n = (size_t)n_heads * (size_t)p.chunks;
    p.counts = round256(n * kTopBins * count_bytes(chunk)) + round256(n * kCoarse * sizeof(uint32_t)) +
               round256(n * sizeof(uint2)) + round256((size_t)n_heads * 2 * sizeof(uint32_t));
    p.list = round256((size_t)n_heads * (size_t)T * sizeof(uint32_t));
    return p;
}

template <typename Count>
__global__ __launch_bounds__(kSelThreads)
void select_count_kernel(const uint32_t* __restrict__ norm_bits, int64_t T, uint32_t flip, SelectSplit sp) {
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kTopBins * kCopies];
    const int64_t head = blockIdx.y;
    const int64_t slot = head * sp.chunks + blockIdx.x;
    const uint32_t* src = norm_bits + head * T;
    const int64_t first = blockIdx.x * sp.chunk;
    const int64_t last = first + sp.chunk < T ? first + sp.chunk : T;
    clear_counts(s_hist, kTopBins * kCopies);
    __syncthreads();
    for (int64_t base = first; base < last; base += kChunkUnit) {
        uint32_t key[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t t = base + u * kSelThreads + threadIdx.x;
            key[u] = src[t < last ? t : last - 1] ^ flip;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (base + u * kSelThreads + threadIdx.x < last) count_digit(s_hist, key[u] >> (32 - kTopBits));
    }
    __syncthreads();
    // lane i: digits 4i .. 4i+3; 16 lanes make up one coarse count
    uint4 c;
    c.x = digit_count(s_hist, 4 * threadIdx.x);
    c.y = digit_count(s_hist, 4 * threadIdx.x + 1);
    c.z = digit_count(s_hist, 4 * threadIdx.x + 2);
    c.w = digit_count(s_hist, 4 * threadIdx.x + 3);
    Count* const fine = static_cast<Count*>(sp.fine) + slot * kTopBins;
    if constexpr (sizeof(Count) == 2) reinterpret_cast<uint2*>(fine)[threadIdx.x] = make_uint2(c.x | (c.y << 16), c.z | (c.w << 16));
    else reinterpret_cast<uint4*>(fine)[threadIdx.x] = c;
    uint32_t sum = c.x + c.y + c.z + c.w;
#pragma unroll
    for (int off = kFinePerCoarse / 8; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (threadIdx.x % (kFinePerCoarse / 4) == 0) sp.coarse[slot * kCoarse + threadIdx.x / (kFinePerCoarse / 4)] = sum;
}

// One wave: the lane whose bin holds the want-th key (bins = the lanes' counts in order).
__device__ __forceinline__ Found find_lane(uint32_t count, uint32_t want) {
    const uint32_t incl = wave_inclusive_sum(count);
    const uint64_t past = __ballot(incl >= want);
    const int at = past != 0 ? (int)__builtin_ctzll(past) : kWaveSize - 1;       // want <= total: some lane qualifies
    return Found{(uint32_t)at, __shfl(incl - count, at), __shfl(count, at)};
}

template <typename Count>
__global__ __launch_bounds__(kSelThreads)
void select_gather_kernel(const uint32_t* __restrict__ norm_bits, int64_t T, uint32_t k, uint32_t flip, SelectSplit sp) {
    __shared__ uint32_t s_sum[2][kSelWaves][kCoarse], s_part[kSelWaves][kFinePerCoarse];
    __shared__ uint32_t s_lt, s_n;
    const int64_t head = blockIdx.y;
    const int64_t slot0 = head * sp.chunks;
    const int64_t slot = slot0 + blockIdx.x;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    // the digit of tau: coarse counts of all chunks, then the 64 digits of the coarse count that
    // holds the k-th key; the waves share the chunks and every wave ends with the same result
    uint32_t n = 0;
#pragma unroll 4
    for (int c = wave; c < sp.chunks; c += kSelWaves) n += sp.coarse[(slot0 + c) * kCoarse + lane];
    s_sum[0][wave][lane] = n;
    if (threadIdx.x == 0) {
        s_lt = 0;
        s_n = 0;
    }
    __syncthreads();
    n = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) n += s_sum[0][w][lane];
    const Found g = find_lane(n, k);
    uint32_t m = 0, part = 0;
#pragma unroll 4
    for (int c = wave; c < sp.chunks; c += kSelWaves) {
        const uint32_t v = static_cast<const Count*>(sp.fine)[(slot0 + c) * kTopBins + g.digit * kFinePerCoarse + lane];
        m += v;
        part += c < (int)blockIdx.x ? v : 0u;
    }
    s_sum[1][wave][lane] = m;
    s_part[wave][lane] = part;
    __syncthreads();
    m = part = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        m += s_sum[1][w][lane];
        part += s_part[w][lane];
    }
    const Found f = find_lane(m, k - g.below);
    // candidates of earlier chunks, which come first: no more than those chunks have keys
    const uint32_t before = (uint32_t)(blockIdx.x * sp.chunk), listed = __shfl(part, (int)f.digit);
    const uint32_t ahead = listed < before ? listed : before;
    const uint32_t digit = g.digit * kFinePerCoarse + f.digit;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sp.head_info[2 * head] = digit;
        sp.head_info[2 * head + 1] = g.below + f.below;
    }
    uint32_t* cand = sp.cand + head * T + ahead;
    const uint32_t* src = norm_bits + head * T;
    const int64_t first = blockIdx.x * sp.chunk;
    const int64_t last = first + sp.chunk < T ? first + sp.chunk : T;
    uint32_t lt = 0;
    for (int64_t base = first; base < last; base += kChunkUnit) {
        uint32_t key[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t t = base + u * kSelThreads + threadIdx.x;
            key[u] = src[t < last ? t : last - 1] ^ flip;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool real = base + u * kSelThreads + threadIdx.x < last;
            const uint32_t d = key[u] >> (32 - kTopBits);
            lt += __popcll(__ballot(real && d < digit));
            const uint64_t in = __ballot(real && d == digit);
            uint32_t at = 0;
            if (in != 0 && lane == 0) at = atomicAdd(&s_n, (uint32_t)__popcll(in));
            at = __builtin_amdgcn_readfirstlane(at);
            // order inside the chunk's stretch of the list does not matter: only counts are taken from it
            if (real && d == digit) cand[at + lanes_below(in)] = key[u];
        }
    }
    if (lane == 0) atomicAdd(&s_lt, lt);
    __syncthreads();
    if (threadIdx.x == 0) sp.info[slot] = make_uint2(s_lt, s_n);
}

__global__ __launch_bounds__(kSelThreads)
void select_emit_kernel(const uint32_t* __restrict__ norm_bits, int64_t T, uint32_t k, uint32_t flip,
                        int32_t* __restrict__ kept_idx, int32_t* __restrict__ kept_count, SelectSplit sp) {
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[(kMidBins + kLowBins) * kCopies];
    __shared__ FindShared s_find;
    __shared__ EmitShared s_emit;
    __shared__ uint32_t s_lt_ahead, s_cand_ahead, s_cands, s_cand_lt, s_cand_eq;
    const int64_t head = blockIdx.y;
    const int64_t slot0 = head * sp.chunks;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    uint32_t* const h_mid = s_hist;
    uint32_t* const h_low = s_hist + kMidBins * kCopies;
    clear_counts(s_hist, (kMidBins + kLowBins) * kCopies);
    if (threadIdx.x < kWaveSize) {
        uint32_t lt = 0, ahead = 0, all = 0;
        for (int c = lane; c < sp.chunks; c += kWaveSize) {
            const uint2 v = sp.info[slot0 + c];
            all += v.y;
            lt += c < (int)blockIdx.x ? v.x : 0u;
            ahead += c < (int)blockIdx.x ? v.y : 0u;
        }
#pragma unroll
        for (int off = kWaveSize / 2; off > 0; off >>= 1) {
            lt += __shfl_xor(lt, off);
            ahead += __shfl_xor(ahead, off);
            all += __shfl_xor(all, off);
        }
        if (lane == 0) {
            s_lt_ahead = lt;
            s_cand_ahead = ahead;
            s_cands = all;
            s_cand_lt = 0;
            s_cand_eq = 0;
        }
    }
    const uint32_t top_digit = sp.head_info[2 * head];
    const uint32_t want = k - sp.head_info[2 * head + 1];
    __syncthreads();
    const uint32_t n = s_cands < (uint32_t)T ? s_cands : (uint32_t)T, ahead = s_cand_ahead < n ? s_cand_ahead : n;
    const uint32_t* cand = sp.cand + head * T;
    constexpr int kCandBatch = 4;
    auto for_cands = [&](uint32_t end, auto&& body) {
        for (uint32_t i0 = 0; i0 < end; i0 += kSelThreads * kCandBatch) {
            uint32_t key[kCandBatch];
#pragma unroll
            for (int u = 0; u < kCandBatch; ++u) {
                const uint32_t i = i0 + u * kSelThreads + threadIdx.x;
                key[u] = cand[i < end ? i : end - 1];
            }
#pragma unroll
            for (int u = 0; u < kCandBatch; ++u) body(key[u], i0 + u * kSelThreads + threadIdx.x < end);
        }
    };
    for_cands(n, [&](uint32_t key, bool real) {
        if (real) count_digit(h_mid, (key >> kLowBits) & (kMidBins - 1));
    });
    __syncthreads();
    const Found mid = find_digit<kMidBins>(h_mid, want, s_find);
    const uint32_t prefix = (top_digit << kMidBits) | mid.digit;
    for_cands(n, [&](uint32_t key, bool real) {
        if (real && key >> kLowBits == prefix) count_digit(h_low, key & (kLowBins - 1));
    });
    __syncthreads();
    const Found low = find_digit<kLowBins>(h_low, want - mid.below, s_find);
    const uint32_t tau = (prefix << kLowBits) | low.digit;
    const uint32_t need_eq = want - mid.below - low.below;

    uint32_t lt = 0, eq = 0;
    for_cands(ahead, [&](uint32_t key, bool real) {
        lt += __popcll(__ballot(real && key < tau));
        eq += __popcll(__ballot(real && key == tau));
    });
    if (lane == 0 && (lt | eq)) {
        atomicAdd(&s_cand_lt, lt);
        atomicAdd(&s_cand_eq, eq);
    }
    __syncthreads();
    const uint32_t* src = norm_bits + head * T;
    const int64_t first = blockIdx.x * sp.chunk;
    const int64_t last = first + sp.chunk < T ? first + sp.chunk : T;
    const int64_t iters = sp.chunk / kSelThreads;
    const uint32_t t0 = (uint32_t)(first + wave * iters * kWaveSize);
    const uint32_t end = (uint32_t)last;
    emit_ordered<4, true>(
        [&](int64_t e) -> uint32_t {
            const uint32_t t = t0 + (uint32_t)e * kWaveSize + lane;
            const uint32_t v = src[t < end ? t : end - 1] ^ flip;
            return t < end ? v : 0xffffffffu;
        },
        iters, t0, tau, need_eq, s_lt_ahead + s_cand_lt, s_cand_eq,
        [&](uint32_t i, int32_t t) { kept_idx[head * (int64_t)k + i] = t; }, k, s_emit);
    if (kept_count != nullptr && blockIdx.x == 0 && threadIdx.x == 0) kept_count[head] = (int32_t)k;
}

template <int E>
static void launch_select(const float* norms, int64_t n_heads, int64_t T, int64_t k, uint32_t flip,
                          int32_t* kept_idx, int32_t* kept_count, hipStream_t stream,
                          RaggedSelect rag = RaggedSelect{nullptr, nullptr, 0, 0, 0}) {
    hipLaunchKernelGGL((select_kernel<E>), dim3((unsigned)n_heads), dim3(kSelThreads), 0, stream,
                       reinterpret_cast<const uint32_t*>(norms), T, (uint32_t)k, flip, kept_idx,
                       kept_count, rag);
}

// Picks the kernel variant from the (longest) head length and launches it.
static void launch_select_for_length(int64_t longest, const float* norms, int64_t n_heads, int64_t T,
                                     int64_t k, uint32_t flip, int32_t* kept_idx, int32_t* kept_count,
                                     hipStream_t stream, RaggedSelect rag) {
    const int64_t per_lane = (longest + kSelThreads - 1) / kSelThreads;
    if (per_lane <= 1)       launch_select<1>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
    else if (per_lane <= 2)  launch_select<2>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
    else if (per_lane <= 4)  launch_select<4>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
    else if (per_lane <= 8)  launch_select<8>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
    else if (per_lane <= 16) launch_select<16>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
    else if (per_lane <= kSelMaxRegKeys)
        launch_select<32>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
    else
        launch_select<0>(norms, n_heads, T, k, flip, kept_idx, kept_count, stream, rag);
}

// Keys of the keep-random control (arXiv 2406.11430 Sec. 4, where a random
// subset of the tokens is kept): a counter-based hash of (seed, head, token) written as bit patterns
// into an fp32 array, on which l2kv_select_k then keeps the k lowest.  The hash
// is x = token*0x9E3779B1 + head*0x85EBCA77 + seed followed by the 32-bit
// finalizer of MurmurHash3.
__global__ __launch_bounds__(256)
void random_keys_kernel(int64_t total, int64_t T, uint32_t seed, uint32_t* __restrict__ keys) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const uint32_t head = (uint32_t)(i / T), t = (uint32_t)(i % T);
    uint32_t x = t * 0x9E3779B1u + head * 0x85EBCA77u + seed;
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    keys[i] = x;
}

l2kv_status random_keys_dispatch(int64_t n_heads, int64_t T, uint32_t seed, float* keys, hipStream_t stream) {
    const int64_t total = n_heads * T;
    const int64_t blocks = (total + 255) / 256;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return L2KV_ERR_SHAPE;
    hipLaunchKernelGGL(random_keys_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, total, T, seed,
                       reinterpret_cast<uint32_t*>(keys));
    return launch_status();
}

size_t select_workspace_bytes(int64_t n_heads, int64_t T) {
    const SelectPlan plan = select_plan(n_heads, T);
    return plan.counts + plan.list;
}

SelectScratch select_scratch(void* workspace, size_t bytes, int64_t n_heads, int64_t T) {
    const SelectPlan plan = select_plan(n_heads, T);
    if (bytes < plan.counts + plan.list) return SelectScratch{};
    return SelectScratch{workspace, plan.counts, static_cast<char*>(workspace) + plan.counts, plan.list};
}

l2kv_status select_dispatch(const float* norms, int64_t n_heads, int64_t T, int64_t k,
                            l2kv_mode mode, int32_t* kept_idx, int32_t* kept_count,
                            const SelectScratch& scratch, hipStream_t stream) {
    if (n_heads > 0x7fffffffLL) return L2KV_ERR_SHAPE;
    const uint32_t flip = mode == L2KV_KEEP_HIGHEST ? 0xffffffffu : 0u;
    const SelectPlan plan = select_plan(n_heads, T);
    if (plan.chunk == 0 || scratch.counts_bytes < plan.counts || scratch.list_bytes < plan.list) {
        launch_select_for_length(T, norms, n_heads, T, k, flip, kept_idx, kept_count, stream,
                                 RaggedSelect{nullptr, nullptr, 0, 0, 0});
        return launch_status();
    }
    SelectSplit sp;
    const size_t n = (size_t)n_heads * (size_t)plan.chunks;
    char* ws = static_cast<char*>(scratch.counts);
    sp.fine = ws;
    ws += round256(n * kTopBins * count_bytes(plan.chunk));
    sp.coarse = reinterpret_cast<uint32_t*>(ws);
    ws += round256(n * kCoarse * sizeof(uint32_t));
    sp.info = reinterpret_cast<uint2*>(ws);
    ws += round256(n * sizeof(uint2));
    sp.head_info = reinterpret_cast<uint32_t*>(ws);
    sp.cand = static_cast<uint32_t*>(scratch.list);
    sp.chunk = plan.chunk;
    sp.chunks = plan.chunks;
    const dim3 grid((unsigned)plan.chunks, (unsigned)n_heads);
    const uint32_t* bits = reinterpret_cast<const uint32_t*>(norms);
    const bool short_counts = count_bytes(plan.chunk) == sizeof(uint16_t);
    hipLaunchKernelGGL((short_counts ? select_count_kernel<uint16_t> : select_count_kernel<uint32_t>), grid, dim3(kSelThreads), 0,
                       stream, bits, T, flip, sp);
    hipLaunchKernelGGL((short_counts ? select_gather_kernel<uint16_t> : select_gather_kernel<uint32_t>), grid, dim3(kSelThreads), 0,
                       stream, bits, T, (uint32_t)k, flip, sp);
    hipLaunchKernelGGL(select_emit_kernel, grid, dim3(kSelThreads), 0, stream, bits, T, (uint32_t)k, flip, kept_idx,
                       kept_count, sp);
    return launch_status();
}

template <int E, bool kAhead>
static void launch_select_compact(const dim3 grid, int row_bytes, const float* norms, int64_t T, int64_t k, int64_t per_share,
                                  const void* K, const void* V, int64_t head_stride_bytes, int32_t* kept_idx, void* Kc,
                                  void* Vc, hipStream_t stream) {
    auto kernel = row_bytes == 128 ? select_compact_kernel<E, 128, kAhead>
                  : row_bytes == 256 ? select_compact_kernel<E, 256, kAhead> : select_compact_kernel<E, 512, kAhead>;
    hipLaunchKernelGGL(kernel, grid, dim3(kSelThreads), 0, stream, reinterpret_cast<const uint32_t*>(norms), T, (uint32_t)k,
                       (uint32_t)per_share, static_cast<const char*>(K), static_cast<const char*>(V), head_stride_bytes, kept_idx,
                       static_cast<char*>(Kc), static_cast<char*>(Vc));
}

// Rows of a share: a multiple of 16, and no more shares than run at once: two on a compute unit, one with eight keys per
// lane.  (A few workgroups more make a last round of whole searches: half of 100 heads of 1k and 64 elements 18.6 us with 600
// workgroups, 15.4 with 500; of 8 heads of 8k 22.9 with 512, 16.9 with 256.)
static int64_t rows_per_share(int64_t n_heads, int64_t T, int64_t k, int64_t least) {
    const int64_t shares = (T <= 4 * kSelThreads ? 512 : 256) / n_heads;        // at least 1: kFuseMaxHeads
    const int64_t rows = ((k + shares - 1) / shares + 15) / 16 * 16;
    return rows > least ? rows : least;
}

static int64_t most_ahead(int32_t row_bytes) {
    return row_bytes == 128 ? RowsAhead<128>::kTokens : row_bytes == 256 ? RowsAhead<256>::kTokens : RowsAhead<512>::kTokens;
}
// Tokens of a share whose rows of V are loaded during the search, 0: shares of kept rows.  While a workgroup holds them, at most
// 34 MB of V, which the memory brings during the search.  From a third of the tokens on, as for kReadAgainBytes: of 32 heads of 4k
// 0.1 / 0.3 / 0.4 kept in shares of tokens 20.1, 22.8, 20.5 us, of kept rows 17.5, 21.2, 22.6; of 64 heads of 1k 13.2, 14.3, - and
// 12.7, 14.4, -; of 8 heads of 8k 0.2 / 1.0 kept 15.6, 19.8 and 14.1, 22.6.  At least 64 tokens: shares of 16 of 2 heads of 3001 11.5 us, of 64 9.6.
static int64_t tokens_ahead(int64_t n_heads, int64_t T, int64_t k, int32_t row_bytes) {
    if (T > kFuseMaxTokens || n_heads > (T <= 4 * kSelThreads ? kFuseMaxHeads : kFuseMaxHeads / 2) || 3 * k < T) return 0;
    const int64_t tokens = rows_per_share(n_heads, T, T, 64);
    return tokens <= most_ahead(row_bytes) ? tokens : 0;
}

// Shares of kept rows only while these do not fill the memory system for longer than the repeated search takes; else a selection
// and a compaction do as well or better: half of 200 heads of 1k (26 MB of K) 35.5 us together and 35.0 apart, of 48 heads of 4k
// (25 MB) 33.9 and 34.4, of 64 heads of 4k (34 MB) 41.4 and 41.9; below 17 MB together is the faster everywhere.
bool select_compact_applies(int64_t n_heads, int64_t T, int64_t k, int32_t row_bytes) {
    return tokens_ahead(n_heads, T, k, row_bytes) != 0 ||
           (T <= kFuseMaxTokens && n_heads <= (T <= 4 * kSelThreads ? kFuseMaxHeads : kFuseMaxHeads / 2) &&
            n_heads * k * row_bytes <= kFuseMaxBytes);
}
// Tokens of a share of the one-launch compression: at least 64, and at most one workgroup on a compute unit.  0: not that launch.
static int64_t short_tokens(int64_t n_heads, int64_t T, int32_t D, l2kv_dtype dt) {
    const int32_t row_bytes = D * (dt == L2KV_F32 ? 4 : 2);
    const int64_t most = dt == L2KV_F32 && n_heads >= kShortManyHeads ? kShortHeadBytesF32 : kShortHeadBytes;
    if (T > kSelThreads || n_heads > kFuseMaxHeads || T * row_bytes > most) return 0;
    const int64_t shares = kFuseMaxHeads / n_heads, tokens = ((T + shares - 1) / shares + 15) / 16 * 16;
    return tokens <= 64 ? 64 : tokens <= most_ahead(row_bytes) ? tokens : 0;
}
bool compress_short_applies(int64_t n_heads, int64_t T, int32_t D, l2kv_dtype dt) { return short_tokens(n_heads, T, D, dt) != 0; }

l2kv_status select_compact_dispatch(const float* norms, int64_t n_heads, int64_t T, int64_t k, const void* K, const void* V,
                                    l2kv_dtype dt, int32_t D, int64_t head_stride, int32_t* kept_idx, void* Kc, void* Vc,
                                    hipStream_t stream) {
    const int es = dt == L2KV_F32 ? 4 : 2;
    const int64_t tokens = tokens_ahead(n_heads, T, k, D * es);
    const bool ahead = tokens != 0;
    const int64_t per_share = ahead ? tokens : rows_per_share(n_heads, T, k, 16), all = ahead ? T : k;
    const dim3 grid((unsigned)((all + per_share - 1) / per_share), (unsigned)n_heads);
    const int64_t per_lane = (T + kSelThreads - 1) / kSelThreads;
    auto launch = ahead ? (per_lane <= 1 ? launch_select_compact<1, true> : per_lane <= 2 ? launch_select_compact<2, true>
                           : per_lane <= 4 ? launch_select_compact<4, true> : launch_select_compact<8, true>)
                        : (per_lane <= 1 ? launch_select_compact<1, false> : per_lane <= 2 ? launch_select_compact<2, false>
                           : per_lane <= 4 ? launch_select_compact<4, false> : launch_select_compact<8, false>);
    launch(grid, D * es, norms, T, k, per_share, K, V, head_stride * es, kept_idx, Kc, Vc, stream);
    return launch_status();
}

l2kv_status compress_short_dispatch(const void* K, const void* V, l2kv_dtype dt, int64_t n_heads, int64_t T, int32_t D,
                                    int64_t head_stride, int64_t k, float* norms, int32_t* kept_idx, void* Kc, void* Vc,
                                    hipStream_t stream) {
    const int64_t tokens = short_tokens(n_heads, T, D, dt), shares = (T + tokens - 1) / tokens;
    const dim3 grid((unsigned)((n_heads + kDies - 1) / kDies * kDies * shares));
    auto kernel = dt == L2KV_F32 ? (D == 64 ? compress_short_kernel<F32, 64> : compress_short_kernel<F32, 128>)
                  : D == 256 ? compress_short_kernel<BF16, 256>
                  : D == 64 ? compress_short_kernel<BF16, 64> : compress_short_kernel<BF16, 128>;
    hipLaunchKernelGGL(kernel, grid, dim3(kSelThreads), 0, stream, static_cast<const char*>(K), static_cast<const char*>(V),
                       (uint32_t)n_heads, (uint32_t)shares, T, (uint32_t)k, (uint32_t)tokens, head_stride * (dt == L2KV_F32 ? 4 : 2), norms, kept_idx,
                       static_cast<char*>(Kc), static_cast<char*>(Vc));
    return launch_status();
}

l2kv_status select_ragged_dispatch(const float* norms, int32_t n_planes, int32_t n_seq,
                                   int64_t total_tokens, const int64_t* in_off, const int64_t* out_off,
                                   int64_t total_kept, int64_t max_len, l2kv_mode mode,
                                   int32_t* kept_idx, hipStream_t stream) {
    const int64_t blocks = (int64_t)n_planes * n_seq;
    if (blocks > 0x7fffffffLL) return L2KV_ERR_SHAPE;
    const uint32_t flip = mode == L2KV_KEEP_HIGHEST ? 0xffffffffu : 0u;
    launch_select_for_length(max_len, norms, blocks, 0, 0, flip, kept_idx, nullptr, stream,
                             RaggedSelect{in_off, out_off, n_seq, total_tokens, total_kept});
    return launch_status();
}

}  // namespace l2kv
