// l2kv_decode_attn, host side: into how many workgroups the launches are cut (no kernel here, so that a
// program for the host alone can ask for a plan).
#include "l2kv_host.hpp"

#include <math.h>

#include <algorithm>

namespace l2kv {

// Ordered ragged batches (a longest-first order of the sequences is known): from this length
// of the longest sequence on, the (sequence, KV head) pairs are handed out one by one to a fixed
// set of workgroups instead of being launched as a grid.
constexpr int64_t kOrderedMinRows = 2048;

int32_t decode_max_splits(int64_t kv_len) {
    if (kv_len <= 0) return 0;
    const int64_t by_rows = (kv_len + kDecodeRowTile - 1) / kDecodeRowTile;
    return (int32_t)(by_rows < kDecodeMaxSplits ? by_rows : kDecodeMaxSplits);
}

DecodePlan decode_plan(int32_t B, int32_t Hkv, int32_t group, int64_t kv_len, int32_t D, int32_t elem_bytes, int32_t requested_splits) {
    const int64_t pairs = (int64_t)B * Hkv;
    const int32_t row_bytes = D * elem_bytes;
    const int64_t cap = decode_max_splits(kv_len);
    int64_t want = requested_splits;
    DecodePlan plan;
    if (want <= 0) {
        // Workgroups (4 waves each) for about three quarters of the compute units,
        // all resident at once.  Measured over batch sizes 1..16 and cache lengths
        // 4k..32k rows per head, the fastest launch always had 192-200 workgroups
        // on the 256 compute units (e.g. 6 splits x 32 heads: 43.5 us, 8 x 32:
        // 45.3 us, 9 x 32, which no longer fits at once: 65 us); fewer streams in
        // flight use the memory system better than one per compute unit.
        // Query groups of 5 and more heads are bound by arithmetic, not memory,
        // and take every compute unit (8 heads per group: 63 us on 256
        // workgroups, 78 us on 192).
        const int64_t cus = device_compute_units();
        const int64_t target = group >= 5 ? cus : 3 * cus / 4;
        want = (2 * target + pairs) / (2 * pairs);                 // nearest integer to target / pairs
        if (want > 1 && want * pairs > cus) --want;
        const int64_t blocks = (kv_len + kDecodeRowTile - 1) / kDecodeRowTile;
        const auto longest_blocks = [&](int64_t splits) { return (blocks + splits - 1) / splits; };
        // Two thirds of the compute units or fewer after rounding leave memory idle; one more split each fits.  us, bf16 rows of 128: 80
        // heads of 9000 rows 64.4 in 2, 60.4 in 3, with 4 query heads 70.3 / 62.6, of 1100 15.4 / 13.3; 56 of 9000 48.7 in 3, 45.1 in 4.  Not
        // where the longest stream does not get shorter by it: 80 of 248 with 3 7.35 in 2, 7.57 in 3.
        if (group < 5 && 3 * want * pairs <= 2 * cus && (want + 1) * pairs <= cus && (want == 0 || longest_blocks(want + 1) < longest_blocks(want))) ++want;
        // More heads than that: a head in one workgroup means rounds of all compute units, the last of which may have little to do; in
        // 3 (2, 5) splits the rounds are shorter and fuller.  us, one / three: bf16 rows of 128 of 5000, 136 heads with 8 query
        // heads 92.7 / 68.5, 288 with 4 166 / 131; 288 of 1500 54.2 / 46.5; fp32 rows of 128, 288 of 5000 with 8 354 / 270; of 64 bf16,
        // 320 of 5000 78.1 / 66.8; two / five: 88 with 6 52.9 / 46.2.  More partial results and shorter streams cost more than that below these lines:
        // 136 of 750 rows with 1 query head 0.95 of the speed, of 1500 with 4 0.98; 341 of 512 with 8 0.87; fp32 rows
        // of 128, 331 of 794 with 7 0.98, 593 of 1311 with 7 0.98, bf16 rows of 256, 593 of 914 0.93.
        const int64_t k_bytes = kv_len * row_bytes, kb = k_bytes >> 10;
        const auto rounds = [&](int64_t workgroups) { return (workgroups + cus - 1) / cus; };
        const bool long_rows = row_bytes > 256;
        int64_t fuller = want;
        if (pairs > cus) {
            if (kb >= (pairs > 2 * cus ? 640 : 384) << (long_rows && group >= 5 ? 1 : 0) && pairs <= 3 * cus && rounds(3 * pairs) <= 3 * rounds(pairs) - 2) fuller = 3;
            else if (kb >= 384 && 2 * pairs <= 3 * cus && group >= 4 && !long_rows) fuller = 2;
        } else if (2 * pairs > cus) {
            if (group >= 5 && !long_rows ? 25 * pairs <= 16 * cus && kb >= 512
                                         : 7 * pairs <= 4 * cus && kb >= (group >= 7 ? 1024 : 2048))
                fuller = 3;
        } else if (group >= 5 && !long_rows && 3 * pairs > cus && 21 * pairs <= 8 * cus && kb >= 1024) {
            fuller = 5;
        }
        // l2kv_decode_attn_static takes the same splits, so their partial results have to fit its scratch memory.  Those of 513 to 597 heads
        // with 6 and more query heads (5 from 530 heads on; rows of 256 elements: 3 and more), and of 331 to 341 with 8, do not; one workgroup
        // each costs them little: bf16 rows of 128, 544 of 4096 with 8 219 in place of 199, 560 of 2600 with 6 151 / 135, 336 of 2048 with 8
        // 75.9 / 69.8; of 256, 513 of 1500 with 4 147.5 / 148.8.
        if (fuller > want && decode_scratch_bytes(B, Hkv, group, (int32_t)fuller, D) > L2KV_STATIC_SCRATCH_BYTES) fuller = want;
        want = fuller;
        // With very few heads that rule asks for so many workgroups per head that
        // the final merge (about 0.2 us per workgroup) outweighs the shorter
        // streams (about 0.025 us per row): the sum is smallest near
        // 0.34 * sqrt(rows) workgroups (measured optima: 32 at 8k rows, 64 at 32k,
        // 128 at 131k with one or two heads).
        int64_t by_merge = (int64_t)(0.34 * sqrt((double)kv_len));
        if (by_merge < 8) by_merge = 8;
        if (want > by_merge) want = by_merge;
        // Short heads: up to 8 workgroups merge in registers (kWideMerge), which saves more than longer streams cost while a
        // head has at most 384 KB of K.  Groups of 5 heads and more, whose merge of more than 8 goes through LDS: 512 KB and, for
        // their arithmetic, 3072 rows.  us, split as above / in 8: 16 heads of 1554 rows of 64 elements, 4 query heads each,
        // 8.7 / 8.2, 4 of 1673 rows of 128 6.5 / 7.0, 3 of 1265 5.7 / 5.6; groups of 5 and more: 24 heads of 1146 rows of 128 11.6 /
        // 10.9, 16 of 3042 rows of 64 11.5 / 10.9, 2 of 3735 9.5 / 10.0; fp32 rows of 128, 4 of 907 11.9 / 10.8, 8 of 1419 10.6 / 10.7.
        // Fewer than 12 of these heads leave the memory idle, so that a longer stream counts: the longest at most 24 KB longer (64 rows at a
        // time, so often not at all), for one or two heads not beyond 384 KB.  bf16 rows of 128, 3 heads of 1615 with 5 query heads 8.8 / 9.4, 8 of
        // 1607 with 6 10.5 / 11.2, 1 of 1804 with 5 6 % slower in 8; fp32 rows of 64, 3 of 1790 with 8 9.3 / 10.3; not longer: fp32 rows of 128, 2 of
        // 929 with 6 10.0 / 9.1.
        auto longest = [&](int64_t splits) { return longest_blocks(splits) * kDecodeRowTile * row_bytes; };
        bool short_head = group < 5 ? k_bytes <= int64_t{384} << 10 : k_bytes <= int64_t{512} << 10 && kv_len <= 3072;
        if (short_head && group >= 5 && pairs < 12 && want > kDecodeNarrowSplits) {
            const int64_t longer = longest(kDecodeNarrowSplits) - longest(want);
            short_head = longer == 0 || (longer <= 24 << 10 && (pairs > 2 || k_bytes <= int64_t{384} << 10));
        }
        if (want > kDecodeNarrowSplits && short_head) want = kDecodeNarrowSplits;
        // Very short heads: a wave has few tiles of 16 rows to read (32 at rows of 128 bytes), and to write, wait for and merge partial
        // results takes longer than the tiles that the other workgroups would have read.  us, split as above / in 1: bf16 rows of 128, 32
        // heads of 83 rows 4.6 / 3.2, 8 of 175 4.3 / 3.4; of 64, 128 of 88 with 4 query heads 6.3 / 4.4; fp32 rows of 64, 128 of 184 with 3
        // 6.7 / 5.7; 4 of 256, 4.2 / 3.3.  Not for more tiles or query heads: bf16 rows of 128, 8 of 189 with 4 5.9 / 6.3; of 256, 8 of 128
        // with 4 7.1 / 7.3.  That is with rows in the caches, as after a compression, where three tiles gain 7 to 29 % and four 1 to 17 % in the mean
        // of 1 to 64 heads (64 heads of 252 rows 0.94 to 0.96).  From memory, where every second tile is one more round trip, three gain 1 to 9 %
        // and four lose 1 to 3 %; the worst are few heads whose last tile is not whole (4 of 188 rows 0.92 to 0.97, of 252 0.87 to 0.89).
        const int64_t tile_rows = row_bytes <= 128 ? 2 * kDecodeRowTile : kDecodeRowTile;      // of the four waves
        const int64_t tiles = (kv_len + tile_rows - 1) / tile_rows;
        if (tiles <= 2 ? !long_rows || group <= 3 : !long_rows && (tiles == 3 ? group <= 3 : tiles == 4 && group <= 2)) want = 1;
        // Few heads: their streams leave memory idle, so that the splits are counted in the 64-row steps of the longest: as many as make
        // its steps and the merge shortest together.  One more partial result costs 0.05 to 0.06 steps of a lone head (0.7 to 1.8 us;
        // least squares over 16 to 128 splits of 1600 to 32000 rows), more beside others, and with up to 4 query heads a lot past 64,
        // where it goes through LDS.  us, 0.34 * sqrt(rows) / here: bf16 rows of 128, 1 head of 16000 8.7 / 7.8, 2 of 4096 with 4
        // query heads 9.1 / 8.2, with 8 13.2 / 11.7; fp32 rows of 128, 1 of 4096 with 8 16.8 / 12.9, 3 with 8 17.5 / 14.0.  Not where less than
        // 5 % (two heads of 256-byte rows 14 %) is to be gained, nor for more heads (4 of 9404 fp32 rows of 64 9.2 / 9.7) or 128-byte rows (1
        // of 49352 10.3 / 10.8).
        // Long rows with up to 4 query heads: a step takes 0.9 us and 0.1 for each further one, a partial result 0.011 to 0.02, twice that
        // past 32 and 2 us past 64.  fp32 rows of 128, 3 heads of 1886 with 2 query heads 7.6 / 6.5, 1 of 9322 10.0 / 8.4, 1 of 53342 with 2
        // 19.7 / 16.0; bf16 rows of 256, 3 of 4121 with 3 12.0 / 10.9.  Four heads beyond 4 MB of K: 8675 bf16 rows of 256 12.0 / 12.2.
        const bool by_long_rows = long_rows && group <= 4;
        const bool few = by_long_rows ? pairs <= 3 || (pairs == 4 && k_bytes <= 4 << 20)
                         : row_bytes > 128 && pairs <= (long_rows ? 4 : 2) && k_bytes >= 768 << 10 && kv_len <= (group > 4 && pairs == 1 ? 65536 : 32768);
        if (want > kDecodeNarrowSplits && few) {
            const int64_t most = std::min<int64_t>((2 * target + pairs) / (2 * pairs), group <= 4 && !long_rows ? std::min<int64_t>(cap, 64) : cap);
            const auto cost = [&](int64_t each, int64_t splits) {
                return by_long_rows ? (0.9 + 0.1 * (group - 1)) * each + (0.008 + 0.003 * group) * (splits > 32 ? 2 : 1) * splits + (splits > 64 ? 2 : 0)
                                    : each + (0.01 * pairs + (group <= 4 ? 0.06 : 0.05)) * splits;
            };
            double least = by_long_rows ? 1e9 : (pairs == 1 || long_rows ? 0.95 : 0.86) * cost((blocks + want - 1) / want, want);
            // all splits together cost less than 32 steps, so that longer streams need not be tried
            // More than 32 partial results of 256 elements are merged in two round trips, which streams of one block each do not make up
            // for: bf16, 4 heads of 2826 rows with 2 query heads 45 splits 0.91 of the speed of 18 and 0.85 of that of 23, 3 of 2886 with 2 0.89 of that of 23; 1 of 2155 1.04.
            const int64_t shortest = std::max<int64_t>(longest_blocks(most), D == 256 && pairs > 2 && blocks > 32 ? 2 : 1);
            for (int64_t each = shortest, splits; each < shortest + 32 && (splits = (blocks + each - 1) / each) > kDecodeNarrowSplits; ++each)
                if (cost(each, splits) < least) least = cost(each, splits), want = splits;
        }
    }
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    plan.n_splits = (int32_t)want;
    return plan;
}

DecodePlan decode_plan_ragged(int32_t n_seq, int32_t Hkv, int64_t max_len, int64_t total_slots, int32_t requested_splits,
                              bool ordered) {
    const int64_t pairs = (int64_t)n_seq * Hkv;
    int64_t want = requested_splits;
    const int64_t cap = decode_max_splits(max_len);
    DecodePlan plan;
    if (ordered && max_len >= kOrderedMinRows) {
        // A longest-first order is known.  The items of the work list are the (sequence, KV head) pairs, in
        // pieces where the kernel finds the sequences long (ragged_plan.hpp), and one workgroup per compute unit
        // draws them from the list.  Measured on the 64-sequence streaming batch (512 pairs of
        // 512..4200 rows, whole): faster than any grid launch of the same batch, whose
        // best (5 workgroups per pair in batch order) took 108 us per layer.
        const int64_t cus = device_compute_units();
        if (want <= 0) {
            const RaggedRule rule = ragged_rule(cus, n_seq, Hkv, total_slots, (int32_t)(cap < kRaggedMostPieces ? cap : kRaggedMostPieces));
            const int32_t bound = (int32_t)(max_len < INT32_MAX ? max_len : INT32_MAX);
            want = ragged_base(rule, bound);
            if (want < kRaggedMostPieces) {              // with more, the load has no say
                plan.rule = rule;
                plan.pieces = ragged_pieces(rule, bound);
                want = rule.most;
            }
        }
        if (plan.rule.most == 0) plan.pieces = (int32_t)(want < cap ? want : cap);
        const int64_t items = pairs * (want < cap ? want : cap);
        if (items <= kDecodeMostCounted) plan.worklist_wgs = (int32_t)(items < cus ? items : cus);     // more, by the caller's count alone: a grid
    } else if (want <= 0) {
        // Lengths differ, so the launch relies on the hardware handing out more
        // workgroups than fit at once: about 1024 rows per workgroup, and never
        // fewer workgroups than compute units.  Workgroups go to the 8 compute
        // dies round-robin by linear id (split + n_splits * pair); an odd
        // n_splits spreads every split index over all dies, which matters here
        // because the high split indices carry less work (measured: 5 splits
        // 108 us, 4 splits 127 us, 8 splits 149 us on the same batch).
        const int64_t by_len = (max_len + 1023) / 1024;
        const int64_t by_cu = (device_compute_units() + pairs - 1) / pairs;
        want = by_len > by_cu ? by_len : by_cu;
        if (want > 1 && want % 2 == 0) want += want < cap ? 1 : -1;
    }
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    plan.n_splits = (int32_t)want;
    // rows per workgroup such that the longest sequence employs all workgroups
    const int64_t rows = (max_len + want - 1) / want;
    plan.rows_per_wg = (int32_t)(rows < kDecodeRowTile ? kDecodeRowTile : rows);
    return plan;
}

}  // namespace l2kv
