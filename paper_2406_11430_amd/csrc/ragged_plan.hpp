// Into how many pieces the work list of an ordered ragged batch cuts its sequences.  The host knows the slots and the compute
// units (ragged_rule), the kernel the length of the longest sequence, the first in the order (ragged_pieces): of the caller's
// bound, which may be any number above it, nothing depends but the room in the workspace.
#pragma once
#include <stdint.h>

namespace l2kv {

constexpr int32_t kOrderedMaxRows = 16384;    // rows one workgroup takes before a sequence is split
constexpr int32_t kRaggedMostPieces = 8;      // that are cut because of the load
constexpr int32_t kRaggedSkewPieces = 5;

struct RaggedRule {
    int32_t by_cu;         // workgroups of a pair by the rule for uniform batches
    int32_t most;          // pieces there is room for, 0: no rule
    int32_t few;           // 3, or 2 if there are nearly as many pairs as workgroups
    int32_t uneven_from;   // rows of a sequence half as long again as the average
    float cut_above;       // 1.3 loads
    float long_rows;       // 1.75 loads
    float pieces_per_row;  // of pieces that just leave every one a workgroup of its own
};

// load: rows of a pair times pairs, as far as the slots tell, for each of the workgroups.
inline RaggedRule ragged_rule(int64_t cus, int32_t n_seq, int32_t Hkv, int64_t total_slots, int32_t most) {
    const int64_t pairs = (int64_t)n_seq * Hkv, total = total_slots * Hkv, load = (total + cus - 1) / cus;
    const int64_t target = 3 * cus / 4, room = cus - pairs / 2, uneven = (3 * total_slots + 2 * n_seq - 1) / (2 * n_seq);
    RaggedRule r;
    r.by_cu = (int32_t)((2 * target + pairs) / (2 * pairs));
    r.most = most;
    r.few = pairs <= cus - cus / 16 ? 3 : 2;
    r.uneven_from = (int32_t)(uneven < INT32_MAX ? uneven : INT32_MAX);
    r.cut_above = 1.3f * (float)load;
    r.long_rows = 1.75f * (float)load;
    r.pieces_per_row = room > 0 ? 20.f * (float)room / (21.f * (float)total) : 0.f;
    return r;
}

// Sequences beyond 16k rows are cut, or all of them where the batch has fewer pairs than the uniform rule wants workgroups.
__host__ __device__ inline int32_t ragged_base(const RaggedRule& r, int32_t longest) {
    const int32_t by_len = longest / kOrderedMaxRows + (longest % kOrderedMaxRows != 0 ? 1 : 0);
    return by_len > r.by_cu ? by_len : r.by_cu;
}
// Sequences much longer than the load are cut as well, or the launch waits for them.  Best into as many pieces as just leave every
// one a workgroup of its own (each sequence's last piece is half full on average, and 5 % for chance).  Where that leaves pieces of
// more than 1.75 loads, into so many that they are no longer, but five at most (each costs a draw for every sequence that is too short
// for it) and three, or two, at least; not where the sequences are much alike (192 pairs of 4000 rows 62, in three 74).
// us per layer, whole / cut so / the best of 1 to 8 pieces.  Sequences of 500 to 4400 rows: 192 pairs 61 / 47 / 44, 240 67 / 56 / 56, 288
// 74 / 70 / 67, 320 79 / 72 / 71; of 250 to 2260, 160 pairs 34 / 27 / 23; one of 8000 and the others of 500: 192 105 / 28.7 / 26.4, 248
// 105 / 29.7 / 29.5, 512 108 / 41 / 40.  Over 376 batches of 4 to 64 sequences 5 % from the best on average, and slower than
// ragged_base alone in ten, by up to 11 % (40 pairs of 1600 to 3300 rows, 7 pieces 16.5, 5 15.1).
__host__ __device__ inline int32_t ragged_pieces(const RaggedRule& r, int32_t longest) {
    const int32_t base = ragged_base(r, longest);
    const float rows = (float)longest;
    int32_t n = 1;
    if (rows > r.cut_above) {
        const float own = rows * r.pieces_per_row;
        n = own < (float)kRaggedMostPieces ? (int32_t)own : kRaggedMostPieces;
        if (rows > (float)n * r.long_rows && longest >= r.uneven_from) {
            int32_t cut = r.few;
            while (cut < kRaggedSkewPieces && rows > (float)cut * r.long_rows) ++cut;
            n = n > cut ? n : cut;
        }
    }
    n = n > base ? n : base;
    return n < r.most ? n : r.most;
}

}  // namespace l2kv
