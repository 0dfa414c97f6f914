// Ragged batches and the streaming slot cache.
//
// arXiv 2406.11430, Sec. 4 ("Language Modelling Tasks"): the cache grows up to a
// pre-defined length, after which the tokens with the highest key norm are
// discarded.  Here every sequence owns a fixed range of slots in each head
// plane; a slot holds the K and V rows, the fp32 squared key norm and the
// original token id of one kept token:
//
//   Kc, Vc  [n_planes][total_slots][D]      n_planes = layers x KV heads
//   norms_c [n_planes][total_slots] fp32    pos_c [n_planes][total_slots] int32
//   sequence s: slots slot_off[s] .. slot_off[s+1]-1, the first lens[s] occupied
//
// Three kernels:
//   compact_ragged : kept rows of a ragged prompt batch -> slot cache (with norms, ids)
//   stream_append  : one new token per sequence -> next free slot, norm computed here
//                    (fixed summation order), so no separate norm pass is ever needed
//   stream_evict   : while a sequence holds more than its budget, drop the slot
//                    with the largest (norm bits, token id) and move the last
//                    slot into the hole -- the reverse of the keep order of
//                    l2kv_select, so the kept set is always "lowest norms, ties
//                    to the lower token id"
#include "l2kv_device.hpp"
#include "l2kv_host.hpp"

namespace l2kv {

// ------------------------------------------------------------ compact_ragged
constexpr int kRagThreads = 256;
constexpr int kRagWaves = kRagThreads / kWaveSize;
constexpr int kRagUnroll = 4;
template <int kRowBytes>
constexpr int kRagRowsPerBlock = kRagWaves * RowCopy<kRowBytes>::kRowsPerWave * kRagUnroll;   // 64, or 128 short ones

// Index of the sequence whose output range holds flat kept row j of a plane: the last s in
// [0, n_seq) with out_off[s] <= j (offsets ascend in a consistent batch, and whatever they hold
// the result is a valid sequence index).  For a wave: j is the same in all lanes, every step reads 64
// offsets at once and narrows the range 64 times, so up to 64 sequences cost one memory round trip (a binary
// search costs six, one after the other).
__device__ __forceinline__ int32_t owner_of_row(const int64_t* __restrict__ out_off, int32_t n_seq, int64_t j) {
    const int lane = threadIdx.x % kWaveSize;
    int32_t lo = 0, count = n_seq;                     // the answer is in [lo, lo + count)
    while (count > 1) {
        const int32_t step = (int32_t)(((int64_t)count + kWaveSize - 1) / kWaveSize);
        const int32_t mine = lo + lane * step;         // first candidate of this lane's stretch
        const bool at_or_before = lane * (int64_t)step < count && out_off[mine < n_seq ? mine : n_seq - 1] <= j;
        const uint64_t mask = __ballot(at_or_before);
        const int32_t last = mask == 0 ? 0 : 63 - __builtin_clzll(mask);
        const int32_t left = count - last * step;
        lo += last * step;
        count = left < step ? left : step;
    }
    return lo;
}

// One sequence's ranges in the input, among the kept rows and among the slots.
struct SeqRanges {
    Range in, slots;
    int64_t out_first, k;                              // kept rows that fit its slots: [out_first, out_first + k)
    __device__ __forceinline__ SeqRanges(const int64_t* in_off, const int64_t* out_off, const int64_t* slot_off, int64_t seq,
                                         int64_t total_tokens, int64_t total_kept, int64_t total_slots)
        : in(clamped_range(in_off, seq, total_tokens)), slots(clamped_range(slot_off, seq, total_slots)) {
        const Range out = clamped_range(out_off, seq, total_kept);
        out_first = out.first;
        k = out.count < slots.count ? out.count : slots.count;       // never write past the sequence's slots
    }
};

// Grid (chunks per plane, alternately of K and of V, x planes): the kept rows of a plane, all sequences back to back
// (as kept_idx holds them), are cut into chunks of 64 (128 short) consecutive rows, so every workgroup has
// a full chunk whatever the lengths of the sequences are (a launch sized by the longest
// sequence would leave almost half of its workgroups without work on a batch of mixed lengths).
// K and V alternate as in compact_kernel; the workgroups of K also move norms and token ids.
// A wave takes 16 (32) consecutive flat rows, 4 per row group.  Short-lived workgroups are bound by the chain of
// loads in front of their rows: owner of the first row, ranges of that sequence, indices, rows.  All
// rows of a wave belong to that sequence as a rule; where a sequence ends among them, each row finds
// its own.  147k kept rows of 8 planes, 64 sequences: 241 -> 213 us (5.7 TB/s).
template <int kRowBytes>
__global__ __launch_bounds__(kRagThreads)
void compact_ragged_kernel(const char* __restrict__ K, const char* __restrict__ V,
                           const float* __restrict__ norms, const int32_t* __restrict__ kept_idx,
                           int32_t n_seq, int64_t total_tokens, const int64_t* __restrict__ in_off,
                           const int64_t* __restrict__ out_off, int64_t total_kept, const int64_t* __restrict__ slot_off,
                           int64_t total_slots, int64_t first_plane, int64_t first_chunk, char* __restrict__ Kc,
                           char* __restrict__ Vc, float* __restrict__ norms_c, int32_t* __restrict__ pos_c) {
    using P = RowCopy<kRowBytes>;
    constexpr int W = P::kWords;
    // from the end, as in compact_kernel
    const bool is_v = blockIdx.x % 2 != 0;
    const int64_t chunk = first_chunk + (gridDim.x - 1 - blockIdx.x) / 2;
    const int64_t plane = first_plane + (gridDim.y - 1 - blockIdx.y);
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int c = lane % P::kLanes;
    const int rg = lane / P::kLanes;

    const int64_t wave_first = chunk * kRagRowsPerBlock<kRowBytes> + wave * (P::kRowsPerWave * kRagUnroll);
    if (wave_first >= total_kept) return;
    const int64_t first = wave_first + rg * kRagUnroll;
    const int32_t* idx = kept_idx + plane * total_kept;

    int32_t t[kRagUnroll];
#pragma unroll
    for (int u = 0; u < kRagUnroll; ++u) t[u] = idx[first + u < total_kept ? first + u : total_kept - 1];

    // per row: its source row and destination slot; a row that the (possibly inconsistent) offset
    // arrays do not place inside its sequence's ranges is skipped
    int64_t src[kRagUnroll], dst[kRagUnroll];
    bool live[kRagUnroll];
    auto place = [&](int u, const SeqRanges& r) {
        const int64_t j = first + u < total_kept ? first + u : total_kept - 1;
        const int64_t local = j - r.out_first;
        live[u] = first + u < total_kept && local >= 0 && local < r.k && r.in.count > 0;
        const int64_t T = r.in.count > 0 ? r.in.count : 1;
        t[u] = t[u] < 0 ? 0 : (t[u] < T ? t[u] : (int32_t)(T - 1));       // stay inside the sequence whatever idx holds
        // a skipped row still gets an in-bounds source (row 0 of the plane) so the loads below need no branch
        src[u] = plane * total_tokens + (live[u] ? r.in.first + t[u] : 0);
        dst[u] = plane * total_slots + r.slots.first + (live[u] ? local : 0);
    };
    int64_t seq = __builtin_amdgcn_readfirstlane(owner_of_row(out_off, n_seq, wave_first));
    // first rows of the next 64 sequences, one per lane
    const int64_t next = seq + 1 + lane;
    const bool there = next < n_seq;
    const int64_t begin = out_off[there ? next : n_seq - 1];
    const bool one_sequence = (__ballot(there && begin < wave_first + P::kRowsPerWave * kRagUnroll) & 1) == 0;
    if (one_sequence) {
        const SeqRanges r(in_off, out_off, slot_off, seq, total_tokens, total_kept, total_slots);
#pragma unroll
        for (int u = 0; u < kRagUnroll; ++u) place(u, r);
    } else {
        // every row counts the sequences that begin up to it (one step along the offsets after the other was a
        // chain of loads: 4000 sequences of 2 to 6 tokens 18.9 us instead of 20.6, 1000 of 8 to 40 25.3 instead of 26.2)
#pragma unroll
        for (int u = 0; u < kRagUnroll; ++u) {
            int64_t mine = seq;
#pragma unroll
            for (int g = 0; g < P::kRowsPerWave; ++g) {               // the same row in all lanes
                const int64_t j = wave_first + g * kRagUnroll + u;
                const uint64_t later = ~__ballot(there && begin <= (j < total_kept ? j : total_kept - 1));
                const int64_t owner = seq + (later == 0 ? kWaveSize : __builtin_ctzll(later));
                mine = rg == g ? owner : mine;
            }
            const int64_t j = first + u < total_kept ? first + u : total_kept - 1;
            while (mine >= seq + kWaveSize && mine + 1 < n_seq && out_off[mine + 1] <= j) ++mine;      // 64 empty ones and more
            place(u, SeqRanges(in_off, out_off, slot_off, mine, total_tokens, total_kept, total_slots));
        }
    }
    const char* from = is_v ? V : K;
    char* to = is_v ? Vc : Kc;
    Words<W> rows[kRagUnroll];
#pragma unroll
    for (int u = 0; u < kRagUnroll; ++u) rows[u] = load_words_stream<W, P::kStride>(from + src[u] * (int64_t)kRowBytes + c * 16);
    float norm[kRagUnroll];
    if (!is_v && c == 0) {
#pragma unroll
        for (int u = 0; u < kRagUnroll; ++u) norm[u] = norms[src[u]];
    }
#pragma unroll
    for (int u = 0; u < kRagUnroll; ++u) {
        if (live[u]) {
            store_words_stream<W, P::kStride>(to + dst[u] * (int64_t)kRowBytes + c * 16, rows[u]);
            if (!is_v && c == 0) {
                norms_c[dst[u]] = norm[u];
                pos_c[dst[u]] = t[u];
            }
        }
    }
}

l2kv_status compact_ragged_dispatch(const void* K, const void* V, const float* norms, l2kv_dtype dt,
                                    const int32_t* kept_idx, int32_t n_planes, int32_t n_seq,
                                    int64_t total_tokens, const int64_t* in_off, const int64_t* out_off,
                                    int64_t total_kept, int64_t max_kept, const int64_t* slot_off,
                                    int64_t total_slots, int32_t D, void* Kc, void* Vc, float* norms_c,
                                    int32_t* pos_c, hipStream_t stream) {
    (void)max_kept;                                    // the launch is sized by total_kept
    const int row_bytes = D * (dt == L2KV_F32 ? 4 : 2);
    if ((total_kept + 63) / 64 * n_planes > 0x7fffffffLL) return L2KV_ERR_SHAPE;
    const int64_t rows_per_block = row_bytes == 128 ? kRagRowsPerBlock<128> : kRagRowsPerBlock<256>;
    static_assert(kRagRowsPerBlock<256> == kRagRowsPerBlock<512>, "one chunk size for rows of 16 lanes");
    const int64_t chunks = (total_kept + rows_per_block - 1) / rows_per_block;
    constexpr int64_t kMaxX = 1 << 22, kMaxY = 65535;  // a launch has fewer than 2^32 lanes in x, 2^16 workgroups in y
    for (int64_t p0 = 0; p0 < n_planes; p0 += kMaxY) {
        for (int64_t c0 = 0; c0 < chunks; c0 += kMaxX) {
            const dim3 grid((unsigned)(2 * (chunks - c0 < kMaxX ? chunks - c0 : kMaxX)),       // of K and of V
                            (unsigned)(n_planes - p0 < kMaxY ? n_planes - p0 : kMaxY));
#define L2KV_RAG(RB)                                                                               \
    hipLaunchKernelGGL((compact_ragged_kernel<RB>), grid, dim3(kRagThreads), 0, stream,            \
                       static_cast<const char*>(K), static_cast<const char*>(V), norms, kept_idx,  \
                       n_seq, total_tokens, in_off, out_off, total_kept, slot_off, total_slots,    \
                       p0, c0, static_cast<char*>(Kc), static_cast<char*>(Vc), norms_c, pos_c)
            switch (row_bytes) {
                case 128: L2KV_RAG(128); break;
                case 256: L2KV_RAG(256); break;
                case 512: L2KV_RAG(512); break;
                default: return L2KV_ERR_SHAPE;
            }
#undef L2KV_RAG
            if (l2kv_status st = launch_status(); st != L2KV_OK) return st;
        }
    }
    return L2KV_OK;
}

// a / b and a % b for 0 <= a <= bound, 0 < b < 2^32: in 32 bits wherever the launch's bound fits (a 64-bit division is
// a hundred instructions at the start of kernels that last five microseconds).
struct DivMod { int64_t quotient, rest; };
__device__ __forceinline__ DivMod divided(int64_t a, int64_t b, int64_t bound) {
    if (bound <= 0xffffffffLL) {
        const uint32_t q = (uint32_t)a / (uint32_t)b;
        return DivMod{q, (uint32_t)a - q * (uint32_t)b};
    }
    return DivMod{a / b, a % b};
}

// -------------------------------------------------------------- stream_append
// One 16-lane row group per (layer, sequence, KV head).  Knew, Vnew are
// [n_layers][n_seq][Hkv][D]; the plane of (layer, head) is layer*Hkv + head.
template <typename E, int D>
__global__ __launch_bounds__(256)
void stream_append_kernel(const char* __restrict__ Knew, const char* __restrict__ Vnew, int64_t n_rows,
                          int64_t n_seq, int64_t Hkv, const int32_t* __restrict__ token_ids,
                          const int64_t* __restrict__ slot_off, int64_t total_slots,
                          const int32_t* __restrict__ lens_in, int32_t* __restrict__ lens_out,
                          char* __restrict__ Kc, char* __restrict__ Vc, float* __restrict__ norms_c,
                          int32_t* __restrict__ pos_c) {
#pragma clang fp contract(off)
    using S = Slice<E, D>;
    const int c = threadIdx.x % kRowLanes;
    int64_t r = (int64_t)blockIdx.x * (256 / kRowLanes) + threadIdx.x / kRowLanes;   // (layer, seq, head) row
    const bool live = r < n_rows;
    r = live ? r : n_rows - 1;                    // idle groups shadow the last row, stores skipped
    const DivMod row = divided(r, Hkv, n_rows);
    const DivMod of = divided(row.quotient, n_seq, n_rows);
    const int64_t head = row.rest, seq = of.rest, layer = of.quotient;
    const int64_t plane = layer * Hkv + head;

    const int32_t len = lens_in[seq];
    const Range slots = clamped_range(slot_off, seq, total_slots);
    const bool room = len >= 0 && len < slots.count;   // a full sequence is left untouched
    const Words<S::kWords> kr = load_words<S::kWords>(Knew + r * S::kRowBytes + c * S::kBytes);
    const Words<S::kWords> vr = load_words<S::kWords>(Vnew + r * S::kRowBytes + c * S::kBytes);

    // squared norm in the library's fixed order (chunk left to right, neighbour tree)
    float x[S::kElems];
    widen<E, D>(kr, x);
    float acc = x[0] * x[0];
#pragma unroll
    for (int e = 1; e < S::kElems; ++e) {
        const float sq = x[e] * x[e];
        acc = acc + sq;
    }
    const float norm = row16_tree_sum(acc);

    if (live && room) {
        const int64_t slot = plane * total_slots + slots.first + len;
        store_words<S::kWords>(Kc + slot * S::kRowBytes + c * S::kBytes, kr);
        store_words<S::kWords>(Vc + slot * S::kRowBytes + c * S::kBytes, vr);
        if (c == 0) {
            norms_c[slot] = norm;
            pos_c[slot] = token_ids[seq];
        }
    }
    if (live && plane == 0 && c == 0) lens_out[seq] = room ? len + 1 : len;
}

l2kv_status stream_append_dispatch(const void* Knew, const void* Vnew, l2kv_dtype dt, int32_t n_layers,
                                   int32_t n_seq, int32_t Hkv, int32_t D, const int32_t* token_ids,
                                   const int64_t* slot_off, int64_t total_slots, const int32_t* lens_in,
                                   int32_t* lens_out, void* Kc, void* Vc, float* norms_c, int32_t* pos_c,
                                   hipStream_t stream) {
    const int64_t n_rows = (int64_t)n_layers * n_seq * Hkv;
    const int64_t blocks = (n_rows + 15) / 16;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return L2KV_ERR_SHAPE;
#define L2KV_APP(EE, DD)                                                                           \
    hipLaunchKernelGGL((stream_append_kernel<EE, DD>), dim3((unsigned)blocks), dim3(256), 0, stream, \
                       static_cast<const char*>(Knew), static_cast<const char*>(Vnew), n_rows,     \
                       (int64_t)n_seq, (int64_t)Hkv, token_ids, slot_off, total_slots, lens_in,     \
                       lens_out, static_cast<char*>(Kc), static_cast<char*>(Vc), norms_c, pos_c)
    if (dt == L2KV_F32) {
        if (D == 64) L2KV_APP(F32, 64); else L2KV_APP(F32, 128);
    } else {
        if (D == 64) L2KV_APP(BF16, 64); else if (D == 128) L2KV_APP(BF16, 128); else L2KV_APP(BF16, 256);
    }
#undef L2KV_APP
    return launch_status();
}

// --------------------------------------------------------------- stream_evict
constexpr int kEvictThreads = 256;
constexpr int kEvictWaves = kEvictThreads / kWaveSize;
// One wave per team from 2048 teams on, and from two for every slot of a sequence: as many waves as the chip holds at
// once hide each other's round trips, while a long scan is the faster for every lane that shares it.  Waves and
// workgroups, us, by teams and slots: 1536 of 512 7.0, 7.1; 2048 of 512 7.0, 8.8; 3072 of 512 7.0, 10.2; 2048 of 1024 7.0, 8.5;
// 3072 of 2048 17.7, 14.4; 4032 of 2048 18.7, 18.0; 6144 of 2048 20.9, 24.3; 1024 of 4096 26, 8; 4032 of 4096 31, 23;
// 8192 of 4096 43, 35; 16384 of 4096 75, 75; 16384 of 1024 29, 51.
constexpr int64_t kEvictWaveTeams = 2048;

// One team of lanes per (plane, sequence): a whole workgroup (kTeam = 256), or one wave of a
// workgroup that serves four of them (kTeam = 64; no LDS and no barrier then).  The work of a team is a chain of
// dependent memory round trips -- lengths, scan, move -- so what counts is how short the chain is
// while the teams are few, and how many of them are in flight when they are many (the dispatch
// has the line).  Every eviction is one arg-max over the occupied slots
// of key = (norm bits, token id): per-lane scan of the norms, wave maximum by lane swaps, and for
// workgroup teams 4 wave results through LDS.  Token ids are read only where two norms tie.  The
// row that would move into the hole is known before the scan (the last one) and requested ahead of
// it.  In the steady state of a growing budget at most one slot goes per step.  One of
// 512 to 4096 slots from each of 64 sequences in 16 planes: 12.1 -> 7.2 us, in 256 planes 31 -> 26 (ids read and
// merged for every lane, the row requested after the scan, one wave per team in both).
template <int W, int kTeam>
__global__ __launch_bounds__(kEvictThreads)
void stream_evict_kernel(int64_t n_seq, int64_t n_teams, const int64_t* __restrict__ slot_off, int64_t total_slots,
                         const int32_t* __restrict__ lens_in, const int32_t* __restrict__ budgets,
                         int32_t* __restrict__ lens_out, char* __restrict__ Kc, char* __restrict__ Vc,
                         float* __restrict__ norms_c, int32_t* __restrict__ pos_c) {
    constexpr int64_t kSliceBytes = 4 * W;
    constexpr int64_t kRowBytes = kRowLanes * kSliceBytes;
    __shared__ uint32_t s_norm[kEvictWaves];
    __shared__ int32_t s_slot[kEvictWaves];
    const int64_t team = (int64_t)blockIdx.x * (kEvictThreads / kTeam) + threadIdx.x / kTeam;
    if (team >= n_teams) return;                   // a whole wave (teams are waves or workgroups)
    const int tid = threadIdx.x % kTeam;           // position in the team
    const DivMod at = divided(team, n_seq, n_teams);
    const int64_t seq = at.rest, plane = at.quotient;
    const int lane = threadIdx.x % kWaveSize;
    [[maybe_unused]] const int wave = threadIdx.x / kWaveSize;

    const Range slots = clamped_range(slot_off, seq, total_slots);
    const int64_t cap = slots.count;
    int32_t len = lens_in[seq];
    len = len < 0 ? 0 : (len < cap ? len : (int32_t)cap);
    int32_t budget = budgets[seq];
    budget = budget < 0 ? 0 : budget;
    const int64_t base = plane * total_slots + slots.first;
    const uint32_t* nb = reinterpret_cast<const uint32_t*>(norms_c) + base;
    float* nw = norms_c + base;
    int32_t* pw = pos_c + base;

    // of two slots with equal norms the one with the larger token id goes first
    auto later = [&](int32_t a, int32_t b) { return (uint32_t)pw[a] > (uint32_t)pw[b]; };
    while (len > budget) {                         // uniform over the team
        const int32_t last = len - 1;
        // first 16 lanes K, next 16 lanes V, one lane norm and id of the last slot
        char* const buf = tid < kRowLanes ? Kc : Vc;
        const int c = tid % kRowLanes;
        Words<W> row;
        float last_norm = 0.f;
        int32_t last_id = 0;
        if (tid < 2 * kRowLanes) {
            row = load_words<W>(buf + (base + last) * kRowBytes + c * kSliceBytes);
        } else if (tid == 2 * kRowLanes) {
            last_norm = nw[last];
            last_id = pw[last];
        }
        // Per-lane scan over the norms only (half of the bytes a scan of norms and token ids would
        // read): eight slots per lane and step, their loads issued before the first compare
        // (positions past the end re-read the last slot, which cannot beat itself).
        uint32_t best_norm = 0;
        int32_t best_slot = -1, best_id = 0;
        bool have_id = false;                                             // best_id is that of best_slot
        constexpr int kScan = 8;
        for (int32_t j0 = tid; j0 < len; j0 += kScan * kTeam) {
            uint32_t nv[kScan];
            int32_t js[kScan];
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                const int32_t j = j0 + u * kTeam;
                js[u] = j < len ? j : len - 1;
                nv[u] = nb[js[u]];
            }
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                if (best_slot < 0 || nv[u] > best_norm) {
                    best_norm = nv[u];
                    best_slot = js[u];
                    have_id = false;
                } else if (nv[u] == best_norm && js[u] != best_slot) {        // rare: equal norms
                    if (!have_id) best_id = pw[best_slot];
                    have_id = true;
                    const int32_t id = pw[js[u]];
                    if ((uint32_t)id > (uint32_t)best_id) {
                        best_id = id;
                        best_slot = js[u];
                    }
                }
            }
        }
        // wave maximum (lanes without a slot hold norm 0), then the lanes that reach it; one as a rule
        const uint32_t top = ~wave_min(~best_norm);
        uint64_t reach = __ballot(best_slot >= 0 && best_norm == top);
        int32_t slot = -1;
        if (reach != 0) {
            if ((reach & (reach - 1)) != 0) {                                 // rare: the largest id among them
                const bool mine = best_slot >= 0 && best_norm == top;
                if (mine && !have_id) best_id = pw[best_slot];
                const uint32_t id = ~wave_min(mine ? ~(uint32_t)best_id : 0xffffffffu);
                reach = __ballot(mine && (uint32_t)best_id == id);
            }
            slot = __builtin_amdgcn_readlane(best_slot, (int)__builtin_ctzll(reach));
        }
        if constexpr (kTeam == kEvictThreads) {
            if (lane == 0) {
                s_norm[wave] = top;
                s_slot[wave] = slot;
            }
            __syncthreads();
            uint32_t norm = s_norm[0];
            slot = s_slot[0];
#pragma unroll
            for (int w = 1; w < kEvictWaves; ++w) {
                const int32_t other = s_slot[w];
                if (other >= 0 && (slot < 0 || s_norm[w] > norm || (s_norm[w] == norm && other != slot && later(other, slot)))) {
                    norm = s_norm[w];
                    slot = other;
                }
            }
        }
        if (slot != last) {
            if (tid < 2 * kRowLanes) {
                store_words<W>(buf + (base + slot) * kRowBytes + c * kSliceBytes, row);
            } else if (tid == 2 * kRowLanes) {
                nw[slot] = last_norm;
                pw[slot] = last_id;
            }
        }
        len = last;
        // moves visible to the team before its next scan (and the LDS reusable)
        if constexpr (kTeam == kEvictThreads) __syncthreads();
        else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    }
    if (plane == 0 && tid == 0) lens_out[seq] = len;
}

l2kv_status stream_evict_dispatch(l2kv_dtype dt, int32_t n_planes, int32_t n_seq, int32_t D,
                                  const int64_t* slot_off, int64_t total_slots, const int32_t* lens_in,
                                  const int32_t* budgets, int32_t* lens_out, void* Kc, void* Vc,
                                  float* norms_c, int32_t* pos_c, hipStream_t stream) {
    const int row_bytes = D * (dt == L2KV_F32 ? 4 : 2);
    const int64_t teams = (int64_t)n_planes * n_seq;
    const bool waves = teams >= kEvictWaveTeams && teams >= 2 * (total_slots / n_seq);
    const int64_t blocks = waves ? (teams + kEvictWaves - 1) / kEvictWaves : teams;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return L2KV_ERR_SHAPE;
#define L2KV_EV(WW)                                                                               \
    hipLaunchKernelGGL((waves ? stream_evict_kernel<WW, kWaveSize> : stream_evict_kernel<WW, kEvictThreads>), \
                       dim3((unsigned)blocks), dim3(kEvictThreads), 0,                            \
                       stream, (int64_t)n_seq, teams, slot_off, total_slots, lens_in, budgets, lens_out,  \
                       static_cast<char*>(Kc), static_cast<char*>(Vc), norms_c, pos_c)
    switch (row_bytes) {
        case 128: L2KV_EV(2); break;
        case 256: L2KV_EV(4); break;
        case 512: L2KV_EV(8); break;
        default: return L2KV_ERR_SHAPE;
    }
#undef L2KV_EV
    return launch_status();
}

// ---------------------------------------------------------------- length order
// order[r] = the sequence with the r-th largest length (equal lengths: lower
// index first), by rank counting in one workgroup: a permutation of 0..n_seq-1
// whatever lens holds.  Meant for batch set-up, not for the decode loop.
constexpr int kOrderLdsSeqs = 8192;    // batches up to this size are ranked out of LDS

__global__ __launch_bounds__(1024)
void length_order_kernel(const int32_t* __restrict__ lens, int32_t n_seq, int32_t from, int32_t* __restrict__ order) {
    __shared__ int32_t s_len[kOrderLdsSeqs];
    const bool in_lds = n_seq <= kOrderLdsSeqs;
    if (in_lds) {
        for (int32_t s = threadIdx.x; s < n_seq; s += (int32_t)blockDim.x) s_len[s] = lens[s];
        __syncthreads();
    }
    for (int32_t s = threadIdx.x; s < n_seq; s += (int32_t)blockDim.x) {
        const int32_t mine = in_lds ? s_len[s] : lens[s];
        int32_t rank = 0;
        if (in_lds) {
            for (int32_t t = 0; t < n_seq; ++t) {
                const int32_t other = s_len[t];
                rank += (other > mine || (other == mine && t < s)) ? 1 : 0;
            }
        } else {
            for (int32_t t = 0; t < n_seq; ++t) {
                const int32_t other = lens[t];
                rank += (other > mine || (other == mine && t < s)) ? 1 : 0;
            }
        }
        order[rank] = from + s;
    }
}

l2kv_status length_order_dispatch(const int32_t* lens, int32_t n_seq, int32_t from, int32_t* order, hipStream_t stream) {
    // small batches need only as many lanes as sequences (fewer waves to start and retire)
    const unsigned threads = n_seq <= 64 ? 64u : (n_seq <= 256 ? 256u : 1024u);
    hipLaunchKernelGGL(length_order_kernel, dim3(1), dim3(threads), 0, stream, lens, n_seq, from, order);
    return launch_status();
}

}  // namespace l2kv
