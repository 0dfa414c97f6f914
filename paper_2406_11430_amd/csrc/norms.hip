// l2kv_norms: squared L2 norm of every cached key row (the quantity the
// eviction rule of arXiv 2406.11430, Sec. 1 / Sec. 3, ranks by).
//
// Pure HBM read stream of K.  16 lanes share a row (one 16-byte load each for
// the 256-byte rows of the supported shapes), a wavefront covers 4 rows per
// load instruction, and every row group takes kNormUnroll consecutive rows
// with independent non-temporal loads.  Small workgroups (32 rows) and very
// many of them measured best: the hardware keeps enough of them in flight.
// The per-row sum follows the library's fixed order: per-lane chunk left to
// right, then the balanced tree of row16_tree_sum.  Contraction to FMA is
// switched off so fp32 inputs round product and sum separately, like the stated
// order says.
//
// 512-byte rows (two 16-byte pieces per lane) are loaded with the row shared among
// the lanes piece by piece (lane c: pieces c and c + 16), which streams better than
// 32 consecutive bytes per lane.  The fixed order is defined over 32-byte chunks,
// chunk i = pieces 2i and 2i + 1, so the left-to-right sum of a chunk runs through
// two neighbouring lanes: the even lane sums its piece, hands the sum to the odd
// lane, which continues over its own piece; the tree then runs over the odd lanes of
// each piece slot and the two slots are added last (chunks 0..7 + chunks 8..15).
#include "l2kv_device.hpp"
#include "l2kv_host.hpp"
#include "row_norm.hpp"

#include <type_traits>

namespace l2kv {

constexpr int kNormThreads = 256;
constexpr int kNormWaves = kNormThreads / kWaveSize;
#ifndef L2KV_NORM_UNROLL
#define L2KV_NORM_UNROLL 2
#endif
constexpr int kNormUnroll = L2KV_NORM_UNROLL;                    // rows per row group
constexpr int kNormRowsPerBlock = kNormWaves * kRowsPerWaveLoad * kNormUnroll;  // 32

// How a pass treats the caches.
//  kStream  rows and results are non-temporal
//  kResults rows are, results are ordinary stores: better up to 1 GiB of K and 16 MB of norms (half of the L2s).  Heads of
//           32k rows: 8 of 128 elements in bf16 12.1 against 12.4 us, 64 of them 78.1 against 80.4, 120 (1 GiB) 148.7 against
//           149.5; the other way round 200 of them 251.4 against 249.2, 1024 1314 against 1284, 200 of 64 elements (0.8 GiB,
//           26 MB of norms) 131.6 against 128.1, 100 of 128 elements in fp32 (1.7 GB, 13 MB) 251.3 against 244.9
//  kTail    as kResults, and workgroups from chunk keep_chunk of head keep_head on read with ordinary loads: the rows
//           that were read last then stay in the 256 MB memory-side cache for the compaction, which reads the kept ones
//           again (kReadAgainBytes)
// A template argument and no condition at run time: two stores that differ in the hint alone are merged into one
// without it.
enum class NormCaching { kStream, kResults, kTail };
template <NormCaching C>
__device__ __forceinline__ void store_norm(float* p, float v) {
    if constexpr (C == NormCaching::kStream) __builtin_nontemporal_store(v, p);
    else *p = v;
}
constexpr int64_t kPlainResultBytes = int64_t{16} << 20, kPlainResultKeys = int64_t{1} << 30;

template <typename E, int D, NormCaching C>
__global__ __launch_bounds__(kNormThreads)
void norms_kernel(const char* __restrict__ K, int64_t T, int64_t head_stride_bytes,
                  int64_t blocks_per_head, float* __restrict__ norms, int32_t keep_head, int32_t keep_chunk) {
#pragma clang fp contract(off)
    using S = Slice<E, D>;
    using P = Pieces<S::kWords>;
    static_assert(P::kCount <= 2, "rows of at most 512 bytes");
    // grid (chunks, heads) when the head count fits the y dimension; else one long x dimension
    // cut by a 32-bit division (the launcher checked that the block count fits 31 bits)
    const int64_t head = blocks_per_head == 0 ? blockIdx.y : blockIdx.x / (uint32_t)blocks_per_head;
    const int64_t chunk = blocks_per_head == 0 ? blockIdx.x : blockIdx.x % (uint32_t)blocks_per_head;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    const int c = lane % kRowLanes;       // slice within the row
    const int rg = lane / kRowLanes;      // row group within the wave

    // Row group (wave, rg) owns kNormUnroll consecutive rows.
    const int local = (wave * kRowsPerWaveLoad + rg) * kNormUnroll;          // first of them, within the block
    const int64_t first = chunk * kNormRowsPerBlock + local;

    // The block's rows through a buffer descriptor: the base is uniform (scalar arithmetic),
    // the lanes add 32-bit offsets, and rows past the end of the head read as zero (their
    // results are not stored), so the short-lived workgroups spend no vector instructions on
    // 64-bit addresses or on clamping.
    const int64_t left = T - chunk * kNormRowsPerBlock;                       // rows of the head from here on
    const int rows_here = left < kNormRowsPerBlock ? (int)left : kNormRowsPerBlock;
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(K + head * head_stride_bytes + chunk * (int64_t)(kNormRowsPerBlock * S::kRowBytes)), 0,
        rows_here * S::kRowBytes, kRawBufferWord3);
    const bool keep = C == NormCaching::kTail && ((int32_t)head > keep_head || ((int32_t)head == keep_head && (int32_t)chunk >= keep_chunk));
    Words<S::kWords> raw[kNormUnroll];
    if (keep) {
#pragma unroll
        for (int u = 0; u < kNormUnroll; ++u)
            raw[u] = buffer_load_words<S::kWords, P::kStride, kBufferPolicyPlain>(rows, (local + u) * S::kRowBytes + c * P::kBytes);
    } else {
#pragma unroll
        for (int u = 0; u < kNormUnroll; ++u)
            raw[u] = buffer_load_words<S::kWords, P::kStride, kBufferPolicyStream>(rows, (local + u) * S::kRowBytes + c * P::kBytes);
    }

    float mine = 0.f;
#pragma unroll
    for (int u = 0; u < kNormUnroll; ++u) {
        float x[S::kElems];
        widen<E, D>(raw[u], x);
        const float total = chunked_sum_of_squares<E, D>(x);
        mine = (c == u) ? total : mine;   // lane c keeps the sum of row u
    }
    const int64_t row = first + c;
    if (c < kNormUnroll && row < T) store_norm<C>(norms + head * T + row, mine);
}

// 128-byte rows (bf16, 64 elements): two consecutive rows are 256 contiguous bytes, so the 16
// lanes of a row group take a PAIR of rows with one 16-byte load each (lanes 0..7 the even row,
// lanes 8..15 the odd one) instead of one row with 8-byte loads.  A lane then holds two of the
// 16 chunks of the fixed summation order (chunk = 4 elements): it sums each left to right, adds
// the two (first level of the tree), and the remaining three levels run over the 8 lanes of
// its row.  Bit-identical to the one-row-per-row-group kernel above.
template <NormCaching C>
__global__ __launch_bounds__(kNormThreads)
void norms_row_pairs_kernel(const char* __restrict__ K, int64_t T, int64_t head_stride_bytes,
                            int64_t blocks_per_head, float* __restrict__ norms, int32_t keep_head, int32_t keep_chunk) {
#pragma clang fp contract(off)
    constexpr int kRowBytes = 128;
    // grid (chunks, heads) when the head count fits the y dimension; else one long x dimension
    // cut by a 32-bit division (the launcher checked that the block count fits 31 bits)
    const int64_t head = blocks_per_head == 0 ? blockIdx.y : blockIdx.x / (uint32_t)blocks_per_head;
    const int64_t chunk = blocks_per_head == 0 ? blockIdx.x : blockIdx.x % (uint32_t)blocks_per_head;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    const int c = lane % kRowLanes;
    const int rg = lane / kRowLanes;
    const int half = c / 8;               // which row of the pair
    const int j = c % 8;                  // 16-byte piece of that row

    // Row group (wave, rg) owns kNormUnroll consecutive pairs of rows.
    const int64_t first = chunk * kNormRowsPerBlock + (wave * kRowsPerWaveLoad + rg) * kNormUnroll;   // in pairs
    const char* head_base = K + head * head_stride_bytes;

    const bool keep = C == NormCaching::kTail && ((int32_t)head > keep_head || ((int32_t)head == keep_head && (int32_t)chunk >= keep_chunk));
    Words<4> raw[kNormUnroll];
#pragma unroll
    for (int u = 0; u < kNormUnroll; ++u) {
        int64_t row = 2 * (first + u) + half;
        row = row < T ? row : T - 1;      // tail: re-read the last row, result unused
        const char* p = head_base + row * kRowBytes + j * 16;
        if (keep) raw[u] = load_words<4>(p);
        else raw[u] = load_words_stream<4>(p);
    }

    float mine = 0.f;
#pragma unroll
    for (int u = 0; u < kNormUnroll; ++u) {
        const float v = row_pair_sum_of_squares(raw[u]);  // of this lane's row
        mine = (j == u) ? v : mine;       // lane j of each half keeps the sum of pair u's row
    }
    const int64_t row = 2 * (first + j) + half;
    if (j < kNormUnroll && row < T) store_norm<C>(norms + head * T + row, mine);
}

template <typename E, int D>
static l2kv_status launch_norms(const void* K, int64_t n_heads, int64_t T, int64_t head_stride,
                                float* norms, int64_t read_again_bytes, hipStream_t stream) {
    constexpr bool kPairs = Slice<E, D>::kRowBytes == 128;                    // a block takes twice the rows then
    const int64_t rows_per_block = kNormRowsPerBlock * (kPairs ? 2 : 1);
    const int64_t bph = (T + rows_per_block - 1) / rows_per_block;
    const int64_t blocks = bph * n_heads;
    if (blocks > 0x7fffffffLL) return L2KV_ERR_SHAPE;
    // not where it would be a small part of K
    const int64_t block_bytes = rows_per_block * Slice<E, D>::kRowBytes;
    const int64_t kept_blocks = blocks * block_bytes <= 8 * read_again_bytes ? read_again_bytes / block_bytes : 0;
    auto pick = [](auto caching) {
        constexpr NormCaching kC = decltype(caching)::value;
        if constexpr (kPairs) return norms_row_pairs_kernel<kC>;
        else return norms_kernel<E, D, kC>;
    };
    auto kernel = kept_blocks > 0 ? pick(std::integral_constant<NormCaching, NormCaching::kTail>{})
                  : n_heads * T * (int64_t)sizeof(float) <= kPlainResultBytes && blocks * block_bytes <= kPlainResultKeys
                      ? pick(std::integral_constant<NormCaching, NormCaching::kResults>{})
                      : pick(std::integral_constant<NormCaching, NormCaching::kStream>{});
    const int64_t keep_from = blocks > kept_blocks ? blocks - kept_blocks : 0;     // counted head by head
    const bool grid2d = n_heads <= 65535;
    hipLaunchKernelGGL(kernel, grid2d ? dim3((unsigned)bph, (unsigned)n_heads) : dim3((unsigned)blocks),
                       dim3(kNormThreads), 0, stream, static_cast<const char*>(K), T,
                       head_stride * (int64_t)E::kBytes, grid2d ? (int64_t)0 : bph, norms, (int32_t)(keep_from / bph),
                       (int32_t)(keep_from % bph));
    return launch_status();
}

// Measurement aid: the bare read stream.  Same access pattern as the norm pass (256 lanes, two
// 16-byte non-temporal loads each, 8 KiB per workgroup), nothing computed but an XOR over the
// lanes, nothing stored (the store below needs a 32-bit coincidence).  What it reaches is the
// ceiling for any kernel that streams this buffer once.
constexpr int kProbeBytesPerBlock = kNormThreads * 16 * 2;
__global__ __launch_bounds__(kNormThreads)
void read_probe_kernel(const char* __restrict__ data, uint32_t* __restrict__ sink) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t block = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(data + (int64_t)blockIdx.x * kProbeBytesPerBlock), 0, kProbeBytesPerBlock, kRawBufferWord3);
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(block, (int)threadIdx.x * 16, 0, kBufferPolicyStream);
    const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(block, (int)threadIdx.x * 16 + kNormThreads * 16, 0, kBufferPolicyStream);
    const uint32_t x = a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w;
    if (x == 0x9E3779B9u) sink[0] = x;
}

l2kv_status read_probe_dispatch(const void* data, size_t bytes, uint32_t* sink, hipStream_t stream) {
    const size_t blocks = bytes / kProbeBytesPerBlock;
    if (blocks == 0 || blocks > 0x7fffffffULL) return L2KV_ERR_SHAPE;
    hipLaunchKernelGGL(read_probe_kernel, dim3((unsigned)blocks), dim3(kNormThreads), 0, stream,
                       static_cast<const char*>(data), sink);
    return launch_status();
}

l2kv_status norms_dispatch(const void* K, l2kv_dtype dt, int64_t n_heads, int64_t T, int32_t D,
                           int64_t head_stride, float* norms, int64_t read_again_bytes, hipStream_t stream) {
    if (dt == L2KV_F32) {
        return D == 64 ? launch_norms<F32, 64>(K, n_heads, T, head_stride, norms, read_again_bytes, stream)
                       : launch_norms<F32, 128>(K, n_heads, T, head_stride, norms, read_again_bytes, stream);
    }
    if (D == 256) return launch_norms<BF16, 256>(K, n_heads, T, head_stride, norms, read_again_bytes, stream);
    return D == 64 ? launch_norms<BF16, 64>(K, n_heads, T, head_stride, norms, read_again_bytes, stream)
                   : launch_norms<BF16, 128>(K, n_heads, T, head_stride, norms, read_again_bytes, stream);
}

}  // namespace l2kv
