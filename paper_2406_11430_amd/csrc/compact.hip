// l2kv_compact: gather of the kept K and V rows into dense caches (arXiv
// 2406.11430 Sec. 1: the lowest-norm keys are kept, each with its value).
//
// A byte copy of whole rows: 16 lanes move one row (16 bytes per lane and
// instruction: one piece of a 256-byte row, pieces c and c + 16 of a 512-byte
// row; 8 lanes share a 128-byte row), a wavefront moves 4 rows (8 short ones) per instruction.  Loads and stores carry the non-temporal hint (every byte is
// touched once).  Dropped rows are never read.
//
// Memory-bound: half of the rows of 256 heads of 32k (4.3 GB in and out) move at 6.2 TB/s (690 us; a plain copy
// of 4 GiB through the runtime reaches 4.8).  K and V go through workgroups of their own, which alternate in
// the launch: one read and one write stream per workgroup, and one row in flight per row group, disturb
// each other less than two of each and four rows (732 us).  Launches so small that all workgroups run at once
// take the two together (the launcher has the line).  Ordinary loads or stores instead of
// non-temporal ones: 768 and 772 us; every compute die on a range of its own: 771 us.
#include "l2kv_device.hpp"
#include "l2kv_host.hpp"

namespace l2kv {

constexpr int kCompactThreads = 256;
constexpr int kCompactWaves = kCompactThreads / kWaveSize;
template <int kRowBytes, int kUnroll>
constexpr int kCompactRowsPerBlock = kCompactWaves * RowCopy<kRowBytes>::kRowsPerWave * kUnroll;

// Who copies K and who V: workgroups of their own in turn, or the same ones; or there is no V.
enum class Tensors { kInTurn, kTogether, kKeysOnly };

// kUnroll: rows of a row group, all loaded before the first is stored.
template <int kRowBytes, Tensors kTensors, int kUnroll>
__global__ __launch_bounds__(kCompactThreads)
void compact_kernel(const char* __restrict__ K, const char* __restrict__ V,
                    const int32_t* __restrict__ kept_idx, int64_t T, int64_t k, int64_t head_stride_bytes,
                    uint32_t first_block, char* __restrict__ Kc, char* __restrict__ Vc) {
    using P = RowCopy<kRowBytes>;
    constexpr int W = P::kWords;
    // from the end: the norm pass has left the last rows of K in the caches (kReadAgainBytes)
    const int64_t head = gridDim.y - 1 - blockIdx.y;
    const uint32_t block = first_block + gridDim.x - 1 - blockIdx.x;
    const uint32_t chunk = kTensors == Tensors::kInTurn ? block / 2 : block;
    const bool is_v = kTensors == Tensors::kInTurn && block % 2 != 0;          // odd workgroups are V's
    const int lane = threadIdx.x % kWaveSize;
    const int wave = threadIdx.x / kWaveSize;
    const int c = lane % P::kLanes;
    const int rg = lane / P::kLanes;

    const int64_t first = (int64_t)chunk * kCompactRowsPerBlock<kRowBytes, kUnroll> + (wave * P::kRowsPerWave + rg) * kUnroll;
    const int32_t* idx = kept_idx + head * k;
    const int64_t from = head * head_stride_bytes + c * 16, to = head * k * kRowBytes + c * 16;
    const char* src = (is_v ? V : K) + from;
    char* dst = (is_v ? Vc : Kc) + to;

    int64_t t[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int64_t j = first + u;
        const int64_t row = idx[j < k ? j : k - 1];   // tail: duplicate the last row, store skipped
        t[u] = row < 0 ? 0 : (row < T ? row : T - 1);  // an index outside [0, T) cannot lead out of the head
    }
    Words<W> rows[kUnroll], v_rows[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) rows[u] = load_words_stream<W, P::kStride>(src + t[u] * (int64_t)kRowBytes);
    if constexpr (kTensors == Tensors::kTogether) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) v_rows[u] = load_words_stream<W, P::kStride>(V + from + t[u] * (int64_t)kRowBytes);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        if (first + u < k) {
            store_words_stream<W, P::kStride>(dst + (first + u) * kRowBytes, rows[u]);
            if constexpr (kTensors == Tensors::kTogether) store_words_stream<W, P::kStride>(Vc + to + (first + u) * kRowBytes, v_rows[u]);
        }
    }
}

template <int kRowBytes>
static l2kv_status launch_compact(const void* K, const void* V, const int32_t* kept_idx,
                                  int64_t n_heads, int64_t T, int64_t k, int64_t head_stride_bytes,
                                  void* Kc, void* Vc, hipStream_t stream) {
    if ((k + 63) / 64 * n_heads > 0x7fffffffLL) return L2KV_ERR_SHAPE;
    constexpr int64_t kFew = kCompactRowsPerBlock<kRowBytes, 4>, kMany = kCompactRowsPerBlock<kRowBytes, 1>;
    const int64_t few = (k + kFew - 1) / kFew, many = (k + kMany - 1) / kMany;
    // While workgroups of 64 rows (128 short ones) of K and V all run at once, 16 MB of either, fewer and larger ones are the
    // better: the eight times as many small ones are bound by how fast they start.  Half of 4k rows, us, together and in turn: 16 heads of
    // 256-byte rows (512 workgroups) 7.5, 8.5; 32 heads 13.3, 13.8; 64 heads 24.4, 24.3; 16 heads of 512-byte rows 12.4, 13.9; 32 heads
    // of 128-byte rows 7.5, 8.4; 32 heads of 512-byte rows (32 MB) 24.0, 24.5, but 0.9 of 16 of them within l2kv_compress 33.8,
    // 31.3.  With fewer rows than a workgroup takes: 1000 heads of 32 rows 7.7, 7.1.
    const bool together = V != nullptr && n_heads * few * kFew * kRowBytes <= int64_t{16} << 20 && k >= kFew;
    const int64_t bph = together ? few : V != nullptr ? 2 * many : many;
    auto kernel = together ? compact_kernel<kRowBytes, Tensors::kTogether, 4>
                  : V != nullptr ? compact_kernel<kRowBytes, Tensors::kInTurn, 1> : compact_kernel<kRowBytes, Tensors::kKeysOnly, 1>;
    constexpr int64_t kMaxX = 1 << 23, kMaxY = 65535;      // a launch has fewer than 2^32 lanes in x, 2^16 workgroups in y
    for (int64_t h1 = n_heads; h1 > 0; h1 -= kMaxY) {
        const int64_t nh = h1 < kMaxY ? h1 : kMaxY, h0 = h1 - nh;
        const int64_t dense = h0 * k * kRowBytes;
        for (int64_t b0 = 0; b0 < bph; b0 += kMaxX) {
            const int64_t nb = bph - b0 < kMaxX ? bph - b0 : kMaxX;
            hipLaunchKernelGGL(kernel, dim3((unsigned)nb, (unsigned)nh), dim3(kCompactThreads), 0, stream,
                               static_cast<const char*>(K) + h0 * head_stride_bytes,
                               V != nullptr ? static_cast<const char*>(V) + h0 * head_stride_bytes : nullptr,
                               kept_idx + h0 * k, T, k, head_stride_bytes, (uint32_t)b0, static_cast<char*>(Kc) + dense,
                               V != nullptr ? static_cast<char*>(Vc) + dense : nullptr);
            if (l2kv_status st = launch_status(); st != L2KV_OK) return st;
        }
    }
    return L2KV_OK;
}

l2kv_status compact_dispatch(const void* K, const void* V, l2kv_dtype dt, const int32_t* kept_idx,
                             int64_t n_heads, int64_t T, int64_t k, int32_t D, int64_t head_stride,
                             void* Kc, void* Vc, hipStream_t stream) {
    const int es = dt == L2KV_F32 ? 4 : 2;
    const int row_bytes = D * es;                      // 128, 256 or 512
    const int64_t hs_bytes = head_stride * es;
    switch (row_bytes) {
        case 128: return launch_compact<128>(K, V, kept_idx, n_heads, T, k, hs_bytes, Kc, Vc, stream);
        case 256: return launch_compact<256>(K, V, kept_idx, n_heads, T, k, hs_bytes, Kc, Vc, stream);
        case 512: return launch_compact<512>(K, V, kept_idx, n_heads, T, k, hs_bytes, Kc, Vc, stream);
    }
    return L2KV_ERR_SHAPE;
}

}  // namespace l2kv
