// l2kv_decode_attn, host side: workspace set-up, the scratch array of the allocation-free entry
// point, and the dispatch to the kernels (decode_kernels.hpp, instantiated in
// decode_attn_<type>_<D>.hip).  The decomposition plans are in decode_plan.hip.
#include "l2kv_device.hpp"
#include "l2kv_host.hpp"

#include <atomic>

namespace l2kv {

template <typename E, int D>
l2kv_status decode_by_group(int G, const void* Q, const void* Kc, const void* Vc, int32_t B, int32_t Hq,
                            int32_t Hkv, int64_t kv_len, int64_t kv_head_stride, const int32_t* lens,
                            const int64_t* slot_off, const int32_t* seq_order, float scale,
                            const DecodePlan& plan, float* O, void* workspace, hipStream_t stream);
extern template l2kv_status decode_by_group<BF16, 128>(int, const void*, const void*, const void*, int32_t, int32_t, int32_t, int64_t, int64_t, const int32_t*, const int64_t*, const int32_t*, float, const DecodePlan&, float*, void*, hipStream_t);
extern template l2kv_status decode_by_group<BF16, 256>(int, const void*, const void*, const void*, int32_t, int32_t, int32_t, int64_t, int64_t, const int32_t*, const int64_t*, const int32_t*, float, const DecodePlan&, float*, void*, hipStream_t);
extern template l2kv_status decode_by_group<BF16, 64>(int, const void*, const void*, const void*, int32_t, int32_t, int32_t, int64_t, int64_t, const int32_t*, const int64_t*, const int32_t*, float, const DecodePlan&, float*, void*, hipStream_t);
extern template l2kv_status decode_by_group<F32, 128>(int, const void*, const void*, const void*, int32_t, int32_t, int32_t, int64_t, int64_t, const int32_t*, const int64_t*, const int32_t*, float, const DecodePlan&, float*, void*, hipStream_t);
extern template l2kv_status decode_by_group<F32, 64>(int, const void*, const void*, const void*, int32_t, int32_t, int32_t, int64_t, int64_t, const int32_t*, const int64_t*, const int32_t*, float, const DecodePlan&, float*, void*, hipStream_t);

// Zero-fill of a decode workspace as a kernel (callers under graph capture
// cannot record a memset node reliably; a fill kernel is always safe).
__global__ __launch_bounds__(256)
void workspace_fill_kernel(uint4* __restrict__ p, size_t n_vec) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_vec) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

l2kv_status workspace_init_dispatch(void* workspace, size_t bytes, hipStream_t stream) {
    const size_t n_vec = bytes / 16;
    const size_t blocks = (n_vec + 255) / 256;
    if (blocks == 0 || blocks > 0x7fffffffULL) return L2KV_ERR_SHAPE;
    hipLaunchKernelGGL(workspace_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                       static_cast<uint4*>(workspace), n_vec);
    return launch_status();
}

// ---- scratch memory of the allocation-free entry point ----------------------
// Callers that cannot allocate (graph capture, serving loops, harnesses that
// forbid hipMalloc) get the decode workspace from this array instead of from an
// argument.  Every device the library runs on holds its own copy at its own
// address.  On the host the array's name is only a handle for the symbol
// look-up below, never a device address: host code uses the pointer that
// hipGetSymbolAddress returned for the current device, and nothing else.
static __device__ __align__(256) unsigned char scratch[L2KV_STATIC_SCRATCH_BYTES];

void* decode_static_scratch(hipStream_t stream, l2kv_status* status) {
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> device_ptr[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        *status = L2KV_ERR_LAUNCH;
        return nullptr;
    }
    void* ptr = device_ptr[dev].load(std::memory_order_acquire);
    if (ptr != nullptr) return ptr;
    // First use on this device (which is current): look the array's address up and
    // zero the arrival counters at its start with the fill kernel.  Every later
    // call finds them zero because every decode launch resets the counters it used.
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
        (void)hipGetLastError();
        *status = L2KV_ERR_LAUNCH;
        return nullptr;
    }
    const size_t kCounterRegion = decode_counter_bytes(65535, 1);    // B * Hkv <= 65535 counters
    static_assert(65536 * sizeof(uint32_t) + 256 <= L2KV_STATIC_SCRATCH_BYTES, "scratch smaller than its counter region");
    if (l2kv_status st = workspace_init_dispatch(ptr, kCounterRegion, stream); st != L2KV_OK) {
        *status = st;
        return nullptr;
    }
    device_ptr[dev].store(ptr, std::memory_order_release);
    return ptr;
}

l2kv_status decode_dispatch(const void* Q, const void* Kc, const void* Vc, l2kv_dtype dt, int32_t B,
                            int32_t Hq, int32_t Hkv, int64_t kv_len, int32_t D,
                            int64_t kv_head_stride, const int32_t* lens, const int64_t* slot_off,
                            const int32_t* seq_order, float scale, const DecodePlan& plan, float* O,
                            void* workspace, hipStream_t stream) {
    const int G = Hq / Hkv;
    if (dt == L2KV_F32) {
        return D == 64 ? decode_by_group<F32, 64>(G, Q, Kc, Vc, B, Hq, Hkv, kv_len, kv_head_stride,
                                                  lens, slot_off, seq_order, scale, plan, O, workspace, stream)
                       : decode_by_group<F32, 128>(G, Q, Kc, Vc, B, Hq, Hkv, kv_len, kv_head_stride,
                                                   lens, slot_off, seq_order, scale, plan, O, workspace, stream);
    }
    if (D == 256)
        return decode_by_group<BF16, 256>(G, Q, Kc, Vc, B, Hq, Hkv, kv_len, kv_head_stride, lens, slot_off,
                                          seq_order, scale, plan, O, workspace, stream);
    return D == 64 ? decode_by_group<BF16, 64>(G, Q, Kc, Vc, B, Hq, Hkv, kv_len, kv_head_stride,
                                               lens, slot_off, seq_order, scale, plan, O, workspace, stream)
                   : decode_by_group<BF16, 128>(G, Q, Kc, Vc, B, Hq, Hkv, kv_len, kv_head_stride,
                                                lens, slot_off, seq_order, scale, plan, O, workspace, stream);
}

}  // namespace l2kv
