// Live-bytes profile of one trace: live[t] = sum of the sizes of the tensors
// alive at op t (first <= t <= last), and its maximum -- a lower bound on the
// arena size of any valid plan, since every tensor alive at t needs its own
// bytes.  Difference array (+size at first, -size at last + 1), then an
// inclusive device-wide prefix sum.  A workgroup takes consecutive tensors, which
// in a recorded trace use consecutive ops: it adds up a window of ops in LDS and
// sends one device atomic for each op of it; ops outside go to memory directly.
// 1 M tensors: 84 us with an atomic for each end (2 M of them), 11 us so; bound by
// the reading then.  A workgroup's tensors are a 256th of all: with one birth an op
// those beyond 1 M in all leave the window (the whole call for 2 M 145 -> 121 us,
// 4 M 250 -> 228); in any order, where hardly any are in it, it is even (148, 142).
#include <mutex>

#include "internal.hpp"
#include "mp_device.hpp"

namespace mp {

namespace {

// Workgroups add to one word, so there are few, one a CU.  Up to a tensor for
// each thread of 256 small ones there is no window: the few atomics go to memory
// at once, where the window's two barriers cost 2 us.
constexpr int kLiveGrid = 256;
constexpr int kLiveSmall = 256, kLiveLarge = 1024;
constexpr int kLiveWindow = 4096;   // ops

__global__ void live_init_kernel(int64_t* __restrict__ live, int32_t num_ops,
                                 int64_t* __restrict__ max_out, uint64_t* __restrict__ sum) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < num_ops; t += stride)
        live[t] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *max_out = 0;
        *sum = 0;
    }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void live_delta_kernel(
    const int64_t* __restrict__ size, const int32_t* __restrict__ first,
    const int32_t* __restrict__ last, int64_t n, int32_t num_ops, int64_t* __restrict__ live,
    uint64_t* __restrict__ sum, int32_t* __restrict__ status) {
    __shared__ uint64_t red[BLOCK / kWave];
    constexpr bool kWindow = BLOCK == kLiveLarge;
    __shared__ unsigned long long win[kWindow ? kLiveWindow : 1];
    const int64_t lo = n * blockIdx.x / gridDim.x, hi = n * (blockIdx.x + 1) / gridDim.x;
    uint32_t bad = 0;
    uint64_t acc = 0;
    int32_t base = 0, window = 0;
    if constexpr (kWindow) {
        base = lo < hi ? min(max(first[lo], 0), num_ops) : 0;
        window = min(kLiveWindow, num_ops - base);
        for (int w = threadIdx.x; w < window; w += BLOCK) win[w] = 0;
        __syncthreads();
    }
    auto add = [&](int32_t t, unsigned long long v) {
        if (kWindow && t >= base && t - base < window) atomicAdd(&win[t - base], v);
        else atomicAdd(reinterpret_cast<unsigned long long*>(live + t), v);
    };
    for (int64_t i = lo + threadIdx.x; i < hi; i += BLOCK) {
        const int64_t s = size[i];
        const int32_t f = first[i], l = last[i];
        if (s <= 0 || f < 0 || f > l || l >= num_ops) {
            bad = 1;
            if (s > 0) acc = sat_add(acc, (uint64_t)s);
            continue;  // no writes for a tensor outside the op range
        }
        acc = sat_add(acc, (uint64_t)s);
        add(f, (unsigned long long)s);
        if (l + 1 < num_ops) add(l + 1, (unsigned long long)(-s));
    }
    if constexpr (kWindow) __syncthreads();
    for (int w = threadIdx.x; w < window; w += BLOCK)
        if (win[w]) atomicAdd(reinterpret_cast<unsigned long long*>(live + base + w), win[w]);
    bad = block_reduce<BLOCK>(bad, OpOr<uint32_t>(), reinterpret_cast<uint32_t*>(red));
    acc = block_reduce<BLOCK>(acc, OpSatAdd(), red);
    if (threadIdx.x == 0) {
        if (bad) raise_status(status, MP_EINVAL);
        // global saturating sum: once past INT64_MAX the overflow is reported
        const uint64_t old = atomicAdd(reinterpret_cast<unsigned long long*>(sum),
                                       (unsigned long long)acc);
        if (acc > (uint64_t)INT64_MAX || old > (uint64_t)INT64_MAX - acc)
            raise_status(status, MP_EOVERFLOW);
    }
}

}  // namespace

size_t live_workspace_bytes(int32_t num_ops) {
    return 256 + scan_workspace_bytes(num_ops > 0 ? num_ops : 1);
}

hipError_t launch_live_profile(const int64_t* size, const int32_t* first, const int32_t* last,
                               int64_t n, int32_t num_ops, int64_t* live_out, int64_t* max_out,
                               void* ws, int32_t* status, hipStream_t st) {
    uint64_t* sum = static_cast<uint64_t*>(ws);
    int64_t* partial = reinterpret_cast<int64_t*>(static_cast<char*>(ws) + 256);
    const int64_t ig = ((int64_t)num_ops + 255) / 256 + 1;
    const unsigned init_grid = (unsigned)(ig < 1024 ? ig : 1024);
    hipLaunchKernelGGL(live_init_kernel, dim3(init_grid), dim3(256), 0, st, live_out, num_ops,
                       max_out, sum);
    if (n > 0) {
        const int64_t g = (n + kLiveSmall - 1) / kLiveSmall;
        if (g <= kLiveGrid)
            hipLaunchKernelGGL(live_delta_kernel<kLiveSmall>, dim3((unsigned)g), dim3(kLiveSmall), 0,
                               st, size, first, last, n, num_ops, live_out, sum, status);
        else
            hipLaunchKernelGGL(live_delta_kernel<kLiveLarge>, dim3(kLiveGrid), dim3(kLiveLarge), 0,
                               st, size, first, last, n, num_ops, live_out, sum, status);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return device_scan_i64(live_out, num_ops, true, partial,
                           reinterpret_cast<unsigned long long*>(max_out), st);
}

// ---- the same profile without a caller workspace (no allocation anywhere)
//
// Scratch of mp_live_bytes_profile_noalloc: the running-sum word and the
// scan's tile partials, for at most MP_LIVE_NOALLOC_MAX_OPS ops.  Each GPU
// the library runs on holds one copy until the process ends; every call on a
// GPU shares it.  Host code never passes `scratch` itself to a kernel (on the
// host it is only a stand-in for the symbol): the device address is looked up
// once per device with that device current and kept in scratch_ptr.
namespace {

constexpr size_t kNoallocScratchBytes = 256 + ((size_t)MP_LIVE_NOALLOC_MAX_OPS / 2048 + 2) * 8;
__device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];

// Device address of this device's scratch (looked up on first use), or
// nullptr if it cannot be resolved.
void* scratch_ptr() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

size_t live_noalloc_scratch_bytes() { return kNoallocScratchBytes; }

hipError_t launch_live_profile_noalloc(const int64_t* size, const int32_t* first,
                                       const int32_t* last, int64_t n, int32_t num_ops,
                                       int64_t* live_out, int64_t* max_out, int32_t* status,
                                       hipStream_t st) {
    static_assert(kNoallocScratchBytes >= 256 + (MP_LIVE_NOALLOC_MAX_OPS + 2047) / 2048 * 8 + 8,
                  "scratch holds the sum word and every tile partial");
    if (num_ops < 0 || live_workspace_bytes(num_ops) > kNoallocScratchBytes)
        return hipErrorInvalidValue;
    void* ws = scratch_ptr();
    if (!ws) return hipErrorInvalidSymbol;
    return launch_live_profile(size, first, last, n, num_ops, live_out, max_out, ws, status, st);
}

}  // namespace mp
