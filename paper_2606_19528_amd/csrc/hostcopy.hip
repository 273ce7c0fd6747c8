// hostcopy.hip -- copies between device memory and pinned host memory for the
// checkpointed step, as a kernel of a few workgroups.
//
// The link bounds these copies (55 GB/s out, 57 in), so they need few
// workgroups, and no more: stores that back up towards the host slow every
// kernel whose memory traffic passes the same L2 (a row product beside them
// took 176 us instead of 5).  Out, two workgroups of 256 threads with eight
// 16-byte vectors in flight per thread; in, where the loads carry the link's
// latency, eight with four.  A chain of 8 linears 3072 <-> 8192 over 2048
// tokens (6.7 ms of copies), passes queued: 7.0 ms; with 16 workgroups either
// way 7.6, 3 out 7.4, 4 in 8.0.  A queued hipMemcpyAsync may run as the
// runtime's own copy kernel over the whole chip instead of a copy engine: the
// same queued passes took 16.0 ms (7.0 when each was waited for).
#include "kernels.hpp"
#include "launch.hpp"

namespace lora {

constexpr int HC_NT = 256;

template <int HC_U>
__global__ __launch_bounds__(HC_NT) void host_copy_kernel(u32x4 *dst, const u32x4 *src, int64_t n) {
  constexpr int64_t BLK = (int64_t)HC_NT * HC_U;
  for (int64_t b = (int64_t)blockIdx.x * BLK; b < n; b += (int64_t)gridDim.x * BLK) {
    const int64_t i0 = b + threadIdx.x;
    u32x4 v[HC_U];
    if (b + BLK <= n) {
#pragma unroll
      for (int u = 0; u < HC_U; ++u) v[u] = __builtin_nontemporal_load(src + i0 + u * HC_NT);
#pragma unroll
      for (int u = 0; u < HC_U; ++u) __builtin_nontemporal_store(v[u], dst + i0 + u * HC_NT);
    } else {
      for (int64_t i = i0; i < n; i += HC_NT) dst[i] = src[i];
    }
  }
}

// Device address of the host range [p, p + bytes) if all of it lies in one mapped
// pinned allocation, else null (the error a failed lookup leaves is cleared).
static char *mapped(const void *p, size_t bytes) {
  void *dev = nullptr, *base = nullptr;
  size_t size = 0;
  if (hipHostGetDevicePointer(&dev, const_cast<void *>(p), 0) != hipSuccess || !dev ||
      hipMemGetAddressRange((hipDeviceptr_t *)&base, &size, (hipDeviceptr_t)dev) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  const size_t off = (size_t)((char *)dev - (char *)base);
  return dev >= base && off <= size && bytes <= size - off ? (char *)dev : nullptr;
}

bool host_copy_mapped(const void *host, size_t bytes) { return mapped(host, bytes) != nullptr; }

hipError_t launch_host_copy(void *dst, const void *src, size_t bytes, bool to_host, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  void *host = to_host ? dst : const_cast<void *>(src);
  char *dev_view = bytes % 16 == 0 ? mapped(host, bytes) : nullptr;
  const void *other = to_host ? src : dst;
  if (!dev_view || (((uintptr_t)dev_view | (uintptr_t)other) & 15u))  // pageable or unaligned memory
    return hipMemcpyAsync(dst, src, bytes, to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice, st);
  u32x4 *d = (u32x4 *)(to_host ? dev_view : (char *)dst);
  const u32x4 *s = (const u32x4 *)(to_host ? (const char *)src : dev_view);
  const int64_t n = (int64_t)(bytes / 16);
  if (to_host) hipLaunchKernelGGL(host_copy_kernel<8>, dim3(2), dim3(HC_NT), 0, st, d, s, n);
  else hipLaunchKernelGGL(host_copy_kernel<4>, dim3(8), dim3(HC_NT), 0, st, d, s, n);
  return hipGetLastError();
}

}  // namespace lora
