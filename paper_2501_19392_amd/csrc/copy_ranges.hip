// Many device-to-device copies in one launch: the row moves of the cache manager (new tokens of every layer and sequence
// into sinks and recent buffers, gathering full buffers, scattering codes to the sequences' ranges).  A generated token is
// 2 x layers x sequences rows of 2 KiB; as one copy each they cost 6 us of host time apiece, as one launch some 3 us of
// GPU time whatever their number (8 layers, 4 sequences: 64 copies).  Bound by launch latency for single tokens, by HBM
// for gathered prompts; a range is cut into slices of 16 KiB (one workgroup of 256 threads, four 16-byte moves per thread)
// so that one long range still fills the chip.
#include "device_utils.h"
#include "kernels.h"

namespace aquakv {
namespace {

constexpr int kThreads = 256;
constexpr int kSlice = kThreads * 64;             // bytes one workgroup moves per step
struct Ranges { CopyRange r[kCopyRangesPerLaunch]; };   // by value: the launch carries the list, nothing is kept

template <typename T> __device__ __forceinline__ void copy_units(const CopyRange& c, int64_t first, int64_t step) {
  const int64_t n = (int64_t)(c.bytes / sizeof(T));
  const T* src = static_cast<const T*>(c.src);
  T* dst = static_cast<T*>(c.dst);
  for (int64_t i = first; i < n; i += step) dst[i] = src[i];
}

__global__ __launch_bounds__(kThreads) void copy_ranges_kernel(const Ranges list) {
  const CopyRange c = list.r[blockIdx.y];
  const uint64_t low = reinterpret_cast<uint64_t>(c.dst) | reinterpret_cast<uint64_t>(c.src) | c.bytes;
  if ((low & 15) == 0) {
    for (int64_t at = (int64_t)blockIdx.x * kSlice; at < (int64_t)c.bytes; at += (int64_t)gridDim.x * kSlice) {
      u32x4 v[4];
      const unsigned char* src = static_cast<const unsigned char*>(c.src) + at;
      unsigned char* dst = static_cast<unsigned char*>(c.dst) + at;
      const int left = (int)((int64_t)c.bytes - at < kSlice ? (int64_t)c.bytes - at : kSlice);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int off = (k * kThreads + (int)threadIdx.x) * 16;
        if (off < left) v[k] = *reinterpret_cast<const u32x4*>(src + off);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int off = (k * kThreads + (int)threadIdx.x) * 16;
        if (off < left) *reinterpret_cast<u32x4*>(dst + off) = v[k];
      }
    }
    return;
  }
  // scales of a range that starts at any token (one fp16 per token), or odd bytes
  const int64_t first = (int64_t)blockIdx.x * kThreads + threadIdx.x, step = (int64_t)gridDim.x * kThreads;
  if ((low & 3) == 0) copy_units<uint32_t>(c, first, step);
  else if ((low & 1) == 0) copy_units<uint16_t>(c, first, step);
  else copy_units<uint8_t>(c, first, step);
}

}  // namespace

hipError_t launch_copy_ranges(const CopyRange* ranges, int n, hipStream_t stream) {
  for (int at = 0; at < n; at += kCopyRangesPerLaunch) {
    const int m = n - at < kCopyRangesPerLaunch ? n - at : kCopyRangesPerLaunch;
    Ranges list;
    size_t longest = 0;
    for (int i = 0; i < m; ++i) {
      list.r[i] = ranges[at + i];
      longest = longest > list.r[i].bytes ? longest : list.r[i].bytes;
    }
    for (int i = m; i < kCopyRangesPerLaunch; ++i) list.r[i] = CopyRange{nullptr, nullptr, 0};
    if (longest == 0) continue;
    const size_t slices = (longest + kSlice - 1) / kSlice;
    const unsigned cap = 2048u / (unsigned)m + 1;         // a few workgroups per CU over all ranges
    copy_ranges_kernel<<<dim3(slices < cap ? (unsigned)slices : cap, (unsigned)m), kThreads, 0, stream>>>(list);
  }
  return hipGetLastError();
}

}  // namespace aquakv
