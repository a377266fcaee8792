// Diagnostics, outside the per-token path:
//  - read-back of what the last MLP call left in a workspace: the per-row h3
//    values of Eq. (1) step 3 (h3 = ReLU(W_gate,i . x) * (W_up,i . x), or
//    ReLU(W_fc1,i . x) without W_up), so that tests can compare every kept
//    row with an independent implementation, not only y;
//  - a plain streaming read of a buffer, the reference against which the
//    benchmark puts the path's bandwidth beside the HBM peak.
#include "si_device.h"
#include "si_launch.h"

namespace si {

// Kept rows get the value the call published for them in this call, or NaN
// when there is none; other rows get 0.
__global__ __launch_bounds__(1024) void k_read_h3(const uint32_t* __restrict__ hdr, const uint64_t* __restrict__ h3e,
                                                  const float* __restrict__ h3p, const uint8_t* __restrict__ mask,
                                                  int k, int b, float* __restrict__ out) {
  const uint32_t form = hdr[H_H3_FORM];
  const uint32_t tag = epoch_tag(hdr[H_EPOCH] - 1u);  // the last call's tag (each call advances the counter once)
  const float nan = __builtin_nanf("");
  for (int i = threadIdx.x; i < k; i += 1024) {
    const bool kept = mask[i] != 0;
    for (int t = 0; t < b; ++t) {
      float v = 0.f;
      if (kept) {
        if (form == kH3ByRow) {
          const uint64_t w = h3e[(size_t)i * b + t];
          v = (uint32_t)(w >> 32) == tag ? __uint_as_float((uint32_t)w) : nan;
        } else if (form == kH3PlainByRow) {
          v = h3p[(size_t)i * b + t];
        } else {
          v = nan;
        }
      }
      out[(size_t)i * b + t] = v;
    }
  }
}

hipError_t launch_read_h3(const void* ws, int k, int b, const uint8_t* mask, float* out, hipStream_t s) {
  const WsLayout L = ws_layout(k, b);
  const char* base = static_cast<const char*>(ws);
  k_read_h3<<<1, 1024, 0, s>>>(reinterpret_cast<const uint32_t*>(base), reinterpret_cast<const uint64_t*>(base + L.h3e),
                               reinterpret_cast<const float*>(base + L.h3), mask, k, b, out);
  return hipGetLastError();
}

// Every 16-byte unit of the buffer read once with non-temporal loads, four
// requests in flight per thread per step; the XOR of the data decides a store
// that never happens for real data, so that the loads stay.
__global__ __launch_bounds__(256) void k_read_probe(const u32x4* __restrict__ p, size_t units, uint32_t* sink) {
  const size_t stride = (size_t)gridDim.x * 256;
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  uint32_t acc = 0;
  for (; i + 3 * stride < units; i += 4 * stride) {
    const u32x4 a = load_nt(p + i), b = load_nt(p + i + stride), c = load_nt(p + i + 2 * stride),
                e = load_nt(p + i + 3 * stride);
    acc ^= (a.x ^ a.w) ^ (b.y ^ b.z) ^ (c.x ^ c.z) ^ (e.y ^ e.w);
  }
  for (; i < units; i += stride) {
    const u32x4 a = load_nt(p + i);
    acc ^= a.x ^ a.y ^ a.z ^ a.w;
  }
  if (acc == 0x9e3779b9u) sink[0] = acc;
}

hipError_t launch_read_probe(const void* buf, size_t bytes, uint32_t* sink, hipStream_t s) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const size_t units = bytes / 16;
  const size_t want = (units + 4 * 256 - 1) / (4 * 256);
  const int blocks = (int)(want < (size_t)cus * 8 ? (want > 0 ? want : 1) : (size_t)cus * 8);
  k_read_probe<<<blocks, 256, 0, s>>>(static_cast<const u32x4*>(buf), units, sink);
  return hipGetLastError();
}

}  // namespace si
