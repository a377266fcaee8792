// Load-time preprocessing: sign packing of W_gate (Section IV-B 1), the
// transpose of W_down (Section IV-B 4), and for INT8 weights their symmetric
// per-row quantization and the packing of their MSBs (Section IV-A).
//
// Packed-sign layout (private to the library).  A unit is 4 consecutive
// 32-bit words (128 elements) of one row; units are stored unit-major over
// the rows, which are padded to a multiple of 64 (kpad):
//     word (row i, w) -> [unit w/4][row i][w%4]
// so that unit q of any run of consecutive rows is one contiguous piece of
// memory, read with one 16-byte load per lane (lane = row): 1 KB for a
// 64-row group, R * 16 bytes for a block's R rows.  Bit j of word w is the
// sign of element 32*w + j.  Padding rows are all zero.
#include <type_traits>

#include "si_device.h"
#include "si_launch.h"

namespace si {

__device__ inline size_t packed_index(int i, int w, int kpad) {
  return ((size_t)(w >> 2) * kpad + i) * 4 + (w & 3);
}

// One thread per (row, word): reads 32 consecutive fp16 (64 bytes; adjacent
// threads read adjacent words of a row).
__global__ __launch_bounds__(256) void k_pack_signs(const uint16_t* __restrict__ w, int k, int d,
                                                    uint32_t* __restrict__ signs) {
  const int W = d >> 5;
  const int kpad = (k + kRowGroup - 1) / kRowGroup * kRowGroup;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (size_t)kpad * W) return;
  const int i = (int)(t / W), wd = (int)(t % W);
  uint32_t word = 0;
  if (i < k) word = sign_word(reinterpret_cast<const u32x4*>(w + (size_t)i * d + 32 * wd));
  signs[packed_index(i, wd, kpad)] = word;
}

// Sign word of 32 consecutive INT8 values (bit j = MSB of byte j).
__device__ inline uint32_t sign_word_i8(const u32x4* p) {
  uint32_t word = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const u32x4 v = p[h];
    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) word |= ((w4[i] >> (8 * j + 7)) & 1u) << (16 * h + 4 * i + j);
  }
  return word;
}

// The INT8 form of k_pack_signs: one thread per (row, word), 32 bytes each.
__global__ __launch_bounds__(256) void k_pack_signs_i8(const int8_t* __restrict__ w, int k, int d,
                                                       uint32_t* __restrict__ signs) {
  const int W = d >> 5;
  const int kpad = (k + kRowGroup - 1) / kRowGroup * kRowGroup;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (size_t)kpad * W) return;
  const int i = (int)(t / W), wd = (int)(t % W);
  uint32_t word = 0;
  if (i < k) word = sign_word_i8(reinterpret_cast<const u32x4*>(w + (size_t)i * d + 32 * wd));
  signs[packed_index(i, wd, kpad)] = word;
}

// 16 bytes at any element boundary (rows of an odd length start anywhere)
typedef u32x4 u32x4_u __attribute__((aligned(2)));
typedef u32x4 u32x4_b __attribute__((aligned(1)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_u __attribute__((aligned(1)));

__device__ inline float fp16_of(u32x4 v, int i) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(v[i >> 1] >> (16 * (i & 1))));
}

// q = rint(w / s) (ties to even, clamped to +-127) for the correctly rounded
// float quotient; inv = 1 / s.  |w / s| is at most about 127, so w * inv is
// within 3e-5 of both the quotient and its rounding and rounds to the same
// integer unless it is that close to a half: only then (about one value in
// 5000 at the 1e-4 tested here, and NaN) is the division made, which costs
// more than everything else here.
__device__ inline int quantize_one(float w, float s, float inv) {
  const float r = w * inv;
  float t = rintf(r);
  if (!(fabsf(fabsf(r - t) - 0.5f) > 1e-4f)) t = rintf(w / s);
  return (int)fminf(fmaxf(t, -127.f), 127.f);
}

// Symmetric per-row INT8 quantization, one block per row of n fp16 values:
// scale = max |w| / 127 and q = rint(w / scale) (ties to even, clamped to
// +-127), in float32 with correctly rounded division; a row of zeros gets
// scale 0 and q = 0.  Memory bound (3 bytes a value): a row of up to 8 NT NV
// values is read once, 16 bytes a lane, all of it requested together, and kept
// in registers between the maximum and the rounding (NV = 0: rows longer
// than that, read twice).  (One value a lane, two reads of the row and a division each:
// 11008 x 4096 in 92.7 us = 1.46 TB/s; now 26.5-29.8 us = 4.5-5.1 TB/s.)
template <int NT, int NV>
__global__ __launch_bounds__(NT) void k_quantize_rows(const uint16_t* __restrict__ w, int n,
                                                       int8_t* __restrict__ q, float* __restrict__ scale) {
  __shared__ float wmax[NT / kWave];
  const size_t base = (size_t)blockIdx.x * n;
  const uint16_t* row = w + base;
  int8_t* out = q + base;
  const int tid = threadIdx.x;
  const int nv = n >> 3;  // whole vectors of 8 values; the rest go one by one
  float m = 0.f;
  u32x4 v[NV > 0 ? NV : 1];
  auto top = [&](u32x4 x) {
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(fp16_of(x, i)));
  };
  auto load = [&](int j) -> u32x4 { return __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(row) + j); };
  if constexpr (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i] = u32x4{0, 0, 0, 0};
      if (tid + NT * i < nv) v[i] = load(tid + NT * i);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) top(v[i]);
  } else {
    for (int j = tid; j < nv; j += NT) top(load(j));
  }
  const bool tail = tid < n - 8 * nv;
  const float wt = tail ? (float)__builtin_bit_cast(_Float16, row[8 * nv + tid]) : 0.f;
  m = fmaxf(m, fabsf(wt));
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
  if ((tid & 63) == 0) wmax[tid >> 6] = m;
  __syncthreads();
  float amax = wmax[0];
#pragma unroll
  for (int i = 1; i < NT / kWave; ++i) amax = fmaxf(amax, wmax[i]);
  const float s = amax / 127.0f;
  const float inv = 1.0f / s;
  auto store = [&](int j, u32x4 x) {
    u32x2 r = {0, 0};
    if (s > 0.f) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        r[i >> 2] |= ((uint32_t)quantize_one(fp16_of(x, i), s, inv) & 0xffu) << (8 * (i & 3));
    }
    reinterpret_cast<u32x2_u*>(out)[j] = r;
  };
  if constexpr (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (tid + NT * i < nv) store(tid + NT * i, v[i]);
  } else {
    for (int j = tid; j < nv; j += NT) store(j, load(j));
  }
  if (tail) out[8 * nv + tid] = s > 0.f ? (int8_t)quantize_one(wt, s, inv) : (int8_t)0;
  if (tid == 0) scale[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void k_signs_to_canonical(const uint32_t* __restrict__ signs, int k,
                                                            int d, uint32_t* __restrict__ out) {
  const int W = d >> 5;
  const int kpad = (k + kRowGroup - 1) / kRowGroup * kRowGroup;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (size_t)k * W) return;
  const int i = (int)(t / W), wd = (int)(t % W);
  out[t] = signs[packed_index(i, wd, kpad)];
}

// out[c][r] = in[r][c] for a rows x cols matrix (fp16 or INT8 elements), rows a
// multiple of 128.  Memory bound (each byte once in, once out): a lane takes a
// square of E x E elements (E = 16 bytes of them), one 16-byte piece of each of E
// rows, turns it around in registers with byte permutes and writes 16 bytes of
// each of E columns; the 64 lanes lie 8 x 8, so that every request reads and
// writes whole 128-byte lines (8 of them).  (Single elements through an LDS
// tile of 64 x 64: 4096 x 11008 in 72.2 us = 2.5 TB/s, INT8 47.0 us = 1.9 TB/s;
// now 34.7 us = 5.2 TB/s and 16.9 us = 5.3 TB/s.)
// Columns at the right edge go element by element.
template <typename T>
__global__ __launch_bounds__(256) void k_transpose(const T* __restrict__ in, int rows, int cols,
                                                   T* __restrict__ out) {
  constexpr int E = 16 / sizeof(T);
  typedef std::conditional_t<sizeof(T) == 2, u32x4_u, u32x4_b> vec_u;  // rows of any length
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c0 = ((blockIdx.x * 4 + wv) * 8 + (lane & 7)) * E;
  const int r0 = (blockIdx.y * 8 + (lane >> 3)) * E;
  if (c0 >= cols) return;
  const T* src = in + (size_t)r0 * cols + c0;
  u32x4 v[E];
  if (c0 + E <= cols) {
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = __builtin_nontemporal_load(reinterpret_cast<const vec_u*>(src + (size_t)i * cols));
  } else {
#pragma unroll
    for (int i = 0; i < E; ++i) {
      v[i] = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (c0 + e < cols) v[i][e / (4 / sizeof(T))] |= (uint32_t)src[(size_t)i * cols + e] << (8 * sizeof(T) * (e % (4 / sizeof(T))));
    }
  }
  T* dst = out + (size_t)c0 * rows + r0;
  auto put = [&](int e, u32x4 o) {
    if (c0 + e < cols) *reinterpret_cast<u32x4*>(dst + (size_t)e * rows) = o;
  };
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint32_t sel = e & 1 ? 0x07060302u : 0x05040100u;  // the high or low halves of two rows
      u32x4 o;
#pragma unroll
      for (int p = 0; p < 4; ++p) o[p] = __builtin_amdgcn_perm(v[2 * p + 1][e >> 1], v[2 * p][e >> 1], sel);
      put(e, o);
    }
  } else {
    // 4 x 4 bytes at a time: two rows' low (high) byte pairs, then two of those
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      u32x4 o[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const uint32_t a = v[4 * p][w], b = v[4 * p + 1][w], c = v[4 * p + 2][w], d = v[4 * p + 3][w];
        const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
        const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
        o[0][p] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
        o[1][p] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
        o[2][p] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
        o[3][p] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) put(4 * w + e, o[e]);
    }
  }
}

hipError_t launch_pack_signs(const uint16_t* w_gate, int k, int d, uint32_t* signs, hipStream_t s) {
  const int kpad = (k + kRowGroup - 1) / kRowGroup * kRowGroup;
  const size_t threads = (size_t)kpad * (d >> 5);
  const unsigned grid = (unsigned)((threads + 255) / 256);
  k_pack_signs<<<grid, 256, 0, s>>>(w_gate, k, d, signs);
  return hipGetLastError();
}

hipError_t launch_signs_to_canonical(const uint32_t* signs, int k, int d, uint32_t* out, hipStream_t s) {
  const size_t threads = (size_t)k * (d >> 5);
  const unsigned grid = (unsigned)((threads + 255) / 256);
  k_signs_to_canonical<<<grid, 256, 0, s>>>(signs, k, d, out);
  return hipGetLastError();
}

// rows (= d) is a multiple of 128, cols (= k) anything
template <typename T>
static hipError_t transpose(const T* in, int rows, int cols, T* out, hipStream_t s) {
  constexpr int E = 16 / sizeof(T);
  dim3 grid((cols + 32 * E - 1) / (32 * E), rows / (8 * E));
  k_transpose<T><<<grid, 256, 0, s>>>(in, rows, cols, out);
  return hipGetLastError();
}

hipError_t launch_transpose(const uint16_t* in, int rows, int cols, uint16_t* out, hipStream_t s) {
  return transpose<uint16_t>(in, rows, cols, out, s);
}

hipError_t launch_transpose_i8(const int8_t* in, int rows, int cols, int8_t* out, hipStream_t s) {
  return transpose<uint8_t>(reinterpret_cast<const uint8_t*>(in), rows, cols, reinterpret_cast<uint8_t*>(out), s);
}

hipError_t launch_pack_signs_i8(const int8_t* w_gate, int k, int d, uint32_t* signs, hipStream_t s) {
  const int kpad = (k + kRowGroup - 1) / kRowGroup * kRowGroup;
  const size_t threads = (size_t)kpad * (d >> 5);
  const unsigned grid = (unsigned)((threads + 255) / 256);
  k_pack_signs_i8<<<grid, 256, 0, s>>>(w_gate, k, d, signs);
  return hipGetLastError();
}

hipError_t launch_quantize_rows(const uint16_t* w, int rows, int n, int8_t* q, float* scale, hipStream_t s) {
  // rows of up to 4096 values: 256 threads with 2 vectors of 8 each; longer
  // ones 512 threads with 3 (12288 values) or 4 (with 256 threads and 6 vectors,
  // 4096 x 11008 took 41.9 us, so 31.0-33.2: too few waves to cover the reads)
  const int nv = n >> 3;
  if (nv <= 512)
    k_quantize_rows<256, 2><<<rows, 256, 0, s>>>(w, n, q, scale);
  else if (nv <= 3 * 512)
    k_quantize_rows<512, 3><<<rows, 512, 0, s>>>(w, n, q, scale);
  else if (nv <= 4 * 512)
    k_quantize_rows<512, 4><<<rows, 512, 0, s>>>(w, n, q, scale);
  else
    k_quantize_rows<512, 0><<<rows, 512, 0, s>>>(w, n, q, scale);
  return hipGetLastError();
}

}  // namespace si
