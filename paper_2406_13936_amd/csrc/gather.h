// The batch gather, as a launch of its own (elementwise.hip) or behind the tiles of a contraction (gemm_small.hip,
// gemm_f32.hip); the first layer then reads its rows from the dataset.
#pragma once
#include "device_utils.h"

namespace absk {
namespace {

template <class T> struct Vec;                      // 16-byte vector of T
template <> struct Vec<float> {
  enum { N = 4 };
  static __device__ __forceinline__ void load(const float *p, float (&o)[4]) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
};
template <> struct Vec<bf16_t> {
  enum { N = 8 };
  static __device__ __forceinline__ void unpack(uint4 v, float (&o)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void load(const bf16_t *p, float (&o)[8]) {
    unpack(*reinterpret_cast<const uint4 *>(p), o);
  }
};

// One wavefront per gathered row, four to a block of 256 threads.  Source rows have d elements (row stride d); the
// destination row stride is ldo >= d (multiple of 8), pad columns are written as zeros.
// Indices outside [0, N) are clamped into the range (the kernels never read out of bounds).
// (Source and destination never overlap: the dataset and the workspace.)
template <class T>
__device__ __forceinline__ float gather_row(const T *__restrict__ src, T *__restrict__ dst, int d, int ldo, int lane) {
  float s = 0.0f;
  constexpr int V = Vec<T>::N;
  if ((d % V) == 0) {
    for (int c = lane * V; c < d; c += 64 * V) {
      const uint4 raw = *reinterpret_cast<const uint4 *>(src + c);
      float f[V];
      Vec<T>::load(src + c, f);
#pragma unroll
      for (int k = 0; k < V; ++k) s = fmaf(f[k], f[k], s);
      *reinterpret_cast<uint4 *>(dst + c) = raw;
    }
  } else {
    for (int c = lane; c < d; c += 64) {
      const T raw = src[c];
      const float f = Elem<T>::ld(&raw);
      s = fmaf(f, f, s);
      dst[c] = raw;
    }
  }
  for (int c = d + lane; c < ldo; c += 64) Elem<T>::st(dst + c, 0.0f);
  return wave_sum(s);
}
template <class T>
__device__ __forceinline__ void gather_rows_block(const GatherP &p, int g, int block) {
  const int i = block * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= (p.rows ? p.rows[g] : p.b)) return;
  const int id = min(max(p.idx[(long long)g * p.ldi + i], 0), p.N - 1);
  const float s = gather_row(static_cast<const T *>(p.X) + (long long)id * p.d,
                             static_cast<T *>(p.A0) + (long long)g * p.sA0g + (long long)i * p.ldo, p.d, p.ldo, lane);
  if (lane == 0) p.an0[(long long)g * p.sNg + i] = s;
}
// block of gather_blocks(p), group by group
template <class T>
__device__ __forceinline__ void gather_riding_block(const GatherP &p, int block) {
  const int nb = (p.b + 3) / 4, g = block / nb;
  if (g < p.groups) gather_rows_block<T>(p, g, block - g * nb);
}
// row i of operand A of group g (GemmP::aidx)
__device__ __forceinline__ int dataset_row(const GemmP &p, int g, int i) {
  return min(max(p.aidx[(long long)g * p.aldi + i], 0), p.aN - 1);
}

}  // namespace
}  // namespace absk
