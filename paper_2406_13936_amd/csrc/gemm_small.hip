// bf16 contractions of launches too small to fill the chip with the tiles of gemm_bf16.hip:
//
//   C[g][m][n] = sum_k A[g][m][k] * B[g][n][k]      (forward, logits: B stored [n][k]; backward-data: B stored [k][n])
//
// What bounds them is a chain of latencies, not traffic or arithmetic: a 64 x 128 tile leaves 32 work-groups for a
// 512-wide layer of 8 replicas at b = 32 and walks its k-tiles one barrier after the other.  Here a work-group owns 32 x 32
// (or 32 x 64) outputs, its four wavefronts take chunks of the reduction in turn, and every fragment goes straight from
// memory to registers, all loads of up to four chunks per wave in flight before the first MFMA; the four partial
// tiles meet in LDS once.
//   * [row][k] operands: a lane's MFMA fragment is 8 consecutive k of one row, a 16-byte load.
//   * [k][row] operands (backward-data): a lane loads the column pair (2 c, 2 c + 1), c = lane % 32, of 8 consecutive k as
//     eight 4-byte words (128 consecutive bytes per k and half wave) and splits the pair with v_perm: accumulator 0
//     holds the even columns of the 64, accumulator 1 the odd ones.
// Logits of at most 32 classes carry the softmax cross-entropy head: a row is held by eight threads at the end.
// Measured (8 replicas, b = 32): forward 784 -> 512 and 512 -> 512 10.2 -> 7.7 us, backward-data 8.5 -> 6.3, logits
// 512 -> 10 9.8 -> 5.0.
// Out-of-range rows and k come back as zeros from the buffer descriptor's range check.
#include "abs_internal.h"
#include "device_utils.h"
#include "gather.h"

namespace absk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr uint32_t OOB = 0x80000000u;   // byte offset beyond any operand (operands are < 2 GiB)

// GA: 1: the batch gather rides behind the tiles; 2: and they read their rows of A from the dataset.
template <bool BT, int EPI, int ACT, int GA>
__global__ void __launch_bounds__(256) gemm_small_kernel(const GemmP p, const int tilesM, const int tilesN, const GatherP ga) {
  constexpr int NJ = BT ? 2 : 1;                          // accumulator tiles of 32 x 32 per wave
  constexpr int BN = 32 * NJ, CPT = 4 * NJ;               // columns per work-group, columns per thread at the end
  constexpr int KC = BT ? 32 : 64, KS = KC / 16;          // k per chunk, MFMA steps per chunk
  constexpr int D = 4;                                    // chunks in flight per wave
  constexpr int RLD = BN + 4;                             // row stride of the reduction buffer (floats)
  __shared__ __attribute__((aligned(16))) float red[4 * 32 * RLD];

  int id = blockIdx.x;
  if (GA != 0) {
    const int tiles = tilesM * tilesN * p.groups;
    if (id >= tiles) { gather_riding_block<bf16_t>(ga, id - tiles); return; }
  }
  const int tn = id % tilesN; id /= tilesN;
  const int tm = id % tilesM, g = id / tilesM;
  const int m0 = tm * 32, n0 = tn * BN;
  const int Md = p.rows ? p.rows[g] : p.Md;               // ragged groups: this group's own extent
  if (m0 >= Md) return;                                   // uniform over the block, before any barrier

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const bf16_t *A = static_cast<const bf16_t *>(p.A) + (long long)g * p.sAg;
  const bf16_t *B = static_cast<const bf16_t *>(p.B) + (long long)g * p.sBg;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(A), 0, (int)((long long)(GA == 2 ? p.aN : Md) * p.lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(B), 0, (int)((long long)(BT ? p.Kd : p.Nd) * p.ldb * 2), 0x00020000);

  // outputs of this thread once the waves' partial tiles are added: row mr, columns nc .. nc + CPT - 1
  const int row = tid >> 3, c8 = tid & 7, mr = m0 + row, nc = n0 + c8 * CPT;
  const bool live = mr < Md && nc < p.Nd;
  // epilogue operands, in flight from the start
  float bv[CPT];
  bf16_t ev[CPT];
#pragma unroll
  for (int e = 0; e < CPT; ++e) { bv[e] = 0.0f; ev[e] = 0; }
  if (EPI != EPI_BWD && p.bias) {
#pragma unroll
    for (int e = 0; e < CPT; ++e) if (nc + e < p.Nd) bv[e] = p.bias[(long long)g * p.sBiasg + nc + e];
  }
  if (EPI == EPI_BWD && ACT != ACT_NONE && live) {        // (Nd is a multiple of 8: a thread's columns are all inside)
    const uint4 w = *reinterpret_cast<const uint4 *>(static_cast<const bf16_t *>(p.E) + (long long)g * p.sEg + (long long)mr * p.lde + nc);
    const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < CPT; ++e) ev[e] = (bf16_t)(w4[(e >> 1) & 3] >> (16 * (e & 1)));
  }

  int label = 0;
  if (EPI == EPI_LOGITS && p.head.y) {
    const int id = p.head.idx[(long long)g * p.head.ldi + min(mr, Md - 1)];
    label = min(max(p.head.y[min(max(id, 0), p.head.N - 1)], 0), p.Nd - 1);
  }

  f32x16 acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

  uint32_t arow = OOB;
  if (m0 + l32 < Md) {
    const int r = GA == 2 ? dataset_row(p, g, m0 + l32) : m0 + l32;
    arow = ((uint32_t)r * (uint32_t)p.lda + (uint32_t)half * 8) * 2u;
  }
  const uint32_t brow = BT ? (n0 + 2 * l32 < p.Nd ? (uint32_t)(half * 8 * p.ldb + n0 + 2 * l32) * 2u : OOB)
                           : (n0 + l32 < p.Nd ? (uint32_t)((n0 + l32) * p.ldb + half * 8) * 2u : OOB);
  for (int kb = wave * KC; kb < p.Kd; kb += D * 4 * KC) {
    u32x4_t fa[D][KS];
    u32x4_t fb[BT ? 1 : D][BT ? 1 : KS];
    uint32_t fw[BT ? D : 1][BT ? KS : 1][8];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const int k = kb + d * 4 * KC + kk * 16;          // this lane: k + 8 half .. + 7
        const bool in = k + half * 8 < p.Kd;              // (A: whole 16-byte chunks, pad columns of a row hold zeros)
        fa[d][kk] = __builtin_amdgcn_raw_buffer_load_b128(ra, in ? arow + (uint32_t)k * 2u : OOB, 0, 0);
        if constexpr (BT) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            fw[d][kk][e] = __builtin_amdgcn_raw_buffer_load_b32(
                rb, k + half * 8 + e < p.Kd ? brow + (uint32_t)(k + e) * (uint32_t)p.ldb * 2u : OOB, 0, 0);
        } else {
          fb[d][kk] = __builtin_amdgcn_raw_buffer_load_b128(rb, in ? brow + (uint32_t)k * 2u : OOB, 0, 0);
        }
      }
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, fa[d][kk]);
        // operands swapped, as in gemm_bf16.hip: a lane owns one row of C and groups of four consecutive column slots
        if constexpr (BT) {
          u32x4_t ce, co;                                 // even and odd columns, 8 consecutive k each
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ce[e] = __builtin_amdgcn_perm(fw[d][kk][2 * e + 1], fw[d][kk][2 * e], 0x05040100u);
            co[e] = __builtin_amdgcn_perm(fw[d][kk][2 * e + 1], fw[d][kk][2 * e], 0x07060302u);
          }
          acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ce), a, acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, co), a, acc[1], 0, 0, 0);
        } else {
          acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[d][kk]), a, acc[0], 0, 0, 0);
        }
      }
  }

  // partial tiles to LDS: red[wave][row][32 j + slot]
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4 *>(red + (wave * 32 + l32) * RLD + j * 32 + q * 8 + half * 4) =
          make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
  __syncthreads();
  float v[CPT];                                           // the four waves' sums, in wave order
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    float4 s = *reinterpret_cast<const float4 *>(red + row * RLD + j * 32 + c8 * 4);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 t = *reinterpret_cast<const float4 *>(red + (w * 32 + row) * RLD + j * 32 + c8 * 4);
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    const float s4[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) v[BT ? 2 * e + j : e] = s4[e];   // (slot s of accumulator j is column 2 s + j)
  }

  if constexpr (EPI == EPI_LOGITS) {
    if (p.head.y) {                                       // uniform: softmax cross-entropy over the row's eight threads
      float z[CPT], mx = -INFINITY, se = 0.0f, sq = 0.0f, ex[CPT], dl[CPT];
#pragma unroll
      for (int e = 0; e < CPT; ++e) { z[e] = nc + e < p.Nd ? v[e] + bv[e] : -INFINITY; mx = fmaxf(mx, z[e]); }
#pragma unroll
      for (int x = 1; x < 8; x <<= 1) mx = fmaxf(mx, __shfl_xor(mx, x, 64));
#pragma unroll
      for (int e = 0; e < CPT; ++e) { ex[e] = nc + e < p.Nd ? expf(z[e] - mx) : 0.0f; se += ex[e]; }
#pragma unroll
      for (int x = 1; x < 8; x <<= 1) se += __shfl_xor(se, x, 64);
      const float inv = 1.0f / se;
#pragma unroll
      for (int e = 0; e < CPT; ++e) {
        dl[e] = nc + e < p.Nd ? ex[e] * inv - (nc + e == label ? 1.0f : 0.0f) : 0.0f;
        const float st = bf2f(f2bf(dl[e]));
        sq = fmaf(st, st, sq);
      }
#pragma unroll
      for (int x = 1; x < 8; x <<= 1) sq += __shfl_xor(sq, x, 64);
      if (mr < Md) {
        if (nc < p.head.ldd)                              // ldd is a multiple of 8
          *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(p.head.D) + (long long)g * p.head.sDg + (long long)mr * p.head.ldd + nc) =
              make_uint2(pack2bf(dl[0], dl[1]), pack2bf(dl[2], dl[3]));
        const long long at = (long long)g * p.head.sNg + mr;
        if (c8 == 0) p.head.dn[at] = sq;
#pragma unroll
        for (int e = 0; e < CPT; ++e) if (nc + e == label) p.head.loss[at] = -(z[e] - mx - logf(se));
      }
      return;
    }
    if (mr < Md) {
      float *C = static_cast<float *>(p.C) + (long long)g * p.sCg + (long long)mr * p.ldc;
#pragma unroll
      for (int e = 0; e < CPT; ++e) if (nc + e < p.Nd) C[nc + e] = v[e] + bv[e];
    }
    return;
  }
  float sq = 0.0f;                                        // this row's squared stored outputs
  uint32_t o[CPT / 2], o2[CPT / 2];
#pragma unroll
  for (int e = 0; e < CPT; e += 2) {
    float a[2], d[2] = {0.0f, 0.0f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (EPI == EPI_FWD_ACT) act_fwd<ACT>(v[e + h] + bv[e + h], a[h], d[h]);
      else {
        const float f = bf2f(ev[e + h]);
        a[h] = ACT == ACT_RELU ? (f > 0.0f ? v[e + h] : 0.0f) : (ACT == ACT_GELU ? v[e + h] * f : v[e + h]);
        if (!live) a[h] = 0.0f;
      }
    }
    o[e / 2] = pack2bf(a[0], a[1]);
    o2[e / 2] = pack2bf(d[0], d[1]);
    const float lo = __uint_as_float(o[e / 2] << 16), hi = __uint_as_float(o[e / 2] & 0xffff0000u);
    sq = fmaf(lo, lo, fmaf(hi, hi, sq));
  }
  auto store = [&](bf16_t *dst, const uint32_t *w) {      // rows and columns are multiples of 8 elements
    if constexpr (CPT == 8) *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    else *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
  };
  if (live) {
    store(static_cast<bf16_t *>(p.C) + (long long)g * p.sCg + (long long)mr * p.ldc + nc, o);
    if (EPI == EPI_FWD_ACT && ACT == ACT_GELU && p.C2)
      store(static_cast<bf16_t *>(p.C2) + (long long)g * p.sC2g + (long long)mr * p.ldc2 + nc, o2);
  }
  if (p.part) {                                           // uniform: the eight threads of a row, fixed order
    if (nc >= p.Nd) sq = 0.0f;
#pragma unroll
    for (int x = 1; x < 8; x <<= 1) sq += __shfl_xor(sq, x, 64);
    if (c8 == 0 && mr < Md) p.part[(long long)g * p.sPartg + (long long)tn * p.sPartTile + mr] = sq;
  }
  if (EPI == EPI_BWD && p.cpart) {                        // column sums of the tile: 8 rows per wave, then the four waves
    float cs[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) {
      cs[e] = __uint_as_float((e & 1) ? (o[e / 2] & 0xffff0000u) : (o[e / 2] << 16));
#pragma unroll
      for (int x = 8; x < 64; x <<= 1) cs[e] += __shfl_xor(cs[e], x, 64);
    }
    __syncthreads();                                      // the partial tiles have been read
    if (lane < 8) {
#pragma unroll
      for (int e = 0; e < CPT; ++e) red[wave * BN + lane * CPT + e] = cs[e];
    }
    __syncthreads();
    if (tid < BN && n0 + tid < p.Nd)
      p.cpart[(long long)g * p.sCpartg + (long long)tm * p.Nd + n0 + tid] =
          ((red[tid] + red[BN + tid]) + red[2 * BN + tid]) + red[3 * BN + tid];
  }
}

template <bool BT, int EPI, int ACT>
hipError_t launch1(const GemmP &p, hipStream_t s) {
  const int tilesM = (p.Md + 31) / 32, tilesN = (p.Nd + (BT ? 63 : 31)) / (BT ? 64 : 32);
  long long nblk = (long long)tilesM * tilesN * p.groups;
  if (nblk <= 0) return hipSuccess;
  if (nblk > 0x3fffffff) return hipErrorInvalidValue;
  if constexpr (EPI != EPI_BWD) {
    if (p.gather) {
      const GatherP &ga = *p.gather;
      nblk += gather_blocks(ga);
      if (p.aidx) hipLaunchKernelGGL((gemm_small_kernel<BT, EPI, ACT, 2>), dim3((unsigned)nblk), dim3(256), 0, s, p, tilesM, tilesN, ga);
      else if constexpr (EPI == EPI_LOGITS)
        hipLaunchKernelGGL((gemm_small_kernel<BT, EPI, ACT, 1>), dim3((unsigned)nblk), dim3(256), 0, s, p, tilesM, tilesN, ga);
      else return hipErrorInvalidValue;
      return hipGetLastError();
    }
  }
  if (p.aidx) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_small_kernel<BT, EPI, ACT, 0>), dim3((unsigned)nblk), dim3(256), 0, s, p, tilesM, tilesN, GatherP{});
  return hipGetLastError();
}
template <bool BT, int EPI>
hipError_t launch_act(const GemmP &p, hipStream_t s) {
  if constexpr (EPI != EPI_LOGITS) {
    if (p.act == ACT_RELU) return launch1<BT, EPI, ACT_RELU>(p, s);
    if (p.act == ACT_GELU) return launch1<BT, EPI, ACT_GELU>(p, s);
  }
  return launch1<BT, EPI, ACT_NONE>(p, s);
}

}  // namespace

// (operand checks shared with the tiled family: launch_gemm_bf16)
hipError_t launch_gemm_small(const GemmP &p, int epi, hipStream_t s) {
  // 16-byte chunks of A (and of [n][k] operands) never cross the end of a row's storage; outputs, E and [k][n] operands are
  // touched in groups of 4 or 8 consecutive columns
  if (epi != EPI_LOGITS && ((p.Nd & 7) || (p.ldc & 7) || (p.sCg & 7) || (reinterpret_cast<uintptr_t>(p.C) & 15)))
    return hipErrorInvalidValue;
  if (p.head.y && (epi != EPI_LOGITS || !gemm_head_fits(1, p.Md, p.Nd, p.groups) || !p.head.idx || p.head.N < 1 || !p.head.D ||
                   !p.head.dn || !p.head.loss || p.head.ldd < p.Nd || p.head.ldd > 32 || (p.head.ldd & 7) || (p.head.sDg & 7) ||
                   (reinterpret_cast<uintptr_t>(p.head.D) & 15)))
    return hipErrorInvalidValue;
  if (p.gather && (epi == EPI_BWD || !gather_ok(*p.gather))) return hipErrorInvalidValue;
  if (epi == EPI_FWD_ACT && p.C2 && ((p.ldc2 & 7) || (p.sC2g & 7) || (reinterpret_cast<uintptr_t>(p.C2) & 15)))
    return hipErrorInvalidValue;
  if (epi == EPI_BWD && p.act != ACT_NONE && (!p.E || (p.lde & 7) || (p.sEg & 7) || (reinterpret_cast<uintptr_t>(p.E) & 15)))
    return hipErrorInvalidValue;
  if (epi == EPI_FWD_ACT && !p.a_trans && !p.b_trans && !(p.Kd & 7)) return launch_act<false, EPI_FWD_ACT>(p, s);
  if (epi == EPI_LOGITS && !p.a_trans && !p.b_trans && !(p.Kd & 7)) return launch_act<false, EPI_LOGITS>(p, s);
  if (epi == EPI_BWD && !p.a_trans && p.b_trans) return launch_act<true, EPI_BWD>(p, s);
  return hipErrorInvalidValue;
}

}  // namespace absk
