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

// memory that work-groups on other XCDs write or read in the same launch
__device__ __forceinline__ void st_agent(bf16_t *p, uint2 v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v.y << 32 | v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint4 ld_agent(const bf16_t *p) {
  const unsigned long long *q = reinterpret_cast<const unsigned long long *>(p);
  const unsigned long long a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
}

// A tile of a chain (small_chain_kernel) waits until the `want` words at wait are set before it reads what other tiles of the same
// launch wrote, and sets *done behind its own outputs.  Both sides go past the XCDs' L2 (agent scope).  After `polls` of them it gives up,
// says so in *failed (host memory, which every read-back looks at) and goes on, so that the launch ends whatever happens.
struct ChainLink { int *wait, want, *done, polls, *failed; };

template <bool BT, int EPI> struct SmallTile {
  static constexpr int NJ = BT ? 2 : 1;                   // accumulator tiles of 32 x 32 per wave
  static constexpr int BN = 32 * NJ, CPT = 4 * NJ;        // columns per work-group, columns per thread at the end
  static constexpr int RLD = BN + 4;                      // row stride of the reduction buffer (floats)
  static constexpr int LDS = 4 * 32 * RLD;
};

__device__ __forceinline__ void chain_wait(const ChainLink &link) {
  if (threadIdx.x < 64) {
    // (what it waits for was numbered before this tile and is running or done)
    int n = 0;
    for (; n < link.polls; ++n) {
      int set = 1;
      for (int i = threadIdx.x; i < link.want; i += 64) set &= __hip_atomic_load(link.wait + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__ballot(set == 0) == 0) break;
      __builtin_amdgcn_s_sleep(1);
    }
    if (n == link.polls && threadIdx.x == 0) __hip_atomic_store(link.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();                           // (loads of the weights stay in flight)
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void chain_done(int *at) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wavefront's outputs have arrived
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (threadIdx.x == 0) __hip_atomic_store(at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// over eight neighbouring lanes, in all of them
__device__ __forceinline__ float sum8(float v) { v += dpp<0xB1>(v); v += dpp<0x4E>(v); return v + dpp<0x141>(v); }
__device__ __forceinline__ float max8(float v) { v = fmaxf(v, dpp<0xB1>(v)); v = fmaxf(v, dpp<0x4E>(v)); return fmaxf(v, dpp<0x141>(v)); }
// over the lanes 8 apart
__device__ __forceinline__ float sum_eighths(float v) {
  v += dpp<0x128>(v);
  uint32_t u = __float_as_uint(v);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  u = __float_as_uint(v);
  r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
constexpr int SC1 = 16;                                   // cache policy of a buffer access: agent scope

// Softmax cross-entropy of a row's (at most 32) classes over its eight threads, four each: the stored signals, packed, their squared
// norm and the loss (in the label's thread)
__device__ __forceinline__ uint2 softmax_head(const float (&v)[4], const float (&bv)[4], int nc, int Nd, int label, float &sq, float &loss) {
  float z[4], mx = -INFINITY, se = 0.0f, ex[4], dl[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) { z[e] = nc + e < Nd ? v[e] + bv[e] : -INFINITY; mx = fmaxf(mx, z[e]); }
  mx = max8(mx);
#pragma unroll
  for (int e = 0; e < 4; ++e) { ex[e] = nc + e < Nd ? expf(z[e] - mx) : 0.0f; se += ex[e]; }
  se = sum8(se);
  const float inv = 1.0f / se;
  sq = loss = 0.0f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    dl[e] = nc + e < Nd ? ex[e] * inv - (nc + e == label ? 1.0f : 0.0f) : 0.0f;
    const float st = bf2f(f2bf(dl[e]));
    sq = fmaf(st, st, sq);
    if (nc + e == label) loss = -(z[e] - mx - logf(se));
  }
  sq = sum8(sq);
  return make_uint2(pack2bf(dl[0], dl[1]), pack2bf(dl[2], dl[3]));
}
__device__ __forceinline__ void store_head(const HeadP &h, int g, int mr, int nc, int c8, int label, uint2 w, float sq, float loss) {
  if (nc < h.ldd)                                         // ldd is a multiple of 8
    *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(h.D) + (long long)g * h.sDg + (long long)mr * h.ldd + nc) = w;
  const long long at = (long long)g * h.sNg + mr;
  if (c8 == 0) h.dn[at] = sq;
  if ((unsigned)(label - nc) < 4u) h.loss[at] = loss;
}

// Epilogue of forward and backward-data: v: this thread's CPT sums, bv: bias, ev: elementwise operand (backward-data)
template <bool BT, int EPI, int ACT, bool CHAIN, int CPT>
__device__ __forceinline__ void small_out(const GemmP &p, const int g, const int tm, const int tn, const int Md, const float (&v)[CPT],
                                          const float (&bv)[CPT], const bf16_t (&ev)[CPT], float *red, const ChainLink &link) {
  constexpr int BN = SmallTile<BT, EPI>::BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c8 = tid & 7, mr = tm * 32 + (tid >> 3), n0 = tn * BN, nc = n0 + c8 * CPT;
  const bool live = mr < Md && nc < p.Nd;
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
    if constexpr (CHAIN) {
      st_agent(dst, make_uint2(w[0], w[1]));
      if constexpr (CPT == 8) st_agent(dst + 4, make_uint2(w[2], w[3]));
    } else if constexpr (CPT == 8) *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    else *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
  };
  if (live) {
    store(static_cast<bf16_t *>(p.C) + (long long)g * p.sCg + (long long)mr * p.ldc + nc, o);
    if (EPI == EPI_FWD_ACT && ACT == ACT_GELU && p.C2)
      store(static_cast<bf16_t *>(p.C2) + (long long)g * p.sC2g + (long long)mr * p.ldc2 + nc, o2);
  }
  if constexpr (CHAIN) { if (link.done) chain_done(link.done); }   // (what follows is for later launches)
  if (p.part) {                                           // uniform: the eight threads of a row, fixed order
    if (nc >= p.Nd) sq = 0.0f;
    sq = sum8(sq);
    if (c8 == 0 && mr < Md) p.part[(long long)g * p.sPartg + (long long)tn * p.sPartTile + mr] = sq;
  }
  if (EPI == EPI_BWD && p.cpart) {                        // column sums of the tile: 8 rows per wave, then the four waves
    float cs[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) {
      cs[e] = __uint_as_float((e & 1) ? (o[e / 2] & 0xffff0000u) : (o[e / 2] << 16));
      cs[e] = sum_eighths(cs[e]);
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

// GA: 2: the tiles read their rows of A from the dataset (CHAIN: this lane's is row src).
template <bool BT, int EPI, int ACT, int GA, bool CHAIN>
__device__ __forceinline__ void small_tile(const GemmP &p, const int g, const int tm, const int tn, float *red, const ChainLink &link, const int src = 0) {
  typedef SmallTile<BT, EPI> T;
  constexpr int NJ = T::NJ, BN = T::BN, CPT = T::CPT, RLD = T::RLD;
  constexpr int KC = BT ? 32 : 64, KS = KC / 16;          // k per chunk, MFMA steps per chunk
  constexpr int D = 4;                                    // chunks in flight per wave
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
  auto load_e = [&]() {
    if (EPI == EPI_BWD && ACT != ACT_NONE && live) {      // (Nd is a multiple of 8: a thread's columns are all inside)
      const bf16_t *e8 = static_cast<const bf16_t *>(p.E) + (long long)g * p.sEg + (long long)mr * p.lde + nc;
      uint4 w;
      if constexpr (CHAIN) w = ld_agent(e8);
      else w = *reinterpret_cast<const uint4 *>(e8);
      const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int e = 0; e < CPT; ++e) ev[e] = (bf16_t)(w4[(e >> 1) & 3] >> (16 * (e & 1)));
    }
  };
  if (!CHAIN) load_e();

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
    const int r = GA != 2 ? m0 + l32 : CHAIN ? src : dataset_row(p, g, m0 + l32);
    arow = ((uint32_t)r * (uint32_t)p.lda + (uint32_t)half * 8) * 2u;
  }
  const uint32_t brow = BT ? (n0 + 2 * l32 < p.Nd ? (uint32_t)(half * 8 * p.ldb + n0 + 2 * l32) * 2u : OOB)
                           : (n0 + l32 < p.Nd ? (uint32_t)((n0 + l32) * p.ldb + half * 8) * 2u : OOB);
  // (a chain's first trip is every wavefront's, with loads beyond k where it has none)
  bool first = CHAIN && GA == 0;
  for (int kb = wave * KC; kb < p.Kd || first; kb += D * 4 * KC) {
    u32x4_t fa[D][KS];
    u32x4_t fb[BT ? 1 : D][BT ? 1 : KS];
    uint32_t fw[BT ? D : 1][BT ? KS : 1][8];
    auto at = [&](int d, int kk) -> int { return kb + d * 4 * KC + kk * 16; };   // this lane: k + 8 half .. + 7
    auto load_b1 = [&](int d, int kk) {
      const int k = at(d, kk);
      if constexpr (BT) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          fw[d][kk][e] = __builtin_amdgcn_raw_buffer_load_b32(
              rb, k + half * 8 + e < p.Kd ? brow + (uint32_t)(k + e) * (uint32_t)p.ldb * 2u : OOB, 0, 0);
      } else {
        fb[d][kk] = __builtin_amdgcn_raw_buffer_load_b128(rb, k + half * 8 < p.Kd ? brow + (uint32_t)k * 2u : OOB, 0, 0);
      }
    };
    auto load_a1 = [&](int d, int kk) {                   // (whole 16-byte chunks, pad columns of a row hold zeros)
      const int k = at(d, kk);
      fa[d][kk] = __builtin_amdgcn_raw_buffer_load_b128(ra, k + half * 8 < p.Kd ? arow + (uint32_t)k * 2u : OOB, 0, CHAIN && GA == 0 ? SC1 : 0);
    };
    if (CHAIN && GA == 0 && first) {                      // the weights are under way while it waits for the signals
#pragma unroll
      for (int i = 0; i < D * KS; ++i) load_b1(i / KS, i % KS);
      chain_wait(link);
      load_e();
#pragma unroll
      for (int i = 0; i < D * KS; ++i) load_a1(i / KS, i % KS);
      first = false;
    } else if (CHAIN) {                                   // (and while the sample indices come)
#pragma unroll
      for (int i = 0; i < D * KS; ++i) load_b1(i / KS, i % KS);
#pragma unroll
      for (int i = 0; i < D * KS; ++i) load_a1(i / KS, i % KS);
    } else {
#pragma unroll
      for (int i = 0; i < D * KS; ++i) { load_a1(i / KS, i % KS); load_b1(i / KS, i % KS); }
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
    if (p.head.y) {                                       // uniform
      float sq, loss;
      const uint2 w = softmax_head(v, bv, nc, p.Nd, label, sq, loss);
      if (mr < Md) store_head(p.head, g, mr, nc, c8, label, w, sq, loss);
      return;
    }
    if (mr < Md) {
      float *C = static_cast<float *>(p.C) + (long long)g * p.sCg + (long long)mr * p.ldc;
#pragma unroll
      for (int e = 0; e < CPT; ++e) if (nc + e < p.Nd) C[nc + e] = v[e] + bv[e];
    }
    return;
  }
  small_out<BT, EPI, ACT, CHAIN>(p, g, tm, tn, Md, v, bv, ev, red, link);
}

// GA: 1: the batch gather rides behind the tiles; 2: and they read their rows of A from the dataset.
template <bool BT, int EPI, int ACT, int GA>
__global__ void __launch_bounds__(256) gemm_small_kernel(const GemmP p, const int tilesM, const int tilesN, const GatherP ga) {
  __shared__ __attribute__((aligned(16))) float red[SmallTile<BT, EPI>::LDS];
  int id = blockIdx.x;
  if (GA != 0) {
    const int tiles = tilesM * tilesN * p.groups;
    if (id >= tiles) { gather_riding_block<bf16_t>(ga, id - tiles); return; }
  }
  const int tn = id % tilesN;
  id /= tilesN;
  small_tile<BT, EPI, ACT, GA, false>(p, id / tilesM, id % tilesM, tn, red, ChainLink{});
}

// The passes of a step in one launch: forward, logits with the head and backward-data, where each of them would be a launch of 32-row
// tiles.  Apart they are bound by their starts and ends: 784-512-512-10, 8 replicas, b = 32: 5 launches of 6 to 9 us, a microsecond or
// two of each its loads and products; in one 22.6, the step 63 -> 51.6 us; 50 nets of 72 to 752 wide hidden layers, 1 to 16 replicas:
// steps 0.77 to 0.99 of the time (one 1.01: 784-456-17, 1 replica, b = 1024).
// A tile needs the tiles of the layer before on its own 32 rows of its replica and nothing else, so each such block of rows is a chain
// of its own: a work-group belongs to one (dealt round-robin, so that with 8 replicas each has its XCD), takes the next number of it
// when it starts, a tile in the order of the passes, reads its weights, waits for the layer before and goes on.  What a tile waits for
// has a lower number and is running or done, however many work-groups are on the chip and whatever else is.  The last work-group of
// a chain puts its words back to zero.  (One number for all chains cost more than it saved: 900 arrivals at one address, 56 us.)
// What bounds it (one chain, us from its start): numbers 0.5, index and rows of the dataset with the weights 3.6 (stragglers 5.4), a
// hand-over 0.9 (stores acknowledged 0.4, seen 0.5), activations past the L2 and products 1.6, epilogue 0.3 to 1.0; end at 17.7.
//
// Logits, head and the first backward-data are one pass: each of its tiles forms the signals of its 32 rows for itself (10 to 32
// classes: a few products per wave), which is shorter than handing them over.
template <int ACT>
__device__ __forceinline__ void head_bwd_tile(const GemmP &pz, const GemmP &p, const int g, const int tm, const int tn, float *red, const ChainLink &link) {
  constexpr int D = 4, KC = 64, KS = 4, RLD = SmallTile<false, EPI_LOGITS>::RLD, RLD2 = SmallTile<true, EPI_BWD>::RLD, SLD = 40;
  __shared__ __attribute__((aligned(16))) bf16_t sig[32 * SLD];
  const int m0 = tm * 32, n0 = tn * 64;
  const int Md = p.rows ? p.rows[g] : p.Md;
  if (m0 >= Md) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5, row = tid >> 3, c8 = tid & 7, mr = m0 + row;
  const int K = pz.Kd, classes = pz.Nd, nz = c8 * 4, nc = n0 + c8 * 8;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t *>(static_cast<const bf16_t *>(pz.A) + (long long)g * pz.sAg), 0, (int)((long long)Md * pz.lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(      // [classes][K] for both products
      const_cast<bf16_t *>(static_cast<const bf16_t *>(pz.B) + (long long)g * pz.sBg), 0, (int)((long long)classes * pz.ldb * 2), 0x00020000);
  const int id = pz.head.idx[(long long)g * pz.head.ldi + min(mr, Md - 1)];
  float bz[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) bz[e] = pz.bias && nz + e < classes ? pz.bias[(long long)g * pz.sBiasg + nz + e] : 0.0f;
  uint32_t fw[2][8];                                      // (wave 0 multiplies the signals: at most 32 of k)
  if (wave == 0) {
    const uint32_t brow = n0 + 2 * l32 < p.Nd ? (uint32_t)(half * 8 * p.ldb + n0 + 2 * l32) * 2u : OOB;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        fw[kk][e] = __builtin_amdgcn_raw_buffer_load_b32(rb, kk * 16 + half * 8 + e < classes ? brow + (uint32_t)(kk * 16 + e) * (uint32_t)p.ldb * 2u : OOB, 0, 0);
  }
  f32x16 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
  const uint32_t arow = m0 + l32 < Md ? ((uint32_t)(m0 + l32) * (uint32_t)pz.lda + (uint32_t)half * 8) * 2u : OOB;
  const uint32_t zrow = l32 < classes ? (uint32_t)(l32 * pz.ldb + half * 8) * 2u : OOB;
  uint4 ew = make_uint4(0, 0, 0, 0);
  int label = 0;
  bool first = true;
  for (int kb = wave * KC; kb < K || first; kb += D * 4 * KC) {
    u32x4_t fa[D * KS], fb[D * KS];
    auto at = [&](int i) -> int { return kb + i / KS * 4 * KC + i % KS * 16; };
#pragma unroll
    for (int i = 0; i < D * KS; ++i) fb[i] = __builtin_amdgcn_raw_buffer_load_b128(rb, at(i) + half * 8 < K ? zrow + (uint32_t)at(i) * 2u : OOB, 0, 0);
    if (first) {
      label = min(max(pz.head.y[min(max(id, 0), pz.head.N - 1)], 0), classes - 1);
      chain_wait(link);
      if (ACT != ACT_NONE && mr < Md && nc < p.Nd) ew = ld_agent(static_cast<const bf16_t *>(p.E) + (long long)g * p.sEg + (long long)mr * p.lde + nc);
      first = false;
    }
#pragma unroll
    for (int i = 0; i < D * KS; ++i) fa[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, at(i) + half * 8 < K ? arow + (uint32_t)at(i) * 2u : OOB, 0, SC1);
#pragma unroll
    for (int i = 0; i < D * KS; ++i)
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[i]), __builtin_bit_cast(bf16x8, fa[i]), acc[0], 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<float4 *>(red + (wave * 32 + l32) * RLD + q * 8 + half * 4) = make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
  __syncthreads();
  float4 s = *reinterpret_cast<const float4 *>(red + row * RLD + nz);
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    const float4 t = *reinterpret_cast<const float4 *>(red + (w * 32 + row) * RLD + nz);
    s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
  }
  const float v4[4] = {s.x, s.y, s.z, s.w};
  float sq, loss;
  const uint2 sg = softmax_head(v4, bz, nz, classes, label, sq, loss);
  *reinterpret_cast<uint2 *>(sig + row * SLD + nz) = sg;
  __syncthreads();                                        // (and the partial logits have been read)
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(sig + l32 * SLD + kk * 16 + half * 8);
      u32x4_t ce, co;                                     // as in small_tile
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ce[e] = __builtin_amdgcn_perm(fw[kk][2 * e + 1], fw[kk][2 * e], 0x05040100u);
        co[e] = __builtin_amdgcn_perm(fw[kk][2 * e + 1], fw[kk][2 * e], 0x07060302u);
      }
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ce), a, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, co), a, acc[1], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4 *>(red + l32 * RLD2 + j * 32 + q * 8 + half * 4) =
            make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
  }
  __syncthreads();
  float v[8], none[8];
  bf16_t ev[8];
  const uint32_t e4[4] = {ew.x, ew.y, ew.z, ew.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) { v[e] = red[row * RLD2 + (e & 1) * 32 + c8 * 4 + (e >> 1)]; none[e] = 0.0f; ev[e] = (bf16_t)(e4[e >> 1] >> (16 * (e & 1))); }
  small_out<true, EPI_BWD, ACT, true>(p, g, tm, tn, Md, v, none, ev, red, link);
  if (tn == 0 && mr < Md) store_head(pz.head, g, mr, nz, c8, label, sg, sq, loss);
}

template <int ACT>
__global__ void __launch_bounds__(256, 2) small_chain_kernel(const SmallChain c) {
  __shared__ __attribute__((aligned(16))) float red[SmallTile<true, EPI_BWD>::LDS];
  __shared__ int ticket;
  const int chain = blockIdx.x % c.chains, groups = c.gather.groups, g = chain % groups, tm = chain / groups, L = c.L;
  const int passes = 2 * L - 2, tiles = c.end[passes - 1];
  int *const words = c.count + (long long)chain * c.words;
  int mine = 0;
  if (threadIdx.x == 0) mine = __hip_atomic_fetch_add(words, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // (under way beside the number: the index of the row that this lane loads in the first pass)
  const int row = tm * 32 + (threadIdx.x & 31);
  const int src = min(max(c.gather.idx[(long long)g * c.gather.ldi + min(row, c.gather.b - 1)], 0), c.gather.N - 1);
  if (threadIdx.x == 0) ticket = mine;
  __syncthreads();
  const int id = __builtin_amdgcn_readfirstlane(ticket);
  if (id < tiles) {
    int ph = 0;
    while (id >= c.end[ph]) ++ph;                          // uniform
    const int before = ph > 0 ? c.end[ph - 1] : 0, before2 = ph > 1 ? c.end[ph - 2] : 0, tn = id - before;
    int *const set = words + 32;                           // a word per tile
    const ChainLink link = {set + before2, before - before2, ph < passes - 1 ? set + id : nullptr, c.polls, c.failed};
    const GemmP &p = c.p[ph < L ? ph : ph + 1];
    if (ph == 0) small_tile<false, EPI_FWD_ACT, ACT, 2, true>(p, g, tm, tn, red, link, src);
    else if (ph < L - 1) small_tile<false, EPI_FWD_ACT, ACT, 0, true>(p, g, tm, tn, red, link);
    else if (ph == L - 1) head_bwd_tile<ACT>(p, c.p[L], g, tm, tn, red, link);
    else small_tile<true, EPI_BWD, ACT, 0, true>(p, g, tm, tn, red, link);
  } else {
    const int blk = tm * 8 + id - tiles;                   // four rows each
    if (blk * 4 < c.gather.b) gather_rows_block<bf16_t>(c.gather, g, blk);
  }
  __syncthreads();
  if (threadIdx.x == 0) ticket = __hip_atomic_fetch_add(words + 16, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (ticket == tiles + 7)                                 // uniform: nobody is left who waits or takes a number
    for (int i = threadIdx.x; i < c.words; i += 256) __hip_atomic_store(words + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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

namespace {
// (beside the operand checks shared with the tiled family: gemm_bf16_operands_ok)
bool small_ok(const GemmP &p, int epi) {
  // 16-byte chunks of A (and of [n][k] operands) never cross the end of a row's storage; outputs, E and [k][n] operands are
  // touched in groups of 4 or 8 consecutive columns
  if (epi != EPI_LOGITS && ((p.Nd & 7) || (p.ldc & 7) || (p.sCg & 7) || (reinterpret_cast<uintptr_t>(p.C) & 15)))
    return false;
  if (p.head.y && (epi != EPI_LOGITS || !gemm_head_fits(1, p.Md, p.Nd, p.groups) || !p.head.idx || p.head.N < 1 || !p.head.D ||
                   !p.head.dn || !p.head.loss || p.head.ldd < p.Nd || p.head.ldd > 32 || (p.head.ldd & 7) || (p.head.sDg & 7) ||
                   (reinterpret_cast<uintptr_t>(p.head.D) & 15)))
    return false;
  if (p.gather && (epi == EPI_BWD || !gather_ok(*p.gather))) return false;
  if (epi == EPI_FWD_ACT && p.C2 && ((p.ldc2 & 7) || (p.sC2g & 7) || (reinterpret_cast<uintptr_t>(p.C2) & 15)))
    return false;
  if (epi == EPI_BWD && p.act != ACT_NONE && (!p.E || (p.lde & 7) || (p.sEg & 7) || (reinterpret_cast<uintptr_t>(p.E) & 15)))
    return false;
  return true;
}
}  // namespace

hipError_t launch_gemm_small(const GemmP &p, int epi, hipStream_t s) {
  if (!small_ok(p, epi)) return hipErrorInvalidValue;
  if (epi == EPI_FWD_ACT && !p.a_trans && !p.b_trans && !(p.Kd & 7)) return launch_act<false, EPI_FWD_ACT>(p, s);
  if (epi == EPI_LOGITS && !p.a_trans && !p.b_trans && !(p.Kd & 7)) return launch_act<false, EPI_LOGITS>(p, s);
  if (epi == EPI_BWD && !p.a_trans && p.b_trans) return launch_act<true, EPI_BWD>(p, s);
  return hipErrorInvalidValue;
}

int small_chain_words(int L, const int *dims) {
  int tiles = 0;
  for (int l = 1; l < L; ++l) tiles += (dims[l] + 31) / 32 + (dims[l] + 63) / 64;
  return 32 + (tiles + 31) / 32 * 32;
}

// Up to 224 chains: more of them share CUs, whose work-groups then poll beside others that work.  Time of a step against launches of their own,
// about 150 nets of 8 to 1600 inputs, 8 to 512 wide hidden layers, 1 to 511 replicas, workers with batches of their own among them: up to
// 128 chains 0.82 to 0.99, on average 0.91; 128 to 224 0.88 to 1.01; 224 to 256 0.98 to 1.06; 300 and more 0.99 to 1.09 (56-16-10, 486
// replicas, b = 6).
bool small_chain_fits(int L, const int *dims, int b, int groups, long long N, const int *rows_host) {
  if (L < 2 || L > SmallChain::MAXL || (long long)groups * ((b + 31) / 32) > SmallChain::MAX_CHAINS) return false;
  if (gather_rides(1, L, b, dims, groups, N, rows_host) != 1 || !gemm_head_fits(1, b, dims[L], groups)) return false;
  for (int l = 1; l < L; ++l)
    if (gemm_bf16_tile_shape(EPI_FWD_ACT, b, dims[l], groups, rows_host) != 5 || gemm_bf16_tile_shape(EPI_BWD, b, dims[l], groups, rows_host) != 5) return false;
  return true;
}

hipError_t launch_small_chain(SmallChain &c, hipStream_t s) {
  const int L = c.L, n = 2 * L - 1;
  if (L < 2 || L > SmallChain::MAXL || !c.count || !c.failed) return hipErrorInvalidValue;
  const int Md = c.p[0].Md, groups = c.p[0].groups, act = c.p[0].act;
  int tiles = 0;
  for (int i = 0; i < n; ++i) {
    const GemmP &p = c.p[i];
    const int epi = i < L - 1 ? EPI_FWD_ACT : i == L - 1 ? EPI_LOGITS : EPI_BWD;
    if (!gemm_bf16_operands_ok(p, epi) || !small_ok(p, epi) || gemm_bf16_tile_shape(epi, p.Md, p.Nd, p.groups, p.rows_host) != 5 ||
        p.a_trans || (p.b_trans != 0) != (epi == EPI_BWD) || (epi != EPI_BWD && (p.Kd & 7)) || p.Md != Md || p.groups != groups ||
        (epi != EPI_LOGITS && p.act != act) || (i == L && (p.Kd != c.p[L - 1].Nd || p.ldb != c.p[L - 1].ldb || p.B != c.p[L - 1].B)) || (i == 0) != (p.aidx != nullptr) || p.gather || (epi == EPI_LOGITS && !p.head.y) || p.rows != c.p[0].rows)
      return hipErrorInvalidValue;
    if (epi == EPI_LOGITS) continue;                       // (with the first backward-data)
    tiles += epi == EPI_BWD ? (p.Nd + 63) / 64 : (p.Nd + 31) / 32;
    c.end[i < L ? i : i - 1] = tiles;
  }
  if (c.words < 32 + tiles || !gather_ok(c.gather) || c.gather.b != Md || c.gather.groups != groups) return hipErrorInvalidValue;
  c.chains = (Md + 31) / 32 * groups;
  const long long blocks = (long long)c.chains * (tiles + 8);
  if (blocks > 0x3fffffff) return hipErrorInvalidValue;
  if (act == ACT_RELU) hipLaunchKernelGGL(small_chain_kernel<ACT_RELU>, dim3((unsigned)blocks), dim3(256), 0, s, c);
  else if (act == ACT_GELU) hipLaunchKernelGGL(small_chain_kernel<ACT_GELU>, dim3((unsigned)blocks), dim3(256), 0, s, c);
  else hipLaunchKernelGGL(small_chain_kernel<ACT_NONE>, dim3((unsigned)blocks), dim3(256), 0, s, c);
  return hipGetLastError();
}

}  // namespace absk
