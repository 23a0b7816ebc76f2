// The passes of a bf16 step over a block of rows of one replica, in one work-group: gather, forward, logits with the softmax head,
// backward-data.
//
// A row of the batch needs nothing of the other rows before the weight gradients, so a work-group that keeps a block of rows in LDS walks
// all layers without ever waiting for another one: the input of a layer lies in LDS, its output takes the same place, the weights
// stream from the XCD's L2 straight into registers as MFMA fragments, each wavefront those of its own columns.  Launches of their own
// (gather, a forward and a backward per layer, logits, head) had each a start, an end and a pass over memory for what the next one reads.
// What bounds it: the stream of weights, 1.2 us for 128 of k of a 512-wide layer, 44 bytes per clock and CU, about what an L2 gives.
// 784-512-512-10, 8 replicas, b = 501, blocks of 32 rows, us from a work-group's start: dataset rows in LDS 7.6, products of the first
// layer 16.8, its output 22.8, second layer 28.6 and 32.1, head 37.8, backward-data 44.8 and 55.1.
//   * v_mfma_f32_16x16x32_bf16 with the weights as the first operand: a lane's accumulators are four slots of one row.
//     Forward, column NT s + f of a wavefront's 16 NT is slot s of fragment f: a lane holds 4 NT consecutive columns.
// Out-of-range rows, columns and k come back as zeros from the buffer descriptor's range check.
#include "abs_internal.h"
#include "device_utils.h"
#include "gather.h"

namespace absk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// Addresses kept for another load's or pass's sake would spill: a value that the compiler takes for a new one
__device__ __forceinline__ void opaque(uint32_t &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ int this_lane() { uint32_t v = threadIdx.x & 63u; opaque(v); return (int)v; }

// byte offsets beyond any operand (weights and dataset are below 1 GiB); their sum, too
constexpr uint32_t OOB = 0x80000000u, OOB_K = 0x40000000u;
constexpr int WAVES = 8, MAX_IN = MlpRows::MAX_INPUTS, XST = MAX_IN + 8;    // wavefronts; the widest rows of the dataset, their stride in LDS
constexpr int MAX_CLASSES = MlpRows::MAX_CLASSES;

__device__ __forceinline__ void lds_barrier() {           // (loads and stores of memory stay in flight)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ float sum16(float v) { v += dpp<0xB1>(v); v += dpp<0x4E>(v); v += dpp<0x141>(v); return v + dpp<0x140>(v); }
template <int LANES> __device__ __forceinline__ float sum_lanes(float v) {      // over 32 neighbouring lanes or all 64, in all of them
  v = sum16(v);
  uint32_t u = __float_as_uint(v);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  if (LANES == 32) return v;
  u = __float_as_uint(v);
  r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float over_groups(float v, bool max) {               // over the lanes 16 apart
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) { const float t = __shfl_xor(v, o, 64); v = max ? fmaxf(v, t) : v + t; }
  return v;
}

// The weights of a pass as one wavefront reads them.
//   backward, [k][n]: a pair of steps of 32 of k at a time (words 0 .. 8 NT - 1 of w).  A lane loads 2 NT consecutive columns of every other
//     k; lanes r and r + 8 of 16, which have the same columns, exchange halves, so that each holds NT columns of 8 consecutive k.
//   forward, [n][k]: 128 of k at a time (16 NT words): word 16 f + 4 j + i.  The 16 lanes of a fragment are 16 rows; loaded as they are, every
//     four lanes would meet four cache lines (75 cycles for a 1 KB load, 2.3 us for 64 of k of a 512-wide layer).  So a quad of
//     lanes loads 64 consecutive bytes of one row, four rows one after the other, and exchanges them: lane i then holds the four
//     16-byte pieces of row i, which are four steps' operands.
struct Weights { __amdgpu_buffer_rsrc_t r; uint32_t base, ldb2; int K; };
__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_rsrc(const GemmP &p, int g, bool bt) {
  const bf16_t *B = static_cast<const bf16_t *>(p.B) + (long long)g * p.sBg;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(B), 0, (int)((long long)(bt ? p.Kd : p.Nd) * p.ldb * 2), 0x00020000);
}
template <bool BT, int NT> __device__ __forceinline__ Weights weights(const GemmP &p, int g, int cw0, int lane) {
  Weights w;
  w.r = weight_rsrc(p, g, BT);
  w.ldb2 = (uint32_t)p.ldb * 2u;
  w.K = p.Kd;
  const int q = lane >> 4, col = cw0 + (BT ? 2 * NT * (lane & 7) : NT * (lane & 12));     // (backward: Nd is a multiple of 8, 2 NT columns are all inside or none)
  w.base = !BT ? (uint32_t)col * w.ldb2 + (uint32_t)(q * 32 + (lane & 3) * 8) * 2u
               : col >= p.Nd ? OOB : (uint32_t)(q * 8 + ((lane >> 3) & 1)) * w.ldb2 + (uint32_t)col * 2u;
  return w;
}
template <int NT, int N> __device__ __forceinline__ void load_pair(uint32_t (&w)[N], int o, const Weights &q, int pair) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t row = q.base + (uint32_t)(64 * pair + 32 * h) * q.ldb2;          // (rows behind the last k lie behind the buffer's end)
    opaque(row);
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const uint32_t at = row + (uint32_t)e * q.ldb2;
      if constexpr (NT == 4) {
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(q.r, at, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[o + 16 * h + 2 * e + i] = v[i];
      } else {
        const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(q.r, at, 0, 0);
        w[o + 8 * h + e] = v[0]; w[o + 8 * h + e + 1] = v[1];
      }
    }
  }
}
// (rows behind the last column lie behind the buffer's end)
template <int NT, int N> __device__ __forceinline__ void load_unit(uint32_t (&w)[N], int o, const Weights &q, int unit, int lane) {
  uint32_t at = 128 * unit + (lane >> 4) * 32 + (lane & 3) * 8 < q.K ? q.base + (uint32_t)unit * 256u : OOB;
  opaque(at);
#pragma unroll
  for (int f = 0; f < NT; ++f)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(q.r, at + (uint32_t)(j * NT + f) * q.ldb2, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) w[o + 16 * f + 4 * j + i] = v[i];
    }
}
template <int CTRL> __device__ __forceinline__ void exchange(uint32_t &a, uint32_t &b, bool upper) {
  const uint32_t fa = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, CTRL, 0xf, 0xf, true), fb = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  a = upper ? fb : a;
  b = upper ? b : fa;
}
template <int NT, int N> __device__ __forceinline__ void transpose_unit(uint32_t (&w)[N], int o, int lane) {
  const bool odd = lane & 1, high = lane & 2;
#pragma unroll
  for (int f = 0; f < NT; ++f)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t *v = w + o + 16 * f + i;
      exchange<0xB1>(v[0], v[4], odd);
      exchange<0xB1>(v[8], v[12], odd);
      exchange<0x4E>(v[0], v[8], high);
      exchange<0x4E>(v[4], v[12], high);
    }
}
template <int NT, int N> __device__ __forceinline__ void transpose_pair(uint32_t (&w)[N], int o, int lane) {
  constexpr int H = NT / 2;                               // words of NT columns
  const bool upper = lane & 8;
#pragma unroll
  for (int v = 0; v < 8 * NT; v += 2 * H)                 // two rows of k
#pragma unroll
    for (int i = 0; i < H; ++i) exchange<0x128>(w[o + v + i], w[o + v + H + i], upper);
}
// step h of a pair (BT) or of a unit
template <bool BT, int NT, int N> __device__ __forceinline__ bf16x8 fragment(const uint32_t (&w)[N], int o, int h, int f) {
  u32x4_t v;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (BT) {                                   // the pair of k (2 i, 2 i + 1) of column f
      constexpr int H = NT / 2;                           // words of a k
      v[i] = __builtin_amdgcn_perm(w[o + 4 * NT * h + (2 * i + 1) * H + f / 2], w[o + 4 * NT * h + 2 * i * H + f / 2], f & 1 ? 0x07060302u : 0x05040100u);
    } else v[i] = w[o + 16 * f + 4 * h + i];
  }
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ void in_order() { __builtin_amdgcn_sched_barrier(0); }     // (moved up, the next step's reads would spill)
// The products of a pair or unit; row: this lane's row of the operand in LDS from its first k, rows 16 apart at 16 * ST
template <bool BT, int MT, int NT, int ST, int N>
__device__ __forceinline__ void multiply(f32x4_t (&acc)[MT][NT], const uint32_t (&w)[N], int o, const bf16_t *row, int lane) {
#pragma unroll
  for (int h = 0; h < (BT ? 2 : 4); ++h) {
    const bf16_t *a = row + (BT ? (lane >> 4) * 8 + 32 * h : (lane >> 4) * 32 + 8 * h);
    bf16x8 av[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) av[m] = *reinterpret_cast<const bf16x8 *>(a + m * 16 * ST);
#pragma unroll
    for (int f = 0; f < NT; ++f) {
      const bf16x8 b = fragment<BT, NT>(w, o, h, f);
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, av[m], acc[m][f], 0, 0, 0);
    }
    in_order();
  }
}
template <bool BT, int NT, int DU, int N> __device__ __forceinline__ void load_first(uint32_t (&w)[N], const Weights &q, int lane) {
  if constexpr (BT) {
#pragma unroll
    for (int u = 0; u < 2; ++u) { load_pair<NT>(w, 8 * NT * u, q, u); in_order(); }
  } else {
#pragma unroll
    for (int u = 0; u < DU; ++u) { load_unit<NT>(w, 16 * NT * u, q, u, lane); in_order(); }
  }
}
// the whole reduction over an input in LDS (row: this lane's), the first weights under way
template <int MT, int NT, int ST, int N>
__device__ __forceinline__ void reduce_backward(f32x4_t (&acc)[MT][NT], uint32_t (&w)[N], const Weights &q, const bf16_t *row, int lane) {
  constexpr int DP = 2;
  const int pairs = (q.K + 63) / 64, full = pairs / DP * DP;
  for (int s = 0; s < full; s += DP)
#pragma unroll
    for (int u = 0; u < DP; ++u) {
      transpose_pair<NT>(w, 8 * NT * u, lane);
      multiply<true, MT, NT, ST>(acc, w, 8 * NT * u, row + 64 * (s + u), lane);
      load_pair<NT>(w, 8 * NT * u, q, s + u + DP);  // (nothing beyond the last)
      in_order();
    }
#pragma unroll
  for (int u = 0; u < DP - 1; ++u)
    if (full + u < pairs) {
      transpose_pair<NT>(w, 8 * NT * u, lane);
      multiply<true, MT, NT, ST>(acc, w, 8 * NT * u, row + 64 * (full + u), lane);
    }
}
template <int MT, int NT, int DU, int ST, int N>
__device__ __forceinline__ void reduce_forward(f32x4_t (&acc)[MT][NT], uint32_t (&w)[N], const Weights &q, const bf16_t *row, int lane) {
  const int units = (q.K + 127) / 128, full = units / DU * DU;
  for (int s = 0; s < full; s += DU)
#pragma unroll
    for (int u = 0; u < DU; ++u) {
      transpose_unit<NT>(w, 16 * NT * u, lane);
      multiply<false, MT, NT, ST>(acc, w, 16 * NT * u, row + 128 * (s + u), lane);
      load_unit<NT>(w, 16 * NT * u, q, s + u + DU, lane);
      in_order();
    }
  if (DU > 1 && full < units) {
    transpose_unit<NT>(w, 0, lane);
    multiply<false, MT, NT, ST>(acc, w, 0, row + 128 * full, lane);
  }
}
template <int MT, int NT> __device__ __forceinline__ void clear(f32x4_t (&acc)[MT][NT]) {
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int f = 0; f < NT; ++f) acc[m][f] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
}

// The block's output to memory, with the squared norms of the stored rows
template <int R, int NT, int ST>
__device__ __forceinline__ void copy_out(const GemmP &p, int g, int m0, int Md, const bf16_t *lds) {
  constexpr int LPR = 16 * NT, PER = 64 / LPR * WAVES;    // lanes to a row, rows at once
  const int lane = this_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = (lane % LPR) * 8, first = wave * (64 / LPR) + lane / LPR;
  bf16_t *C = static_cast<bf16_t *>(p.C) + (long long)g * p.sCg;
#pragma unroll 4
  for (int i = 0; i < R / PER; ++i) {
    const int row = i * PER + first;
    if (m0 + row >= Md || c >= p.Nd) continue;
    const uint4 v = *reinterpret_cast<const uint4 *>(lds + row * ST + c);
    *reinterpret_cast<uint4 *>(C + (long long)(m0 + row) * p.ldc + c) = v;
  }
  if (!p.part) return;
#pragma unroll 4
  for (int i = 0; i < R / PER; ++i) {
    const int row = i * PER + first;
    float s = 0.0f, x[8];
    if (c < p.Nd) {
      Vec<bf16_t>::load(lds + row * ST + c, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) s = fmaf(x[e], x[e], s);
    }
    s = sum_lanes<LPR>(s);
    if (lane % LPR == 0 && m0 + row < Md) p.part[(long long)g * p.sPartg + m0 + row] = s;
  }
}

template <int MT, int NT, int ACT>
__global__ void __launch_bounds__(64 * WAVES, 2) mlp_rows_kernel(const MlpRows c) {
  constexpr int R = 16 * MT, CW = 16 * NT, ST = WAVES * CW + 8, DU = 2;
  constexpr int SST = MAX_CLASSES + 8, FZ = MAX_CLASSES / 16;
  constexpr int MAIN = 2 * R * ST > R * XST ? 2 * R * ST : R * XST;
  __shared__ __attribute__((aligned(16))) bf16_t lds[MAIN];                  // a layer's input, then its output; behind it the elementwise operand of backward-data
  __shared__ __attribute__((aligned(16))) bf16_t sig[R * SST];               // signals of the last layer
  // work-groups are dealt to the XCDs round-robin: each XCD takes a contiguous share of the blocks, so that few replicas' weights lie in its L2
  const int id = (int)(blockIdx.x & 7) * c.share + (int)(blockIdx.x >> 3);
  if (id >= c.blocks) return;
  const int g = id / c.per, blk = id - g * c.per, m0 = blk * R;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, q = lane >> 4, L = c.L, Md = c.p[0].Md;
  const int cw0 = wave * CW, col = cw0 + q * 4 * NT;      // this wavefront's columns, this lane's 4 NT of them
  f32x4_t acc[MT][NT];
  uint32_t w[16 * NT * DU];
  // (what the head needs of its rows, on its way from the start)
  int label = 0;
  if (wave < MT) {
    const HeadP &h = c.p[L - 1].head;
    const int n = h.idx[(long long)g * h.ldi + min(m0 + 16 * wave + r, Md - 1)];
    label = min(max(h.y[min(max(n, 0), h.N - 1)], 0), c.p[L - 1].Nd - 1);
  }

  // ---- first layer: the dataset's rows, on their way to the gathered batch
  {
    const GatherP &ga = c.gather;
    const GemmP &p = c.p[0];
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(ga.X), 0, (int)((long long)ga.N * ga.d * 2), 0x00020000);
    bf16_t *A0 = static_cast<bf16_t *>(ga.A0) + (long long)g * ga.sA0g + (long long)m0 * ga.ldo;
    // row by row, half a wavefront to each of two: 256 columns at a time
    constexpr int ROUNDS = R / 16, PIECES = (MAX_IN + 255) / 256;
    const int xr = tid >> 5, xc = (tid & 31) * 8;
    uint32_t src[ROUNDS];
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
      const int row = m0 + 16 * i + xr, at = ga.idx[(long long)g * ga.ldi + min(row, Md - 1)];
      src[i] = row < Md ? ((uint32_t)min(max(at, 0), ga.N - 1) * (uint32_t)ga.d + (uint32_t)xc) * 2u : OOB;
    }
    // Every line of the weights, shared out among the replica's work-groups on this XCD, and of the block's rows is touched once: all walk
    // the layers side by side, and each would otherwise wait for each new line to come from beyond the L2
    constexpr int PF = 2;
    uint32_t touched[PF];
    {
      const int lo = max((int)(blockIdx.x & 7) * c.share, g * c.per), hi = min(((int)(blockIdx.x & 7) + 1) * c.share, (g + 1) * c.per);
      const int peers = min(hi - lo, 32), at = id - lo;   // (32 CUs)
      const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<bf16_t *>(static_cast<const bf16_t *>(p.B) + (long long)g * p.sBg), 0, c.weight_bytes, 0x00020000);
#pragma unroll
      for (int i = 0; i < PF; ++i)
        touched[i] = __builtin_amdgcn_raw_buffer_load_b32(rw, at < peers ? (uint32_t)((i * peers + at) * 512 + tid) * 128u : OOB, 0, 0);
    }
    u32x4_t x[ROUNDS][PIECES];
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i)
#pragma unroll
      for (int k = 0; k < PIECES; ++k)
        x[i][k] = __builtin_amdgcn_raw_buffer_load_b128(rx, src[i] + (256 * k + xc < ga.d ? 512u * k : OOB_K), 0, 0);
    const Weights ww = weights<false, NT>(p, g, cw0, lane);
    if (MT <= 2) load_first<false, NT, DU>(w, ww, lane);  // (64 rows: no registers left beside them)
    clear(acc);
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
      float norm = 0.0f;
      const int row = 16 * i + xr;
#pragma unroll
      for (int k = 0; k < PIECES; ++k) {
        const u32x4_t v = x[i][k];
        float f[8];
        Vec<bf16_t>::unpack(make_uint4(v[0], v[1], v[2], v[3]), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) norm = fmaf(f[e], f[e], norm);
        if (256 * k + xc < MAX_IN) *reinterpret_cast<u32x4_t *>(lds + row * XST + 256 * k + xc) = v;
        if (m0 + row < Md && 256 * k + xc < ga.d) *reinterpret_cast<u32x4_t *>(A0 + (long long)row * ga.ldo + 256 * k + xc) = v;
      }
      norm = sum_lanes<32>(norm);
      if ((tid & 31) == 0 && m0 + row < Md) ga.an0[(long long)g * ga.sNg + m0 + row] = norm;
    }
    if (MT > 2) load_first<false, NT, DU>(w, ww, lane);
    lds_barrier();
    if (cw0 < p.Nd) reduce_forward<MT, NT, DU, XST>(acc, w, ww, lds + r * XST, lane);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < PF; ++i) asm volatile("" ::"v"(touched[i]));
  }
  // ---- hidden layers; acc: a layer's products, its input read
  auto output = [&](const GemmP &p) {
    const int lane = this_lane(), r = lane & 15, q = lane >> 4, col = cw0 + q * 4 * NT;
    if (cw0 < (p.Nd + 127) / 128 * 128) {                 // (the next pass reads 128 columns at a time: zeros behind the last one)
      float bias[4 * NT];
#pragma unroll
      for (int e = 0; e < 4 * NT; ++e) bias[e] = 0.0f;
      if (p.bias) {
#pragma unroll
        for (int e = 0; e < 4 * NT; e += 8)
          if (col + e < p.Nd) {                           // (Nd is a multiple of 8)
            const float4 *b = reinterpret_cast<const float4 *>(p.bias + (long long)g * p.sBiasg + col + e);
            const float4 lo = b[0], hi = b[1];
            bias[e] = lo.x; bias[e + 1] = lo.y; bias[e + 2] = lo.z; bias[e + 3] = lo.w;
            bias[e + 4] = hi.x; bias[e + 5] = hi.y; bias[e + 6] = hi.z; bias[e + 7] = hi.w;
          }
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        uint32_t o[2 * NT], o2[2 * NT];
#pragma unroll
        for (int e = 0; e < 4 * NT; e += 2) {
          float a[2], d[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) act_fwd<ACT>(acc[m][(e + h) % NT][e / NT] + bias[e + h], a[h], d[h]);
          o[e / 2] = pack2bf(a[0], a[1]);
          if (ACT == ACT_GELU) o2[e / 2] = pack2bf(d[0], d[1]);
        }
#pragma unroll
        for (int e = 0; e < 2 * NT; e += 4) {
          *reinterpret_cast<uint4 *>(lds + (16 * m + r) * ST + col + 2 * e) =
              col + 2 * e < p.Nd ? make_uint4(o[e], o[e + 1], o[e + 2], o[e + 3]) : make_uint4(0, 0, 0, 0);
          if (ACT == ACT_GELU && m0 + 16 * m + r < Md && col + 2 * e < p.Nd)
            *reinterpret_cast<uint4 *>(static_cast<bf16_t *>(p.C2) + (long long)g * p.sC2g + (long long)(m0 + 16 * m + r) * p.ldc2 + col + 2 * e) =
                make_uint4(o2[e], o2[e + 1], o2[e + 2], o2[e + 3]);
        }
        in_order();
      }
    }
    lds_barrier();
    copy_out<R, NT, ST>(p, g, m0, Md, lds);
  };
  for (int l = 1; l < L - 1; ++l) {
    const Weights ww = weights<false, NT>(c.p[l], g, cw0, this_lane());
    load_first<false, NT, DU>(w, ww, lane);
    output(c.p[l - 1]);
    clear(acc);
    if (cw0 < c.p[l].Nd) reduce_forward<MT, NT, DU, ST>(acc, w, ww, lds + r * ST, lane);
    lds_barrier();
  }
  // the weights of the logits, 16 classes at a time (k: at most 128 NT)
  const Weights wz = weights<false, 1>(c.p[L - 1], g, 0, this_lane());
  uint32_t hw[16 * NT];
  auto head_weights = [&](int f) {
    Weights v = wz;
    v.base += (uint32_t)(16 * f) * wz.ldb2;
#pragma unroll
    for (int u = 0; u < NT; ++u) load_unit<1>(hw, 16 * u, v, u, lane);
  };
  if (wave < MT) head_weights(0);
  output(c.p[L - 2]);
  // ---- logits and head: 16 rows to a wavefront
  if (wave < MT) {
    const GemmP &p = c.p[L - 1];
    const HeadP &h = p.head;
    const int lane = this_lane(), r = lane & 15, q = lane >> 4;
    const int row = m0 + 16 * wave + r, classes = p.Nd;
    f32x4_t z[FZ];
    const bf16_t *a = lds + (16 * wave + r) * ST + q * 32;
#pragma unroll
    for (int f = 0; f < FZ; ++f) {
      z[f] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
      if (16 * f >= classes) continue;                    // uniform
      if (f > 0) head_weights(f);
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        transpose_unit<1>(hw, 16 * u, lane);
        if (128 * u < p.Kd) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            z[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fragment<false, 1>(hw, 16 * u, j, 0), *reinterpret_cast<const bf16x8 *>(a + 128 * u + 8 * j),
                                                           z[f], 0, 0, 0);
        }
      }
    }
    float mx = -INFINITY, se = 0.0f;
    // (rows of a lane's four classes lie in its registers; 16 classes that are not there cost nothing)
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.bias ? p.bias + (long long)g * p.sBiasg : nullptr), 0,
                                                                        p.bias ? classes * 4 : 0, 0x00020000);
#pragma unroll
    for (int f = 0; f < FZ; ++f) {
      if (16 * f >= classes) continue;
      float bz[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) bz[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rz, (uint32_t)(16 * f + 4 * q + e) * 4u, 0, 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        z[f][e] = 16 * f + 4 * q + e < classes ? z[f][e] + bz[e] : -INFINITY;
        mx = fmaxf(mx, z[f][e]);
      }
    }
    mx = over_groups(mx, true);
    float ex[FZ][4];
#pragma unroll
    for (int f = 0; f < FZ; ++f) {
#pragma unroll
      for (int e = 0; e < 4; ++e) ex[f][e] = 0.0f;
      if (16 * f >= classes) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) { ex[f][e] = 16 * f + 4 * q + e < classes ? expf(z[f][e] - mx) : 0.0f; se += ex[f][e]; }
    }
    se = over_groups(se, false);
    const float inv = 1.0f / se, log_se = logf(se);
    float sq = 0.0f;
    const int padded = (classes + 63) / 64 * 64;          // what the first backward pass reads
    bf16_t *Drow = static_cast<bf16_t *>(h.D) + (long long)g * h.sDg + (long long)row * h.ldd;
#pragma unroll
    for (int f = 0; f < FZ; ++f) {
      const int k0 = 16 * f + 4 * q;
      if (16 * f >= padded) continue;                     // uniform
      float dl[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dl[e] = row < Md && k0 + e < classes ? ex[f][e] * inv - (k0 + e == label ? 1.0f : 0.0f) : 0.0f;
        const float st = bf2f(f2bf(dl[e]));
        sq = fmaf(st, st, sq);
        if (row < Md && k0 + e == label) h.loss[(long long)g * h.sNg + row] = -(z[f][e] - mx - log_se);
      }
      const uint2 v = make_uint2(pack2bf(dl[0], dl[1]), pack2bf(dl[2], dl[3]));
      *reinterpret_cast<uint2 *>(sig + (16 * wave + r) * SST + k0) = v;
      if (row < Md && k0 < h.ldd) *reinterpret_cast<uint2 *>(Drow + k0) = v;
    }
    sq = over_groups(sq, false);
    if (q == 0 && row < Md) h.dn[(long long)g * h.sNg + row] = sq;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the stores of the forward passes, which other lanes of this work-group read below
  load_first<true, NT, DU>(w, weights<true, NT>(c.p[L], g, cw0, lane), lane);
  lds_barrier();
  // ---- backward-data
  for (int i = L;; ++i) {
    const GemmP &p = c.p[i];
    const int lane = this_lane(), r = lane & 15, q = lane >> 4, col = cw0 + q * 4 * NT;
    const bool last = i == 2 * L - 2;
    clear(acc);
    // the elementwise operand, on its way beside the products: rows as copy_out has them
    constexpr int LPR = 16 * NT, PER = 64 / LPR * WAVES, EP = R / PER;
    const int ec = (lane % LPR) * 8, er = wave * (64 / LPR) + lane / LPR;
    uint4 ev[EP];
#pragma unroll
    for (int k = 0; k < EP; ++k) {
      ev[k] = make_uint4(0, 0, 0, 0);
      const int row = m0 + k * PER + er;
      if (ACT != ACT_NONE && row < Md && ec < p.Nd)
        ev[k] = *reinterpret_cast<const uint4 *>(static_cast<const bf16_t *>(p.E) + (long long)g * p.sEg + (long long)row * p.lde + ec);
    }
    if (cw0 < p.Nd) {
      const Weights ww = weights<true, NT>(p, g, cw0, lane);
      if (i == L) reduce_backward<MT, NT, SST>(acc, w, ww, sig + r * SST, lane);
      else reduce_backward<MT, NT, ST>(acc, w, ww, lds + r * ST, lane);
    }
    if (!last) {
      const Weights wn = weights<true, NT>(c.p[i + 1], g, cw0, lane);
      load_first<true, NT, DU>(w, wn, lane);
    }
    if (ACT != ACT_NONE) {
#pragma unroll
      for (int k = 0; k < EP; ++k) *reinterpret_cast<uint4 *>(lds + R * ST + (k * PER + er) * ST + ec) = ev[k];
    }
    lds_barrier();                                        // the input has been read
    if (cw0 < (p.Nd + 127) / 128 * 128) {
      // slot 4 q + j of fragment f: column 2 NT ((4 q + j) % 8) + NT (q / 2) + f
      const int c0 = cw0 + 8 * NT * (q & 1) + NT * (q >> 1);
      float cs[4 * NT];
#pragma unroll
      for (int e = 0; e < 4 * NT; ++e) cs[e] = 0.0f;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const bool live = m0 + 16 * m + r < Md;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          bf16_t *at = lds + (16 * m + r) * ST + c0 + 2 * NT * j;
          uint32_t ew[NT / 2], o[NT / 2];
#pragma unroll
          for (int i = 0; i < NT / 2; ++i) ew[i] = 0;
          if (ACT != ACT_NONE) {
            if constexpr (NT == 4) { const uint2 v = *reinterpret_cast<const uint2 *>(at + R * ST); ew[0] = v.x; ew[1] = v.y; }
            else ew[0] = *reinterpret_cast<const uint32_t *>(at + R * ST);
          }
#pragma unroll
          for (int f = 0; f < NT; f += 2) {
            float a[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const float v = acc[m][f + h][j], d = h ? __uint_as_float(ew[f / 2] & 0xffff0000u) : __uint_as_float(ew[f / 2] << 16);
              a[h] = ACT == ACT_RELU ? (d > 0.0f ? v : 0.0f) : ACT == ACT_GELU ? v * d : v;
              if (!live) a[h] = 0.0f;
            }
            o[f / 2] = pack2bf(a[0], a[1]);
            cs[NT * j + f] += __uint_as_float(o[f / 2] << 16);
            cs[NT * j + f + 1] += __uint_as_float(o[f / 2] & 0xffff0000u);
            if (c0 + 2 * NT * j >= p.Nd) o[f / 2] = 0;
          }
          if constexpr (NT == 4) *reinterpret_cast<uint2 *>(at) = make_uint2(o[0], o[1]);
          else *reinterpret_cast<uint32_t *>(at) = o[0];
        }
        in_order();
      }
      if (p.cpart) {
        float mine = 0.0f;
#pragma unroll
        for (int e = 0; e < 4 * NT; ++e) {
          const float s = sum16(cs[e]);
          mine = r == e ? s : mine;
        }
        const int to = c0 + 2 * NT * (r / NT) + r % NT;
        if (r < 4 * NT && to < p.Nd) p.cpart[(long long)g * p.sCpartg + (long long)blk * p.Nd + to] = mine;
      }
    }
    lds_barrier();
    copy_out<R, NT, ST>(p, g, m0, Md, lds);
    if (last) break;
  }
}

template <int MT, int NT> hipError_t launch_act(const MlpRows &c, hipStream_t s) {
  const dim3 grid((unsigned)(c.share * 8)), block(64 * WAVES);
  if (c.p[0].act == ACT_RELU) hipLaunchKernelGGL((mlp_rows_kernel<MT, NT, ACT_RELU>), grid, block, 0, s, c);
  else if (c.p[0].act == ACT_GELU) hipLaunchKernelGGL((mlp_rows_kernel<MT, NT, ACT_GELU>), grid, block, 0, s, c);
  else hipLaunchKernelGGL((mlp_rows_kernel<MT, NT, ACT_NONE>), grid, block, 0, s, c);
  return hipGetLastError();
}
template <int NT> hipError_t launch_rows(const MlpRows &c, hipStream_t s) {
  return c.rows == 16 ? launch_act<1, NT>(c, s) : c.rows == 32 ? launch_act<2, NT>(c, s) : launch_act<4, NT>(c, s);
}

}  // namespace

// The fewer rows to a block the more CUs have one, and all of them stream the weights, which is what the time goes by: 16 rows while that
// makes one round of 256 CUs, then 32, then 64; of 32 rows of layers up to 256 two blocks fit a CU, which suits
// all larger batches better.  Fewer blocks than the first line leave CUs idle that tiles of 32 x 32 outputs would use; more than one round
// of a wide layer's blocks reads the weights more often than tiles of 128 or 256 rows do (784-512-512-10, 8 replicas, b = 4096: 248 us per
// step in tiles, 250 in blocks of 64, 303 in blocks of 32).
// Time of a step against tiles, about 1300 nets of 8 to 896 inputs and one to three hidden layers of 8 to 512, 1 to 600 replicas, b = 2 to 8192:
//   16 rows, and 32 up to 256 blocks: 0.73 to 1.03, on average 0.91 (one 1.07: 464-112-114, 1 replica, b = 2283);
//   64 rows in one round, layers up to 256: 0.71 to 1.03, on average 0.91; in two rounds up to 1.25 (400-56-272-64-18, 133 replicas, b = 77);
//   64 rows, wider layers: from 192 blocks on 0.83 to 1.00; fewer of them with 800 and more inputs and hidden units 0.87 to 1.00, with less
//     0.93 to 1.06: half the CUs idle, and little for each to load;
//   32 rows, 257 to 768 blocks: 0.74 to 1.02 (one 1.04: 56-56-84, 21 replicas, b = 945), except where replicas of less than half a block make
//     them mostly empty (up to 1.10);
//   more of them: a round costs what its barriers do however few wavefronts have columns, or rows of the head, while tiles cost by the widths and
//     get better with every round.  490 nets: with hidden layers of 128 on average, each from 64, to 1536 blocks and 64 classes 0.77 to 1.00, from 320
//     inputs, whose gather is spared, to 2048 and 96 classes 0.77 to 1.00, both 0.90 on average (220 nets outside the fit 0.91, at most 1.03); narrower layers up to 1.37 (16-56-8-8-4, 31
//     replicas, b = 3547 192 -> 261 us), one of them among wide ones up to 1.06, more classes up to 1.13 (32-168-107, 11 replicas, b = 5369
//     141 -> 159), more blocks up to 1.26 (32-152-40-256-103, 95 replicas, b = 4599 1133 -> 1424).
// Inputs end at 896, 784 to the next 128: registers and LDS would hold 1024, which nothing has measured.
// For example, us per step: 784-512-512-10, 8 replicas, b = 1000 120 -> 104, 784-160-160-160-3 (GELU), 7 replicas, b = 479 87 -> 69,
// 784-328-328-328-34 (GELU), 16 replicas, b = 669 198 -> 166.
int mlp_rows_block(int L, const int *dims, int b, int groups, long long N) {
  if (L < 2 || L > MlpRows::MAXL || dims[L] > MAX_CLASSES || dims[0] > MAX_IN || N * dims[0] * 2 >= (1LL << 30)) return 0;
  int width = 0, sum = 0, narrowest = 64 * WAVES;
  for (int l = 1; l < L; ++l) { width = dims[l] > width ? dims[l] : width; narrowest = dims[l] < narrowest ? dims[l] : narrowest; sum += dims[l]; }
  auto blocks = [&](int rows) { return (long long)((b + rows - 1) / rows) * groups; };
  const bool wide = width > 32 * WAVES;
  if (width > 64 * WAVES || blocks(16) < (wide ? 216 : 140)) return 0;
  if (blocks(16) <= 256) return 16;
  if (blocks(32) <= 256) return 32;
  if (blocks(64) <= 256) return !wide || blocks(64) >= 192 || dims[0] + sum >= 800 ? 64 : 0;
  if (wide || (long long)b * groups < 16 * blocks(32)) return 0;
  if (blocks(32) <= 768) return 32;
  if (sum < 128 * (L - 1) || narrowest < 64) return 0;
  const bool deep = dims[0] >= 320;
  return blocks(32) <= (deep ? 2048 : 1536) && dims[L] <= (deep ? 96 : 64) ? 32 : 0;
}

hipError_t launch_mlp_rows(MlpRows &c, hipStream_t s) {
  const int L = c.L;
  if (L < 2 || L > MlpRows::MAXL || (c.rows != 16 && c.rows != 32 && c.rows != 64)) return hipErrorInvalidValue;
  const GemmP &f = c.p[0], &z = c.p[L - 1];
  const GatherP &ga = c.gather;
  int width = 0;
  for (int i = 0; i < 2 * L - 1; ++i) {
    const GemmP &p = c.p[i];
    const bool fwd = i < L - 1, bwd = i >= L;
    if (p.Md != f.Md || p.groups != f.groups || p.rows || p.gather || p.a_trans || (p.b_trans != 0) != bwd || p.Nd < 1 || p.Kd < 1) return hipErrorInvalidValue;
    if (!p.B || (p.ldb & 7) || (p.sBg & 7) || (reinterpret_cast<uintptr_t>(p.B) & 15) || p.ldb < (bwd ? p.Nd : p.Kd) ||
        (long long)(bwd ? p.Kd : p.Nd) * p.ldb * 2 >= (1LL << 30)) return hipErrorInvalidValue;
    if (i > 0 && p.Kd != c.p[i - 1].Nd) return hipErrorInvalidValue;            // a pass reads what the one before left
    if (i == L - 1) continue;
    if (p.act != f.act || (p.Nd & 7) || p.Nd > 64 * WAVES || !p.C || (p.ldc & 7) || p.ldc < p.Nd || (p.sCg & 7) || (reinterpret_cast<uintptr_t>(p.C) & 15)) return hipErrorInvalidValue;
    if (fwd && ((p.Kd & 7) || (p.bias && ((p.sBiasg & 3) || (reinterpret_cast<uintptr_t>(p.bias) & 15))))) return hipErrorInvalidValue;
    if (fwd && p.act == ACT_GELU && (!p.C2 || (p.ldc2 & 7) || p.ldc2 < p.Nd || (p.sC2g & 7) || (reinterpret_cast<uintptr_t>(p.C2) & 15))) return hipErrorInvalidValue;
    if (bwd && p.act != ACT_NONE && (!p.E || (p.lde & 7) || p.lde < p.Nd || (p.sEg & 7) || (reinterpret_cast<uintptr_t>(p.E) & 15))) return hipErrorInvalidValue;
    width = p.Nd > width ? p.Nd : width;
  }
  if (z.Nd > MAX_CLASSES || (z.Kd & 7) || !z.head.y || !z.head.idx || z.head.N < 1 || !z.head.D || !z.head.dn || !z.head.loss || z.head.ldd < z.Nd ||
      z.head.ldd > MAX_CLASSES || (z.head.ldd & 7) || (z.head.sDg & 7) || (reinterpret_cast<uintptr_t>(z.head.D) & 15)) return hipErrorInvalidValue;
  if (!ga.X || !ga.idx || !ga.A0 || !ga.an0 || ga.ldo < ga.d || ga.ldi < ga.b || ga.b != f.Md || ga.groups != f.groups || ga.d != f.Kd || (ga.d & 7) || (ga.ldo & 7) || (ga.sA0g & 7) || ga.d > MAX_IN || ga.rows || ga.N < 1 ||
      (long long)ga.N * ga.d * 2 >= (1LL << 30) || (reinterpret_cast<uintptr_t>(ga.X) & 15) || (reinterpret_cast<uintptr_t>(ga.A0) & 15)) return hipErrorInvalidValue;
  c.per = (f.Md + c.rows - 1) / c.rows;
  const long long blocks = (long long)c.per * f.groups;
  if (blocks > 0x3fffffff) return hipErrorInvalidValue;
  c.blocks = (int)blocks;
  c.share = (c.blocks + 7) / 8;
  const long long bytes = (static_cast<const bf16_t *>(z.B) - static_cast<const bf16_t *>(f.B) + (long long)z.Nd * z.ldb) * 2;
  if (bytes <= 0 || bytes > f.sBg * 2) return hipErrorInvalidValue;             // (layer behind layer in a replica's vector)
  c.weight_bytes = (int)bytes;
  return width <= 32 * WAVES ? launch_rows<2>(c, s) : launch_rows<4>(c, s);
}

}  // namespace absk
