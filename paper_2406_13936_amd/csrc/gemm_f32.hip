// Replica-batched fp32 GEMM (plain vector ALU, LDS-tiled) for the fp32 precision mode:
//   C[g][m][n] = sum_k A[g][m][k] * B[g][n][k]
// with the same operand-layout flags and epilogues as the bf16 matrix-core family.  The fp32
// mode serves small problems (logistic regression), whose launches are bound by latency: a serial walk over k in a few
// work-groups.  So the tile is small and the k-step long where the output is small (TS x TS outputs per block and BK of k
// per step: 16 x 256, 32 x 128 or 64 x 32; 256 threads, (TS / 16)^2 outputs per thread), every load of a step is in flight at
// once, and the next step's operands are fetched into registers while the current one is multiplied.  Operands sit in LDS as
// [row][BK + 4], so that four k of a row are one 16-byte read without bank conflicts.  Generality (arbitrary strides and
// extents) comes before peak rate.  Measured against 32 x 32 x 32 tiles on 4 replicas, 256 features, 10 classes: logits
// 11.1 -> 5.7 us at b = 16, 12.0 -> 6.0 at b = 512; weight gradient with the bias sums at b = 512 10.3 us in one launch, before
// 7.8 + 4.9 (split and finish) + 3.3 + 1.9 (column sums).
// Weight gradients on 64 x 64 tiles, whose operands both come row-contiguous, keep them so in LDS ([k][64 + 4], four rows of a
// k per read): as [row][BK + 4] their stores met in 16 of the 64 banks and the loop took 180 registers, two waves to a SIMD
// (106 and four now): 256 x 1024 outputs of 8 replicas, b = 8192: 683 -> 512 us.
#include <algorithm>
#include "abs_internal.h"
#include "device_utils.h"
#include "gather.h"

namespace absk {
namespace {

constexpr int KSTEP[5] = {0, 256, 128, 0, 32};     // k-step of the tile of 16 times the index

// (EPI_WGRAD with GemmP::upd_x: ACT carries the optimizer, NO_STEP without)
constexpr int NO_STEP = 15;

// GA: the batch gather rides in slices of the grid behind the tiles, which read their rows of A from the dataset.
template <int EPI, int ACT, int TS, int BK, bool GA>
__global__ void __launch_bounds__(256) gemm_f32_kernel(const GemmP pin, const GatherP ga) {
  constexpr int PT = TS * BK / 256;              // elements per thread, operand and k-step
  constexpr int R = TS / 16;                     // outputs per thread and dimension
  constexpr int LD = BK + 4;
  constexpr bool AT = EPI == EPI_WGRAD, BT = EPI == EPI_WGRAD || EPI == EPI_BWD;   // operand layouts (GemmP::a_trans, b_trans)
  constexpr bool KM = EPI == EPI_WGRAD && TS == 64;   // operands in LDS as [k][TS + 4]: a thread's rows and columns are R neighbours
  constexpr int STAGE = KM ? BK * (TS + 4) : TS * LD;
  __shared__ __attribute__((aligned(16))) float lds[2 * STAGE];
  float *const As = lds, *const Bs = lds + STAGE;
  auto slot = [](int rr, int kk) -> int { return KM ? kk * (TS + 4) + rr : rr * LD + kk; };
  if (GA && (int)blockIdx.z >= pin.groups) {
    gather_riding_block<float>(ga, ((int)(blockIdx.z - pin.groups) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
    return;
  }
  // blockIdx.z = group, or (group, k-slice) of a weight gradient whose reduction is split
  const int ksplit = (EPI == EPI_WGRAD && pin.ksplit > 1) ? pin.ksplit : 1;
  const int g = blockIdx.z / ksplit, ksl = blockIdx.z - g * ksplit;
  const int m0 = blockIdx.y * TS, n0 = blockIdx.x * TS;
  GemmP p = pin;
  if (p.rows) {                                   // ragged groups: this group's own extent
    const int r = p.rows[g];
    if (p.rows_is_k) { p.Kd = r; p.alpha = 1.0f / (float)r; } else p.Md = r;
    if (m0 >= p.Md) return;                       // uniform over the block, before any barrier
  }
  int kbeg = 0;
  if (ksplit > 1) {                               // this block's slice; an empty one writes zeros
    kbeg = ksl * p.kchunk;
    const int kend = kbeg + p.kchunk;
    if (kend < p.Kd) p.Kd = kend;
    if (kbeg > p.Kd) kbeg = p.Kd;
  }
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const float *A = static_cast<const float *>(p.A) + (long long)g * p.sAg;
  const float *B = static_cast<const float *>(p.B) + (long long)g * p.sBg;
  float acc[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[i][j] = 0.0f;
  // row sums of A over k (bias gradients: the first column of blocks takes them): four chains per k-step, then a sum of steps
  const bool row_sums = EPI == EPI_WGRAD && p.rowsum && blockIdx.x == 0;
  float rs[R];
#pragma unroll
  for (int i = 0; i < R; ++i) rs[i] = 0.0f;

  int labels[R];                                  // (two dependent loads: under way while the operands arrive)
  if (EPI == EPI_LOGITS && p.head.y) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int id = p.head.idx[(long long)g * p.head.ldi + min(m0 + ty + 16 * i, p.Md - 1)];
      labels[i] = min(max(p.head.y[min(max(id, 0), p.head.N - 1)], 0), p.Nd - 1);
    }
  }

  float ra[PT], rb[PT];
  // element e of this thread: (row rr, k kk) of a stage; consecutive threads walk the operand's contiguous dimension
  auto where = [&](int e, bool trans, int &rr, int &kk) {
    const int id = tid + e * 256;
    if (!trans) { kk = id % BK; rr = id / BK; } else { rr = id % TS; kk = id / TS; }
  };
  int src[GA ? PT : 1];                           // rows of the dataset
  if constexpr (GA) {
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      int rr, kk;
      where(e, false, rr, kk);
      src[e] = dataset_row(p, g, min(m0 + rr, p.Md - 1));
    }
  }
  // addresses are clamped into the operand here; what lies outside it is replaced by zeros on the way to LDS, so that
  // nothing waits for these loads before the multiplications they overlap with
  auto fetch = [&](int k0) {
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      int rr, kk;
      where(e, AT, rr, kk);
      const int m = min(m0 + rr, p.Md - 1), k = min(k0 + kk, p.Kd - 1);
      if constexpr (GA) ra[e] = A[(long long)src[e] * p.lda + k];
      else ra[e] = AT ? A[(long long)k * p.lda + m] : A[(long long)m * p.lda + k];
    }
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      int rr, kk;
      where(e, BT, rr, kk);
      const int n = min(n0 + rr, p.Nd - 1), k = min(k0 + kk, p.Kd - 1);
      rb[e] = BT ? B[(long long)k * p.ldb + n] : B[(long long)n * p.ldb + k];
    }
  };
  // Weight gradients sum over the batch, which may be long: in one chain per output the sum loses a digit against one cut into
  // slices (784 -> 10, b = 1024: relative error 5.4e-7, in slices 1.7e-7, as here 1.3e-7; the same time).  So at most 128
  // products follow one another (in the smaller tiles 32 in each of four chains), and these sums are added up.
  float part[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) part[i][j] = 0.0f;
  auto join = [&]() {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j) { acc[i][j] += part[i][j]; part[i][j] = 0.0f; }
  };
  if (kbeg < p.Kd) fetch(kbeg);
  for (int k0 = kbeg; k0 < p.Kd; k0 += BK) {
    float fs = 0.0f;
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      int rr, kk;
      where(e, AT, rr, kk);
      const float av = m0 + rr < p.Md && k0 + kk < p.Kd ? ra[e] : 0.0f;
      As[slot(rr, kk)] = av;
      if (KM) fs += av;                           // (a thread fetches PT of k of one row)
      where(e, BT, rr, kk);
      Bs[slot(rr, kk)] = n0 + rr < p.Nd && k0 + kk < p.Kd ? rb[e] : 0.0f;
    }
    __syncthreads();
    if (k0 + BK < p.Kd) fetch(k0 + BK);
    if constexpr (KM) {
      if (row_sums) rs[0] += fs;                 // (uniform; the four threads of a row meet below)
#pragma unroll
      for (int k = 0; k < BK; ++k) {             // (all of them: what lies beyond Kd is zero)
        const float4 a4 = *reinterpret_cast<const float4 *>(As + k * (TS + 4) + ty * R);
        const float4 b4 = *reinterpret_cast<const float4 *>(Bs + k * (TS + 4) + tx * R);
        const float a[4] = {a4.x, a4.y, a4.z, a4.w}, b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j) part[i][j] = fmaf(a[i], b[j], part[i][j]);
      }
      if ((k0 & 96) == 96) join();               // (uniform: kbeg is a multiple of 128)
    } else if constexpr (EPI == EPI_WGRAD) {
      const int k4 = (min(BK, p.Kd - k0) + 3) / 4;
      for (int q0 = 0; q0 < k4; q0 += 32) {
        float4 ks[R], c4[R][R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          ks[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int j = 0; j < R; ++j) c4[i][j] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const int q1 = min(q0 + 32, k4);
#pragma unroll 8
        for (int q = q0; q < q1; ++q) {
          float4 a[R], b[R];
#pragma unroll
          for (int i = 0; i < R; ++i) a[i] = *reinterpret_cast<const float4 *>(As + (ty + 16 * i) * LD + q * 4);
#pragma unroll
          for (int j = 0; j < R; ++j) b[j] = *reinterpret_cast<const float4 *>(Bs + (tx + 16 * j) * LD + q * 4);
#pragma unroll
          for (int i = 0; i < R; ++i) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
              c4[i][j].x = fmaf(a[i].x, b[j].x, c4[i][j].x); c4[i][j].y = fmaf(a[i].y, b[j].y, c4[i][j].y);
              c4[i][j].z = fmaf(a[i].z, b[j].z, c4[i][j].z); c4[i][j].w = fmaf(a[i].w, b[j].w, c4[i][j].w);
            }
            ks[i].x += a[i].x; ks[i].y += a[i].y; ks[i].z += a[i].z; ks[i].w += a[i].w;
          }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
          rs[i] += (ks[i].x + ks[i].y) + (ks[i].z + ks[i].w);
#pragma unroll
          for (int j = 0; j < R; ++j) acc[i][j] += (c4[i][j].x + c4[i][j].y) + (c4[i][j].z + c4[i][j].w);
        }
      }
    } else {
      const int k4 = (min(BK, p.Kd - k0) + 3) / 4;
#pragma unroll 8
      for (int q = 0; q < k4; ++q) {
        float4 a[R], b[R];
#pragma unroll
        for (int i = 0; i < R; ++i) a[i] = *reinterpret_cast<const float4 *>(As + (ty + 16 * i) * LD + q * 4);
#pragma unroll
        for (int j = 0; j < R; ++j) b[j] = *reinterpret_cast<const float4 *>(Bs + (tx + 16 * j) * LD + q * 4);
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j)
            acc[i][j] = fmaf(a[i].w, b[j].w, fmaf(a[i].z, b[j].z, fmaf(a[i].y, b[j].y, fmaf(a[i].x, b[j].x, acc[i][j]))));
      }
    }
    __syncthreads();
  }
  if constexpr (KM) {                             // (the last k-step ended with a barrier)
    join();
    if (row_sums) {                               // uniform
      As[tid] = rs[0];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int r = ty + 16 * i;
        rs[i] = (As[r] + As[TS + r]) + (As[2 * TS + r] + As[3 * TS + r]);
      }
      __syncthreads();
    }
    // outputs from R x R neighbours to rows ty + 16 i and columns tx + 16 j, whose accesses are runs of 64 bytes (a step of
    // AdamW touches seven words per output)
    static_assert(2 * STAGE >= TS * (TS + 4), "the tile passes through LDS");
#pragma unroll
    for (int i = 0; i < R; ++i)
      *reinterpret_cast<float4 *>(lds + (ty * R + i) * (TS + 4) + tx * R) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j) acc[i][j] = lds[(ty + 16 * i) * (TS + 4) + tx + 16 * j];
  }
  // the optimizer step where the gradient is finished: parameter, state and squared entry of the gradient at offset o of group g
  constexpr bool STEP = EPI == EPI_WGRAD && ACT != NO_STEP;
  constexpr int OPT = STEP ? ACT : OPT_SGD;
  OptHyper h = {p.upd_lr, p.upd_momentum, p.upd_beta1, p.upd_beta2, p.upd_eps, p.upd_wd, p.upd_c1, p.upd_c2};
  if (STEP && p.upd_scal) { h.lr = p.upd_scal[0]; h.c1 = p.upd_scal[1]; h.c2 = p.upd_scal[2]; }
  double sq = 0.0;
  auto step = [&](long long o, float gr) {
    float x = p.upd_x[o], v = OPT != OPT_SGD ? p.upd_v[o] : 0.0f, m = OPT == OPT_ADAMW ? p.upd_m[o] : 0.0f;
    opt_step_elem<OPT>(x, gr, v, m, h);
    p.upd_x[o] = x;
    if (OPT != OPT_SGD) p.upd_v[o] = v;
    if (OPT == OPT_ADAMW) p.upd_m[o] = m;
    sq += (double)(gr * gr);
  };
  if (row_sums && tx == 0) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int m = m0 + ty + 16 * i;
      float *o = p.rowsum + (long long)g * p.sRowsumg + m;
      if (m < p.Md) {
        const float gr = p.accumulate ? fmaf(rs[i], p.alpha, *o) : rs[i] * p.alpha;
        *o = gr;
        if (STEP) step((long long)g * p.sCg + (p.rowsum - static_cast<float *>(p.C)) + m, gr);
      }
    }
  }

  const float *bias = p.bias ? p.bias + (long long)g * p.sBiasg : nullptr;
  if (EPI == EPI_LOGITS && p.head.y) {            // uniform: softmax cross-entropy, class tx of row ty + 16 i (at most 16 classes)
    const float bv = bias && tx < p.Nd ? bias[tx] : 0.0f;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int m = m0 + ty + 16 * i;
      const int label = labels[i];
      const float z = tx < p.Nd ? acc[i][0] + bv : -INFINITY;
      float mx = z;
#pragma unroll
      for (int x = 1; x < 16; x <<= 1) mx = fmaxf(mx, __shfl_xor(mx, x, 64));
      const float ex = tx < p.Nd ? expf(z - mx) : 0.0f;
      float se = ex;
#pragma unroll
      for (int x = 1; x < 16; x <<= 1) se += __shfl_xor(se, x, 64);
      const float dl = tx < p.Nd ? ex * (1.0f / se) - (tx == label ? 1.0f : 0.0f) : 0.0f;
      float sq = dl * dl;
#pragma unroll
      for (int x = 1; x < 16; x <<= 1) sq += __shfl_xor(sq, x, 64);
      if (m < p.Md) {
        const long long at = (long long)g * p.head.sNg + m;
        if (tx < p.head.ldd) static_cast<float *>(p.head.D)[(long long)g * p.head.sDg + (long long)m * p.head.ldd + tx] = dl;
        if (tx == 0) p.head.dn[at] = sq;
        if (tx == label) p.head.loss[at] = -(z - mx - logf(se));
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int m = m0 + ty + 16 * i;
    if (m >= p.Md) continue;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int n = n0 + tx + 16 * j;
      const bool nin = n < p.Nd;
      const float v = acc[i][j];
      const float bv = (bias && nin) ? bias[n] : 0.0f;
      if (EPI == EPI_FWD_ACT) {
        if (n < p.ldc && (nin || p.pad_to_ld)) {
          float a = 0.0f, d = 0.0f;
          if (nin) act_fwd<ACT>(v + bv, a, d);
          static_cast<float *>(p.C)[(long long)g * p.sCg + (long long)m * p.ldc + n] = a;
          if (ACT == ACT_GELU && p.C2)
            static_cast<float *>(p.C2)[(long long)g * p.sC2g + (long long)m * p.ldc2 + n] = d;
        }
      } else if (EPI == EPI_LOGITS) {
        if (nin) static_cast<float *>(p.C)[(long long)g * p.sCg + (long long)m * p.ldc + n] = v + bv;
      } else if (EPI == EPI_BWD) {
        if (n < p.ldc && (nin || p.pad_to_ld)) {
          float o = 0.0f;
          if (nin) {
            float e = 1.0f;
            if (ACT != ACT_NONE) e = static_cast<const float *>(p.E)[(long long)g * p.sEg + (long long)m * p.lde + n];
            o = (ACT == ACT_RELU) ? (e > 0.0f ? v : 0.0f) : (ACT == ACT_GELU ? v * e : v);
          }
          static_cast<float *>(p.C)[(long long)g * p.sCg + (long long)m * p.ldc + n] = o;
        }
      } else if (EPI == EPI_WGRAD) {
        if (nin && ksplit > 1) {                  // raw partial product of this k-slice, packed Md x Nd
          p.kpart[((long long)g * ksplit + ksl) * p.Md * p.Nd + (long long)m * p.Nd + n] = v;
        } else if (nin) {
          float *o = static_cast<float *>(p.C) + (long long)g * p.sCg + (long long)m * p.ldc + n;
          const float gr = p.accumulate ? fmaf(v, p.alpha, *o) : v * p.alpha;
          *o = gr;
          if (STEP) step((long long)g * p.sCg + (long long)m * p.ldc + n, gr);
        }
      }
    }
  }
  if (STEP) {
    __shared__ double red[4];
    const double t = block_sum<4>(sq, red);
    if (tid == 0) p.upd_sq[(long long)g * p.upd_sSqg + p.upd_slot0 + blockIdx.y * gridDim.x + blockIdx.x] = (float)t;
  }
}

constexpr int F32_MAX_SPLIT = 8, F32_MAX_SPLIT_BLOCKS = 1024;   // slices of a reduction; blocks of a launch that is split

int tile_size(int Md, int Nd, long long groups) {
  // 32 x 32 tiles while 64 x 64 ones would leave most CUs without a work-group, 16 x 16 while 32 x 32 ones would
  auto blocks = [&](int ts) { return (long long)((Nd + ts - 1) / ts) * ((Md + ts - 1) / ts) * groups; };
  return blocks(64) >= 128 ? 64 : blocks(32) >= 128 ? 32 : 16;
}

template <int EPI, int ACT, bool GA>
hipError_t launch2(const GemmP &p, const GatherP &ga, int ts, dim3 grid, hipStream_t s) {
  if (ts == 16) hipLaunchKernelGGL((gemm_f32_kernel<EPI, ACT, 16, KSTEP[1], GA>), grid, dim3(256), 0, s, p, ga);
  else if (ts == 32) hipLaunchKernelGGL((gemm_f32_kernel<EPI, ACT, 32, KSTEP[2], GA>), grid, dim3(256), 0, s, p, ga);
  else hipLaunchKernelGGL((gemm_f32_kernel<EPI, ACT, 64, KSTEP[4], GA>), grid, dim3(256), 0, s, p, ga);
  return hipGetLastError();
}

template <int EPI, int ACT>
hipError_t launch1(const GemmP &p, hipStream_t s) {
  const int ks = (EPI == EPI_WGRAD && p.ksplit > 1) ? p.ksplit : 1;
  if ((p.a_trans != 0) != (EPI == EPI_WGRAD) || (p.b_trans != 0) != (EPI == EPI_WGRAD || EPI == EPI_BWD)) return hipErrorInvalidValue;
  if (p.head.y && (EPI != EPI_LOGITS || !gemm_head_fits(0, p.Md, p.Nd, p.groups) || !p.head.idx || p.head.N < 1 || !p.head.D ||
                   !p.head.dn || !p.head.loss || p.head.ldd < p.Nd || p.head.ldd > 16))
    return hipErrorInvalidValue;
  if (p.rowsum && (EPI != EPI_WGRAD || ks > 1)) return hipErrorInvalidValue;
  if (ks > 1 && (!p.kpart || p.kchunk <= 0 || (p.kchunk & 31) || (long long)p.kchunk * ks < p.Kd)) return hipErrorInvalidValue;
  const int ts = EPI == EPI_WGRAD && p.f32_tile ? p.f32_tile : tile_size(p.Md, p.Nd, (long long)p.groups * ks);
  if (ts != 16 && ts != 32 && ts != 64) return hipErrorInvalidValue;
  dim3 grid((p.Nd + ts - 1) / ts, (p.Md + ts - 1) / ts, p.groups * ks);
  if (grid.y > 65535 || grid.z > 65535) return hipErrorInvalidValue;
  if constexpr (EPI == EPI_FWD_ACT || EPI == EPI_LOGITS) {
    if (p.gather) {                             // (one variant: the gather rides with the launch that reads the dataset)
      if (!p.aidx || p.aN < 1 || p.aldi < p.Md || p.sAg || !gather_ok(*p.gather)) return hipErrorInvalidValue;
      grid.z += (unsigned)((gather_blocks(*p.gather) + grid.x * grid.y - 1) / (grid.x * grid.y));
      return launch2<EPI, ACT, true>(p, *p.gather, ts, grid, s);
    }
  }
  if (p.gather || p.aidx) return hipErrorInvalidValue;
  return launch2<EPI, ACT, false>(p, GatherP{}, ts, grid, s);
}
template <int EPI>
hipError_t launch_act(const GemmP &p, hipStream_t s) {
  if constexpr (EPI == EPI_FWD_ACT || EPI == EPI_BWD) {
    if (p.act == ACT_RELU) return launch1<EPI, ACT_RELU>(p, s);
    if (p.act == ACT_GELU) return launch1<EPI, ACT_GELU>(p, s);
  }
  if constexpr (EPI == EPI_WGRAD) {
    if (!p.upd_x) return launch1<EPI, NO_STEP>(p, s);
    if (p.ksplit > 1 || p.accumulate || !p.upd_sq || (p.upd_opt != OPT_SGD && !p.upd_v) || (p.upd_opt == OPT_ADAMW && !p.upd_m))
      return hipErrorInvalidValue;
    switch (p.upd_opt) {
      case OPT_SGD: return launch1<EPI, OPT_SGD>(p, s);
      case OPT_SHB: return launch1<EPI, OPT_SHB>(p, s);
      case OPT_ADAMW: return launch1<EPI, OPT_ADAMW>(p, s);
      case OPT_ADAGRAD: return launch1<EPI, OPT_ADAGRAD>(p, s);
      default: return hipErrorInvalidValue;
    }
  } else {
    return launch1<EPI, ACT_NONE>(p, s);
  }
}

}  // namespace

int gemm_f32_upd_slots(int Md, int Nd, int tile) { return ((Nd + tile - 1) / tile) * ((Md + tile - 1) / tile); }

// Tile and number of slices of a weight gradient's reduction over Kd samples.  Up to 256 samples (one k-step of the smallest
// tile) the tile follows from the number of outputs alone and nothing is split.  Beyond, the pair of least modelled time, in
// microseconds per 256 samples walked by a block with n blocks on its CU, measured on 64 x 12 to 1024 x 256 outputs of 1 to 16
// replicas, b = 512 to 8192 (alone; 2, 4 and more blocks to a CU):
//   64 x 64 tiles 14; 17, 30   32 x 32 tiles 7.0; 8.4, 14 (16: 51)   16 x 16 tiles 3.5; 3.9, 5.6 (7: 9.9, 32: 43)
// A split adds its finish, the column sums of the bias gradient and the separate optimizer step: about 12 us and the traffic.
// The tile that is launched decides, not the smallest one: 100 x 1024 outputs of 4 replicas, b = 8192, are 128 tiles of
// 64 x 64, un-split 436 us on half of the CUs, 121 in eight slices (step 758 -> 339 us; 256 x 100,
// 16 replicas: 766 -> 358); 1024-256-100, 8 replicas, a step at b = 2048 437 -> 417, at b = 8192 1515 -> 1376.
F32WgradPlan gemm_f32_wgrad_plan(int Md, int Nd, int Kd, int groups, size_t kpart_floats) {
  F32WgradPlan best = {tile_size(Md, Nd, groups), 1};
  if (Kd <= 256) return best;
  const double outputs = (double)Md * Nd * groups, split_bytes = 4.0 * groups * Kd * Md;
  const int KT = (Kd + 255) / 256;
  double best_cost = 0.0;
  for (int i = 1; i <= 4; i *= 2)
    for (int S = 1; S <= F32_MAX_SPLIT && S <= KT; ++S) {
      const int tile = 16 * i;
      const long long blocks = (long long)gemm_f32_upd_slots(Md, Nd, tile) * groups * S;
      if (S > 1 && (((long long)Md * Nd & 3) || blocks > F32_MAX_SPLIT_BLOCKS || S * outputs > (double)kpart_floats)) break;
      const int len = std::min(Kd, (KT + S - 1) / S * 256), step = KSTEP[i];
      const double n = (double)((blocks + 255) / 256);
      const double t = i == 4 ? std::max(14.0, 2.0 + 7.2 * n) : i == 2 ? std::max(7.0, 1.0 + 3.2 * n) : std::max(3.5, 1.35 * n);
      double cost = (len + step - 1) / step * (step / 256.0) * t;
      if (S > 1) cost += 12.0 + (8.0 * S * outputs + split_bytes) / 4.5e6;
      if (best_cost == 0.0 || cost < best_cost) { best.tile = tile; best.ksplit = S; best_cost = cost; }
    }
  return best;
}

size_t gemm_f32_kpart_floats(int Md, int Nd, int groups) {
  if ((long long)Md * Nd & 3) return 0;
  return std::min((size_t)F32_MAX_SPLIT * groups * Md * Nd, (size_t)F32_MAX_SPLIT_BLOCKS * 64 * 64);
}

hipError_t launch_gemm_f32(const GemmP &p, int epi, hipStream_t s) {
  if (p.Md <= 0 || p.Nd <= 0 || p.groups <= 0) return hipSuccess;
  switch (epi) {
    case EPI_FWD_ACT: return launch_act<EPI_FWD_ACT>(p, s);
    case EPI_LOGITS: return launch_act<EPI_LOGITS>(p, s);
    case EPI_BWD: return launch_act<EPI_BWD>(p, s);
    case EPI_WGRAD: return launch_act<EPI_WGRAD>(p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace absk
