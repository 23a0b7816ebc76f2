// The whole fp32 step of a net without hidden layers (logistic regression, up to 16 classes) in one launch: gather, logits,
// softmax head, batch gradient, optimizer step and statistics.
//
// What bounds such a step is the chain of its launches, not bytes or flops: 256 features, 10 classes and 16 samples are 16 KB of
// rows and 10 KB of weights per replica, and three launches (logits with the head, weight gradient with the step, statistics) of 5
// to 8 us each, or four beyond 256 samples, whose sums are two.  Here a work-group of sixteen wavefronts takes CH samples of a
// replica; their rows pass through LDS once and serve the logits and the gradient, both on 16x16x4 fp32 MFMAs (fp32 products and sums
// throughout).  Replicas of several work-groups leave partial gradients; the last one of them to arrive adds these in order of the
// chunks, takes the step and delivers the sums.  The partials are written and read past the XCDs' L2 (agent scope), so that the
// hand-over needs no cache write-back: a counter per replica, no waiting, and the last work-group puts it back to zero.
// Inner products <g_i, gbar> follow in the same launch where a replica is one work-group, else in a second one.
// 256 features, 10 classes, 4 replicas, us per step with test and rule: b = 16 28.7 -> 15.8, b = 512 36.5 -> 22.6.  What is left of the
// launch at b = 16 (6.0 us inside; at b = 512 12.6): rows 1.8 (3.4), logits 0.6 (1.2), head 0.7 (1.0), gradient and step 1.1 (1.7; the
// hand-over 1.4 and the sum over the chunks 2.5 behind it), sums and their way to the host 1.8; around it 8 us of launch and host.
#include <algorithm>
#include <mutex>
#include "abs_internal.h"
#include "device_utils.h"

namespace absk {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 1024, NW = NT / 64;
constexpr int FRAG = 8;                          // 16-byte pieces per lane of a row slice, and of an operand slice
constexpr int KC = 16;                           // classes
constexpr int KLD = KC + 4;                      // row stride of signals and partial logits in LDS: rows 4 q apart lie 16 banks apart
constexpr int LDS_MAX = 160 * 1024 - 512;        // (beside the static part)

// LDS of a work-group, in floats: rows [CH][LDX], partial logits [KS][CH][KLD], signals [CH][KLD], per-sample scalars, signals summed over each four samples
__host__ __device__ constexpr int row_ld(int d) { return (d + 15) / 16 * 16 + 4; }
constexpr size_t lds_floats(int ch, int d) { return (size_t)ch * row_ld(d) + NW * KC * KLD + (size_t)ch * KLD + 4 * ch + ch / 4 * KC; }
static_assert(lds_floats(64, 512) * 4 <= LDS_MAX && lds_floats(32, 1024) * 4 <= LDS_MAX && lds_floats(16, 2048) * 4 <= LDS_MAX, "LDS budget");

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
// barrier for what passes through LDS alone: global stores stay in flight
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) { return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false)); }
// sum over a wavefront, in its last lane (row shifts and broadcasts on DPP: no trip through LDS)
__device__ __forceinline__ float wave_sum_last(float v) {
  v = dpp_add<0x111, 0xf>(v); v = dpp_add<0x112, 0xf>(v); v = dpp_add<0x114, 0xf>(v); v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}
// and over each sixteen lanes, in all of them
__device__ __forceinline__ float sum16(float v) {
  v += dpp<0x121>(v); v += dpp<0x122>(v); v += dpp<0x124>(v);      // row_ror: 1, 2, 4, 8
  return v + dpp<0x128>(v);
}
__device__ __forceinline__ float max16(float v) {
  v = fmaxf(v, dpp<0x121>(v)); v = fmaxf(v, dpp<0x122>(v)); v = fmaxf(v, dpp<0x124>(v));
  return fmaxf(v, dpp<0x128>(v));
}

// rows s0 .. s0 + ns - 1 of group g to LDS, zeros beyond them and beyond d, and their squared norms.  A wavefront takes rows
// wave + 16 j; all loads of its rows are in flight together.
template <int CH, bool VEC>
__device__ __forceinline__ void load_rows(const SoftmaxStepP &p, int g, int s0, int ns, float *xs, float *an) {
  constexpr int ST = CH / 16, J = FRAG / ST;
  const int lane = threadIdx.x & 63, wave = wave_id(), d = p.d, ld = row_ld(d), dp = ld - 4;
  const float *src[ST];
#pragma unroll
  for (int i = 0; i < ST; ++i) {
    const int id = p.idx[(long long)g * p.ldi + s0 + min(wave + 16 * i, ns - 1)];
    src[i] = p.X + (long long)min(max(id, 0), p.N - 1) * d;
  }
  f32x4 v[ST][J];
#pragma unroll
  for (int i = 0; i < ST; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) {
      v[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (256 * j >= d) continue;                // uniform
      if constexpr (VEC) {                       // (addresses inside the row; what lies beyond it becomes zero below)
        v[i][j] = *reinterpret_cast<const f32x4 *>(src[i] + min(4 * lane + 256 * j, d - 4));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][j][e] = src[i][min(lane + 64 * (4 * j + e), d - 1)];
      }
    }
#pragma unroll
  for (int i = 0; i < ST; ++i) {
    const int row = wave + 16 * i;
    const bool live = row < ns;
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = VEC ? 4 * lane + 256 * j : lane + 64 * (4 * j + e);
        v[i][j][e] = live && c < d ? v[i][j][e] : 0.0f;
        s = fmaf(v[i][j][e], v[i][j][e], s);
      }
      if constexpr (VEC) {
        const int c = 4 * lane + 256 * j;
        if (c < dp) *reinterpret_cast<f32x4 *>(xs + row * ld + c) = v[i][j];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = lane + 64 * (4 * j + e);
          if (c < dp) xs[row * ld + c] = v[i][j][e];
        }
      }
    }
    s = wave_sum_last(s);
    if (lane == 63) an[row] = s;
  }
}

// A wavefront's slice of the operand rows B[class][k] (memory [K][d]): steps ks, ks + KS, ... of 16 k; lane l holds class l % 16
// and four k from 4 (l / 16), one per MFMA
template <int CH, bool VEC>
__device__ __forceinline__ void load_classes(const float *B, int K, int d, f32x4 (&b)[FRAG]) {
  constexpr int ST = CH / 16, KS = NW / ST;
  const int lane = threadIdx.x & 63, ks = wave_id() / ST, c = lane & 15, q = lane >> 4;
  const float *row = B + (long long)min(c, K - 1) * d;
#pragma unroll
  for (int u = 0; u < FRAG; ++u) {
    b[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if ((ks + u * KS) * 16 >= d) continue;       // uniform
    const int k = (ks + u * KS) * 16 + 4 * q;
    if constexpr (VEC) {
      const f32x4 w = *reinterpret_cast<const f32x4 *>(row + min(k, d - 4));
      b[u] = c < K && k < d ? w : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w = row[min(k + e, d - 1)];
        b[u][e] = c < K && k + e < d ? w : 0.0f;
      }
    }
  }
}
// partial products of this wavefront's sample tile and k-slice: zred[ks][sample][class]
template <int CH>
__device__ __forceinline__ void contract(const float *xs, int d, const f32x4 (&b)[FRAG], float *zred) {
  constexpr int ST = CH / 16, KS = NW / ST;
  const int lane = threadIdx.x & 63, wave = wave_id(), st = wave % ST, ks = wave / ST, ld = row_ld(d);
  const int r = lane & 15, q = lane >> 4, steps = (ld - 4) / 16;
  const float *row = xs + (st * 16 + r) * ld + 4 * q;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int u = 0; u < FRAG; ++u) {
    const int s = ks + u * KS;
    if (s < steps) {                             // uniform
      const f32x4 a = *reinterpret_cast<const f32x4 *>(row + s * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[u][e], acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) zred[(ks * CH + st * 16 + 4 * q + e) * KLD + r] = acc[e];
}
// of sample t / 16, class t % 16
template <int CH>
__device__ __forceinline__ float contracted(const float *zred) {
  constexpr int KS = NW / (CH / 16);
  float z = 0.0f;
#pragma unroll
  for (int k = 0; k < KS; ++k) z += zred[(k * CH + (threadIdx.x >> 4)) * KLD + (threadIdx.x & 15)];
  return z;
}
// memory that work-groups on other XCDs write or read in the same launch
__device__ __forceinline__ void put(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float get(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double get(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Whether this work-group is the last of its group's n to come here, after all its puts; the last one leaves the counter at zero.
__device__ __forceinline__ bool last_of(int *count, int n, int *flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wavefront's puts have arrived
  __syncthreads();
  if (threadIdx.x == 0) {
    const int before = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before == n - 1) __hip_atomic_store(count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = before == n - 1;
  }
  __syncthreads();
  return *flag != 0;
}

// sums of group g, in its slots of the statistics and of their mirror, then the ticket; by one wavefront, sum k in lane k < 5 (sel:
// those that exist).  The host reads nothing but the mirror, so that its stores and their arrival are all that the ticket waits for.
__device__ __forceinline__ void deliver(const SoftmaxStepP &p, int g, int sel, double v) {
  const int t = threadIdx.x & 63;
  double *const host = p.stats_host + g * 8;
  if (t < 5 && ((sel >> t) & 1)) {
    if (p.stats_host) __hip_atomic_store(host + t, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (t == 0 && p.stats_host) __hip_atomic_store(host + 7, p.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (t < 5 && ((sel >> t) & 1)) p.stats[g * 8 + t] = v;
}

template <int OPT>
__device__ __forceinline__ void load_param(const SoftmaxStepP &p, long long o, float &x, float &v, float &m) {
  x = p.upd_x[o]; v = OPT != OPT_SGD ? p.upd_v[o] : 0.0f; m = OPT == OPT_ADAMW ? p.upd_m[o] : 0.0f;
}
template <int OPT>
__device__ __forceinline__ void step_at(const SoftmaxStepP &p, const OptHyper &h, long long o, float gr, float x, float v, float m, double &sq) {
  p.grad[o] = gr;
  opt_step_elem<OPT>(x, gr, v, m, h);
  p.upd_x[o] = x;
  if (OPT != OPT_SGD) p.upd_v[o] = v;
  if (OPT == OPT_ADAMW) p.upd_m[o] = m;
  sq += (double)(gr * gr);
}

// OPT < 0: the second launch of a step with inner products over several chunks: rows, signals and the finished gradient -> q
template <int OPT, int CH, bool VEC>
__global__ void __launch_bounds__(NT) softmax_step_kernel(const SoftmaxStepP p) {
  constexpr int ST = CH / 16;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int d = p.d, K = p.K, ld = row_ld(d);
  float *const xs = lds, *const zred = xs + CH * ld, *const dl = zred + NW * KC * KLD, *const an = dl + CH * KLD, *const sn = an + CH,
              *const sl = sn + CH, *const sq_ = sl + CH, *const bs = sq_ + CH;
  __shared__ double fin[NW];
  __shared__ int flag;
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int bg = p.rows ? p.rows[g] : p.b, chunks = (bg + CH - 1) / CH, s0 = blockIdx.x * CH;
  constexpr bool IP_ONLY = OPT < 0;
  if (s0 >= bg || (IP_ONLY && chunks == 1)) return;        // uniform over the block (one chunk: the first launch has delivered)
  const int ns = min(CH, bg - s0);
  const float alpha = p.rows ? 1.0f / (float)bg : p.alpha;
  const long long base = (long long)g * p.sPg;
  constexpr int O = OPT < 0 ? 0 : OPT;
  const int smp = tid >> 4, cls = tid & 15;      // (head: a lane per sample and class)
  const bool mine = smp < ns;

  f32x4 bf[FRAG];
  load_classes<CH, VEC>((IP_ONLY ? p.grad : p.upd_x) + base, K, d, bf);
  const float bias = p.has_bias && cls < K ? (IP_ONLY ? p.grad : p.upd_x)[base + p.offB + cls] : 0.0f;
  int label = 0;
  float delta = 0.0f;
  if (mine) {
    if constexpr (IP_ONLY) delta = cls < K ? p.D[(long long)g * p.sDg + (long long)(s0 + smp) * p.ldd + cls] : 0.0f;
    else {
      const int id = p.idx[(long long)g * p.ldi + s0 + smp];
      label = min(max(p.y[min(max(id, 0), p.N - 1)], 0), K - 1);
    }
  }
  // one chunk: the parameters of this wavefront's first gradient tile, and its bias, on their way from the start
  const int r = lane & 15, q = lane >> 4;
  const bool one = chunks == 1;
  float x[4], v[4], m[4], xb, vb, mb;
  auto load_tile = [&](int col) {
#pragma unroll
    for (int e = 0; e < 4; ++e) load_param<O>(p, base + (long long)min(4 * q + e, K - 1) * d + min(col, d - 1), x[e], v[e], m[e]);
  };
  if (!IP_ONLY && one) {
    load_tile(wave * 16 + r);
    if (p.has_bias) load_param<O>(p, base + p.offB + min(lane, K - 1), xb, vb, mb);
  }
  load_rows<CH, VEC>(p, g, s0, ns, xs, an);
  lds_barrier();
  contract<CH>(xs, d, bf, zred);
  lds_barrier();

  double *const csum = p.csums + ((long long)g * p.chunks + blockIdx.x) * 4;      // this chunk's n, loss, q, q^2
  auto inner_products = [&](float u) {           // u: this lane's (Gbar a_i + gbias)_c
    const float q = sum16(delta * u);
    if (mine && cls == 0) {
      sq_[smp] = q;
      if (p.q_out) p.q_out[(long long)g * p.sNg + s0 + smp] = q;
    }
    __syncthreads();
  };

  if constexpr (!IP_ONLY) {
    if (smp < CH) {                              // uniform over a wavefront: softmax cross-entropy
      const float z = cls < K ? contracted<CH>(zred) + bias : -INFINITY;
      const float mx = max16(z);
      const float ex = cls < K ? expf(z - mx) : 0.0f;
      const float se = sum16(ex);
      delta = cls < K ? ex * (1.0f / se) - (cls == label ? 1.0f : 0.0f) : 0.0f;
      if (!mine) delta = 0.0f;
      dl[smp * KLD + cls] = delta;
      const float dn = sum16(delta * delta);
      float four = delta + __shfl_xor(delta, 16, 64);
      four += __shfl_xor(four, 32, 64);
      if (lane < KC) bs[wave * KC + lane] = four;
      if (mine) {
        if (cls == label) sl[smp] = -(z - mx - logf(se));
        if (cls == 0) {
          const float n = dn * (an[smp] + (p.has_bias ? 1.0f : 0.0f));
          sn[smp] = n;
          if (p.n_out) p.n_out[(long long)g * p.sNg + s0 + smp] = n;
        }
        if (p.do_q && chunks > 1 && cls < p.ldd) p.D[(long long)g * p.sDg + (long long)(s0 + smp) * p.ldd + cls] = delta;
      }
    }
    lds_barrier();

    // batch gradient: 16 classes x 16 features per MFMA tile, samples four at a time
    const int tiles = (ld - 4) / 16;
    float *const part = p.part + ((long long)g * p.chunks + blockIdx.x) * p.part_ld;
    OptHyper h = {p.lr, p.momentum, p.beta1, p.beta2, p.eps, p.wd, p.c1, p.c2};
    if (p.scal) { h.lr = p.scal[0]; h.c1 = p.scal[1]; h.c2 = p.scal[2]; }
    double sq = 0.0;
    for (int t = wave; t < tiles; t += NW) {
      const int col = t * 16 + r;
      auto at = [&](int e) -> long long { return base + (long long)(4 * q + e) * d + col; };
      if (one && t > wave) load_tile(col);       // (the first one's are here)
      f32x4 acc[4];                              // four chains: sums of CH / 4 products
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < CH / 4; ++s) {         // four lane groups on rows four apart: sixteen banks each
        const int row = (s >> 2) * 16 + 4 * q + (s & 3);
        acc[s & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(dl[row * KLD + r], xs[row * ld + col], acc[s & 3], 0, 0, 0);
      }
      acc[0] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
      if (col < d) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = 4 * q + e;
          if (c >= K) continue;
          if (one) step_at<O>(p, h, at(e), acc[0][e] * alpha, x[e], v[e], m[e], sq);
          else put(part + (long long)c * d + col, acc[0][e]);
        }
      }
    }
    if (p.has_bias && wave == NW - 2 && lane < K) {
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k < CH / 4; ++k) s += bs[k * KC + lane];
      if (one) step_at<O>(p, h, base + p.offB + lane, s * alpha, xb, vb, mb, sq);
      else put(part + (long long)K * d + lane, s);
    }
    double s1 = 0.0, loss = 0.0;                 // (the last wavefront has the fewest tiles)
    if (wave == NW - 1) {
      s1 = wave_sum(lane < ns ? (double)sn[lane] : 0.0);
      loss = wave_sum(lane < ns ? (double)sl[lane] : 0.0);
      if (!one && lane == 0) { put(csum, s1); put(csum + 1, loss); }
    }
    if (!one) {
      if (!last_of(p.count + 16 * g, chunks, &flag)) return;
      const float *parts = p.part + (long long)g * p.chunks * p.part_ld;
      const int n = K * d + (p.has_bias ? K : 0);
      constexpr int U = 4, C = 8;                // parameters to a thread, and chunks, in flight together
      auto where = [&](int i) -> long long { return base + (i < K * d ? i : p.offB + i - K * d); };
      for (int i0 = tid; i0 < n; i0 += U * NT) {
        float s[U], x[U], v[U], m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          s[u] = 0.0f;
          if (i0 + u * NT < n) load_param<O>(p, where(i0 + u * NT), x[u], v[u], m[u]);
        }
        for (int c0 = 0; c0 < chunks; c0 += C) {
          float w[C][U];
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int u = 0; u < U; ++u) w[c][u] = get(parts + (long long)min(c0 + c, chunks - 1) * p.part_ld + min(i0 + u * NT, n - 1));
#pragma unroll
          for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int c = 0; c < C; ++c) if (c0 + c >= chunks) w[c][u] = 0.0f;
            s[u] += ((w[0][u] + w[1][u]) + (w[2][u] + w[3][u])) + ((w[4][u] + w[5][u]) + (w[6][u] + w[7][u]));
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + u * NT < n) step_at<O>(p, h, where(i0 + u * NT), s[u] * alpha, x[u], v[u], m[u], sq);
      }
      if (wave == NW - 1) {
        const double *cs = p.csums + (long long)g * p.chunks * 4;
        s1 = loss = 0.0;
        for (int c = lane; c < chunks; c += 64) { s1 += get(cs + 4 * c); loss += get(cs + 4 * c + 1); }
        s1 = wave_sum(s1); loss = wave_sum(loss);
      }
    }
    const double w = wave_sum(sq);
    if (lane == 0) fin[wave] = w;
    const bool finish_q = p.do_q && one;
    lds_barrier();
    if (finish_q) {
      __syncthreads();                           // the gradient is visible to the whole work-group
      load_classes<CH, VEC>(p.grad + base, K, d, bf);
      const float gb = p.has_bias && cls < K ? p.grad[base + p.offB + cls] : 0.0f;
      contract<CH>(xs, d, bf, zred);
      __syncthreads();
      inner_products(smp < CH && cls < K ? contracted<CH>(zred) + gb : 0.0f);
    }
    if (wave == NW - 1) {
      double q1 = 0.0, q2 = 0.0, s2 = 0.0;
      if (finish_q) {
        const double qv = lane < ns ? (double)sq_[lane] : 0.0;
        q1 = wave_sum(qv); q2 = wave_sum(qv * qv);
      }
#pragma unroll
      for (int k = 0; k < NW; ++k) s2 += fin[k];
      const double v = lane == 0 ? s1 : lane == 1 ? s2 : lane == 2 ? q2 : lane == 3 ? q1 : loss;
      if (p.do_q && !one) {                      // (delivered with the inner products)
        const int sel = 1 | 2 | 16;
        if (lane < 5 && ((sel >> lane) & 1)) p.stats[g * 8 + lane] = v;
        return;
      }
      deliver(p, g, p.do_q ? 31 : 1 | 2 | 16, v);
    }
  } else {
    inner_products(smp < CH && cls < K ? contracted<CH>(zred) + bias : 0.0f);
    double q1 = 0.0, q2 = 0.0;
    if (wave == NW - 1) {
      const double qv = lane < ns ? (double)sq_[lane] : 0.0;
      q1 = wave_sum(qv); q2 = wave_sum(qv * qv);
      if (lane == 0) { put(csum + 2, q1); put(csum + 3, q2); }
    }
    if (!last_of(p.count + 16 * g, chunks, &flag)) return;
    if (wave == NW - 1) {
      const double *cs = p.csums + (long long)g * p.chunks * 4;
      q1 = q2 = 0.0;
      for (int c = lane; c < chunks; c += 64) { q1 += get(cs + 4 * c + 2); q2 += get(cs + 4 * c + 3); }
      q1 = wave_sum(q1); q2 = wave_sum(q2);
      const double v = lane == 2 ? q2 : lane == 3 ? q1 : lane < 5 ? p.stats[g * 8 + lane] : 0.0;
      deliver(p, g, 31, v);
    }
  }
}

// Samples to a work-group: the whole batch while one can hold it, else 32: 64 make the loads of the rows longer, 16 the sum over the
// chunks.  us per step, 64 -> 32 -> 16: 256-10, 4 replicas, b = 512 23.2 -> 23.0 -> 24.9; 512-2, 4, b = 100 27.1 -> 23.0; 256-16, 16,
// b = 512 27.7 (32) -> 38.2; 512-10, 8, b = 512 29.2 (32) -> 34.0.  Long rows in a few chunks are still faster in 16: 784-16, 4
// replicas, b = 100 41.2 -> 36.1; 1024-16, 8, b = 100 51.4 -> 44.8; 512-10, 4, b = 100 25.9 -> 24.2.  (Beyond 1024 features 16 is what fits.)
// Up to 128 of them, since the sum takes eight chunks at a time: 512, 640, 784 and 1024 features, 1 to 16 replicas, 32 -> 16: b = 65 6 to 14 %
// faster, b = 128 6 to 13 % (784-10, 8 replicas 24.8 -> 22.1 and 25.3 -> 22.7), b = 129 1 % faster to 6 % slower (25.0 -> 25.0; 1024-16, 16
// replicas 32.6 -> 34.5).
int chunk_of(int d, int b) {
  if (b <= 16 || d > 1024 || (d >= 512 && b > 64 && b <= 128)) return 16;
  return b > 32 && b <= 64 && d <= 512 ? 64 : 32;
}

template <int OPT, int CH, bool VEC>
hipError_t launch2(const SoftmaxStepP &p, hipStream_t s) {
  auto kern = softmax_step_kernel<OPT, CH, VEC>;
  static std::once_flag attr_once;               // once per variant, whatever thread launches it first
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MAX);
  });
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL(kern, dim3(p.chunks, p.groups), dim3(NT), lds_floats(CH, p.d) * sizeof(float), s, p);
  return hipGetLastError();
}
template <int OPT>
hipError_t launch1(const SoftmaxStepP &p, hipStream_t s) {
  const bool vec = (p.d & 3) == 0;
  switch (chunk_of(p.d, p.b)) {
    case 64: return vec ? launch2<OPT, 64, true>(p, s) : launch2<OPT, 64, false>(p, s);
    case 32: return vec ? launch2<OPT, 32, true>(p, s) : launch2<OPT, 32, false>(p, s);
    default: return vec ? launch2<OPT, 16, true>(p, s) : launch2<OPT, 16, false>(p, s);
  }
}

}  // namespace

int softmax_step_chunks(int d, int b) { return (b + chunk_of(d, b) - 1) / chunk_of(d, b); }

// Up to 32 chunks and 2 MB of partial gradients to a replica.  us per step, general launches -> one: 256-10, 4 replicas, b = 16 28.7 ->
// 15.8, b = 512 36.5 -> 23.0; 64-2, 1 replica, b = 257 32.5 -> 19.6; 256-2, 16, b = 1024 65.9 -> 34.7; 1024-10, 16, b = 512 110 -> 41;
// with inner products 784-10, 16, b = 1024 165 -> 87, 1024-16, 4, b = 512 58.9 -> 53.5, 1024-16, 1, b = 512 56.0 -> 55.4.  At the line
// both cost the same: 1024-16, 16, b = 1024 134 and 137.
// Time of a step against the general launches, 1060 nets of 1 to 2048 features, 1 to 600 replicas, b = 2 to 1024:
//   one work-group to a replica 0.17 to 0.99, on average 0.62 (many replicas of few features: softmax_step_taken);
//   several, up to 768 in all 0.35 to 0.99, with 256 and more features 0.36 to 1.01 up to 2048: beyond, waves of work-groups come one after
//     the other for few products each (23-6, 540 replicas, b = 588 273 -> 552 us; 1210-11, 307, b = 467 955 -> 1333);
//   except that with fewer than 8 replicas the last work-group of each adds the partial gradients while other CUs idle: beyond 320 k floats of
//     them, and beyond 8192 parameters where rows are not whole 16-byte pieces, 0.74 to 1.28 (1511-16, 1 replica, b = 199 38.8 -> 49.8).
bool softmax_step_fits(int K, int d, int b, int groups) {
  if (K > KC || d > 2048) return false;
  const int chunks = softmax_step_chunks(d, b);
  const long long parts = (long long)chunks * softmax_step_part_floats(K, d);
  if (chunks > SOFTMAX_STEP_CHUNKS || parts > SOFTMAX_STEP_PARTS) return false;
  if (chunks == 1) return true;
  if ((long long)chunks * groups > (d < 256 ? 768 : 2048)) return false;
  return groups >= 8 || (d & 3 ? K * d <= 8192 : parts <= 320 * 1024);
}

// Many replicas of one work-group each come one round of CUs after the other, each with a way to the host of its own sums at its end, which the
// general launches have once.  Step and test, 80 nets of 1 to 1038 features, 62 to 1420 replicas, b = 2 to 62, without inner products: from
// 96 features 0.41 to 0.92 of the time; less of them with up to 384 replicas 0.63 to 1.03, with 385 to 620 0.92 to 1.10, beyond 1.01 to 1.13
// (7-14, 743 replicas, b = 10 96.6 -> 108.7 us; steps without a test 46.8 -> 44).  With inner products, four to five general launches, 0.73 at most.
bool softmax_step_taken(int K, int d, int b, int groups, int ip) {
  return softmax_step_fits(K, d, b, groups) && (ip || d >= 96 || groups <= 384);
}

int softmax_step_max_chunks(int K, int d, int cap, int groups) {
  int most = 0;
  for (int b = 2; b <= std::min(cap, 64 * SOFTMAX_STEP_CHUNKS); ++b)            // (no chunk is longer than 64)
    if (softmax_step_fits(K, d, b, groups)) most = std::max(most, softmax_step_chunks(d, b));
  return most;
}

hipError_t launch_softmax_step(SoftmaxStepP p, hipStream_t s) {
  if (!softmax_step_fits(p.K, p.d, p.b, p.groups) || p.K < 2 || p.d < 1 || p.b < 1 || p.groups < 1 || p.groups > 65535 || p.N < 1 || p.ldi < p.b ||
      !p.X || !p.y || !p.idx || !p.upd_x || !p.grad || !p.stats || (p.opt != OPT_SGD && !p.upd_v) || (p.opt == OPT_ADAMW && !p.upd_m) ||
      (reinterpret_cast<uintptr_t>(p.X) & 15) || (reinterpret_cast<uintptr_t>(p.upd_x) & 15) || (reinterpret_cast<uintptr_t>(p.grad) & 15) ||
      (p.sPg & 3) || p.ldd < p.K)
    return hipErrorInvalidValue;
  p.chunks = softmax_step_chunks(p.d, p.b);
  p.part_ld = softmax_step_part_floats(p.K, p.d);
  if (p.chunks > 1 && (p.chunks > p.max_chunks || !p.part || !p.csums || !p.count || (p.do_q && !p.D))) return hipErrorInvalidValue;
  hipError_t e;
  switch (p.opt) {
    case OPT_SGD: e = launch1<OPT_SGD>(p, s); break;
    case OPT_SHB: e = launch1<OPT_SHB>(p, s); break;
    case OPT_ADAMW: e = launch1<OPT_ADAMW>(p, s); break;
    case OPT_ADAGRAD: e = launch1<OPT_ADAGRAD>(p, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e == hipSuccess && p.do_q && p.chunks > 1) e = launch1<-1>(p, s);
  return e;
}

}  // namespace absk
