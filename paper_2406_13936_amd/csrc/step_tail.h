// Device code of the end of a step that more than one kernel runs: the bias gradients with their optimizer step and the
// per-sample part of the statistics, as launches of their own (elementwise.hip) or in front of a weight-gradient launch.
#pragma once
#include "device_utils.h"

namespace absk {
namespace {

// Block bx of the nx that share the columns of layer l, group g (p.cb columns each): 256 threads, red: 256 floats, 8-byte aligned.
template <int OPT>
__device__ __forceinline__ void col_finish_block(const ColFinishMany &p, int bx, int nx, int l, int g, float *red) {
  const int cols = p.cols[l];
  const bf16_t *src = p.src[l];
  // columns x row-lanes at a time: 64 x 4; 256 x 1 over few partials; 16 x 16 for a narrow layer summed directly (a shorter
  // serial walk per lane)
  const int CL = src ? (cols <= 16 ? 16 : 64) : p.cb, RL = 256 / CL;
  const int cl = threadIdx.x & (CL - 1), rl = threadIdx.x / CL;
  double gg = 0.0;
  for (int c0 = bx * p.cb; c0 < cols && c0 < (bx + 1) * p.cb; c0 += CL) {       // uniform over the block
    const int c = c0 + cl;
    float alpha = p.alpha;
    int ns = src ? p.b : p.nsplit[l];
    if (p.rows) {
      alpha = 1.0f / (float)p.rows[g];
      if (src) ns = p.rows[g];
      else if (p.tile_m[l] > 0) ns = (p.rows[g] + p.tile_m[l] - 1) / p.tile_m[l] * p.parts_per_tile[l];
    }
    float s = 0.0f;
    if (c < cols) {
      if (src) {                                   // (a long chain of additions: in double)
        const bf16_t *q = src + (long long)g * p.sXg[l] + c;
        double s64 = 0.0;
#pragma unroll 8
        for (int r = rl; r < ns; r += RL) s64 += (double)bf2f(q[(long long)r * p.ldx[l]]);
        s = (float)s64;
      } else {
        const float *q = p.part[l] + (long long)g * p.nsplit[l] * cols + c;
#pragma unroll 4
        for (int r = rl; r < ns; r += RL) s += q[(long long)r * cols];
      }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (rl == 0 && c < cols) {
      float t = red[cl];
      for (int k = 1; k < RL; ++k) t += red[k * CL + cl];
      const long long off = (long long)g * p.sOg + p.out_off[l] + c;
      float *o = p.out + off;
      const float gr = p.accumulate ? fmaf(alpha, t, *o) : alpha * t;
      *o = gr;
      if constexpr (OPT >= 0) {
        OptHyper h = {p.upd_lr, p.upd_momentum, p.upd_beta1, p.upd_beta2, p.upd_eps, p.upd_wd, p.upd_c1, p.upd_c2};
        if (p.upd_scal) { h.lr = p.upd_scal[0]; h.c1 = p.upd_scal[1]; h.c2 = p.upd_scal[2]; }
        float x = p.upd_x[off], v = OPT != OPT_SGD ? p.upd_v[off] : 0.0f, m = OPT == OPT_ADAMW ? p.upd_m[off] : 0.0f;
        opt_step_elem<OPT>(x, gr, v, m, h);
        p.upd_x[off] = x;
        if (OPT != OPT_SGD) p.upd_v[off] = v;
        if (OPT == OPT_ADAMW) p.upd_m[off] = m;
        if (p.upd_shadow) p.upd_shadow[off] = f2bf(x);
        gg += (double)(gr * gr);
      }
    }
    __syncthreads();                               // red is free again
  }
  if constexpr (OPT >= 0) {                        // blocks beyond the layer leave zeros
    const double r = block_sum<4>(gg, reinterpret_cast<double *>(red));
    if (threadIdx.x == 0) p.sq[(long long)g * p.sSqg + p.slot0 + l * nx + bx] = (float)r;
  }
}

// Per-sample squared gradient norms  n_i = sum_l ||delta_i^l||^2 (||a_i^{l-1}||^2 + [bias])  and inner products
// q_i = sum_l sum_parts ..., their sums (n, q, q^2, the loss) and ||gbar||^2, in double.
//
// What bounds these launches is the chain of dependent loads per sample (a norm is the sum of up to 64 tile partials),
// so four thread groups of a block share a sample: group j takes the layers j, j + 4, ..., with both norms' partials eight
// at a time in flight (b = 64 of config 3, one thread per sample: 12.6 us, of which 11 were these chains).
// Summation order: partials in index order, a group's layers in order, the four groups in order.
__device__ __forceinline__ void sum_partials2(const float *__restrict__ a, int na, const float *__restrict__ d, int nd,
                                              long long stride, float &sa, float &sd) {
  sa = sd = 0.0f;
  for (int k = 0; k < na || k < nd; k += 8) {
    float va[8], vd[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) va[u] = k + u < na ? a[(long long)(k + u) * stride] : 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) vd[u] = k + u < nd ? d[(long long)(k + u) * stride] : 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) { sa += va[u]; sd += vd[u]; }
  }
}

struct StatsSums { double s[5]; };      // n, ||gbar||^2, q^2, q, loss

// Blocks 0 .. nb-1 of a group share its samples: block j owns samples (NT / 4) j + t, then strides of nb NT / 4.
template <int NT>
__device__ __forceinline__ void stats_samples(const StatsP &p, int g, int blk, int nb, StatsSums &o, float *lds) {
  constexpr int SL = NT / 4;
  float(*comb)[4][SL] = reinterpret_cast<float(*)[4][SL]>(lds);      // [2][4][SL]
  const int gl = threadIdx.x / SL, sl = threadIdx.x % SL;
  const float hb = p.has_bias ? 1.0f : 0.0f;
  const int bg = p.rows ? p.rows[g] : p.b;
  for (int base = blk * SL; base < bg; base += nb * SL) {        // uniform over the block
    const int i = base + sl;
    const bool live = i < bg;
    float n = 0.0f, q = 0.0f;
    if (live) {
      for (int l = gl; l < p.L; l += 4) {
        if (p.do_n) {
          float a, d;
          sum_partials2(p.an[l] + (long long)g * p.an_sg[l] + i, p.an_parts[l], p.dn[l] + (long long)g * p.dn_sg[l] + i,
                        p.dn_parts[l], p.sPart, a, d);
          n = fmaf(d, a + hb, n);
        }
        if (p.do_q) {
          const float *qp = p.qpart[l] + (long long)g * p.sQg[l] + i;
          for (int k = 0; k < p.nparts[l]; k += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = k + u < p.nparts[l] ? qp[(long long)(k + u) * p.sQpart[l]] : 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) q += v[u];
          }
        }
      }
    }
    comb[0][gl][sl] = n;
    comb[1][gl][sl] = q;
    __syncthreads();
    if (gl == 0 && live) {
      const long long at = (long long)g * p.sNg + i;
      if (p.do_n) {
        n = ((n + comb[0][1][sl]) + comb[0][2][sl]) + comb[0][3][sl];
        if (p.n_out) p.n_out[at] = n;
        o.s[0] += (double)n;
        if (p.loss) o.s[4] += (double)p.loss[at];
      }
      if (p.do_q) {
        q = ((q + comb[1][1][sl]) + comb[1][2][sl]) + comb[1][3][sl];
        if (p.q_out) p.q_out[at] = q;
        o.s[3] += (double)q;
        o.s[2] += (double)q * (double)q;
      }
    }
    __syncthreads();
  }
}
// Sum over a block, fixed order; sum k ends in thread k < 5.
template <int NT>
__device__ __forceinline__ double stats_block_sums(const StatsSums &o, double *lds) {
  constexpr int NW = NT / 64;
  double(*fin)[NW] = reinterpret_cast<double(*)[NW]>(lds);           // [5][NW]
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double v = wave_sum(o.s[k]);
    if ((threadIdx.x & 63) == 0) fin[k][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x < 5)
    for (int w = 0; w < NW; ++w) r += fin[threadIdx.x][w];
  return r;
}

}  // namespace
}  // namespace absk
