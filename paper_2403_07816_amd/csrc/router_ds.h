// The router's part of the backward pass that needs only what BWD_ACT leaves: ds[T,E], and W_router laid out expert-major for the
// last step of dX.  A launch of its own, or workgroups in the launch of the weight gradients.
#pragma once
#include "common.h"

namespace btx {

struct RouterDs {
  const float* Wr; int d; float* WrT;
  int T, E, k, mode, lb_mode; float lb_alpha, lam; unsigned flags;
  const float* noise; float inv_tau;
  const int32_t* topk_idx; const float* gates; const float* probs; const int32_t* inv_pos;
  const float* gate_sum; const float* prob_sum; const int32_t* counts; const float* dg_part; int n_part, slots_log2; float* ds;
};
RouterDs router_ds_args(const RouterBwdArgs& a);
// Beside the weight gradients, if it is no more workgroups than run at a time there: two on a compute unit (strips) or five (fp32).
// Training pass, us, own launch / beside: 64 tokens of 256, f = 688, 4 experts (20 workgroups) 65.8 / 62.7; 100 of 1000, f = 264, 16 experts (88)
// 81.4 / 77.7; 1500 of 512, f = 1376, 64 experts (503) 307 / 303; 1750 of 1024, f = 688, 16 experts (502) 157.1 / 155.0; fp32 2003 of 512, f = 1376,
// 8 experts (517) 533.6 / 529.5, 4000 of them (1016) 966.6 / 962.5; f = 64: 4000 (1016) 147.2 / 143.9, 5000 (1266) 165.0 / 161.4.  Beyond, it
// gains or loses: 2500 of 1024, f = 688, 16 experts (689) 194.8 / 192.1, 3500 of 512, f = 1376, 4 experts (883) 256.7 / 256.8; fp32 f = 64:
// 5400 (1366) 177.0 / 178.9, 6000 (1516) 178.4 / 174.5.
inline bool router_ds_rides(int T, int d, int E, bool f32) {
  return ceil_div(T, 4) + (int64_t)ceil_div((int64_t)d * E, 256) <= 256 * (f32 ? 5 : 2);
}
inline unsigned router_ds_blocks(const RouterDs& a) { return (unsigned)(ceil_div(a.T, 4) + ceil_div(a.d * a.E, 256)); }

// One wavefront per token, 4 to a workgroup of 256 threads; the workgroups behind the tokens' lay W_router out (a launch less, 5 us).
__device__ __forceinline__ void router_ds(const RouterDs& a, unsigned block) {
  const int lane = threadIdx.x & (kWave - 1);
  const int token_blocks = (a.T + 3) / 4;
  if ((int)block >= token_blocks) {
    const int64_t i = (int64_t)((int)block - token_blocks) * 256 + threadIdx.x;
    if (i < (int64_t)a.d * a.E) {
      const int e = (int)(i / a.d), c = (int)(i - (int64_t)e * a.d);
      a.WrT[i] = a.Wr[(size_t)c * a.E + e];
    }
    return;
  }
  const int t = (int)block * 4 + threadIdx.x / kWave;
  if (t >= a.T) return;
  const bool live = lane < a.E;
  const float lbc = a.lb_alpha * (float)a.E / (float)a.T;
  const float pbar = live ? a.prob_sum[lane] / (float)a.T : 0.f;
  // lane j < k: slot j of this token
  int my_e = -1;
  float g = 0.f, dg = 0.f;
  if (lane < a.k) {
    my_e = a.topk_idx[(size_t)t * a.k + lane];
    g = a.gates[(size_t)t * a.k + lane];
  }
  // its dg: the partial sums of slot j by lanes j, j + slots, ..., so that they are requested together (22 of them one after
  // another: 8.6 us)
  const int slots = 1 << a.slots_log2, j = lane & (slots - 1);
  const int r = j < a.k ? a.inv_pos[(size_t)t * a.k + j] : -1;
  if (r >= 0) {                              // a dropped pair produced no output: dg = 0
    const float* part = a.dg_part + (size_t)r * a.n_part;
    for (int p = lane >> a.slots_log2; p < a.n_part; p += kWave >> a.slots_log2) dg += part[p];
  }
  for (int step = slots; step < kWave; step *= 2) dg += __shfl_xor(dg, step, kWave);
  if (lane >= a.k) dg = 0.f;
  if (a.flags & BTX_FLAG_LB_GRAD_THROUGH_U) {
    const float pb = __shfl(pbar, my_e < 0 ? 0 : my_e, kWave);
    if (lane < a.k) dg += a.lam * lbc * pb;
  }
  const float p = live ? a.probs[(size_t)t * a.E + lane] : 0.f;
  float dsv = 0.f;
  if (a.mode == BTX_ROUTE_TOPK_RENORM) {
    const float inner = wave_sum(g * dg);  // lanes >= k contribute 0
    const float mine = g * (dg - inner);
    for (int j = 0; j < a.k; ++j) {
      const int e = __shfl(my_e, j, kWave);
      const float v = __shfl(mine, j, kWave);
      if (lane == e) dsv = v;
    }
  } else if (a.mode == BTX_ROUTE_GUMBEL_TOP1) {
    // gate = y_e, y = softmax((logits + noise) / tau), rebuilt from log p (= logits up to a
    // constant per token): d gate / d logit_j = y_e (delta_ej - y_j) / tau
    const int e = __shfl(my_e, 0, kWave);
    const float dg0 = __shfl(dg, 0, kWave);
    const float v = live ? (__logf(p) + a.noise[(size_t)t * a.E + lane]) * a.inv_tau : -INFINITY;
    const float vmax = wave_max(v);
    const float z = live ? __expf(v - vmax) : 0.f;
    const float y = z / wave_sum(z);
    const float ye = __shfl(y, e, kWave);
    dsv = dg0 * ye * ((lane == e ? 1.f : 0.f) - y) * a.inv_tau;
  } else {
    const int e = __shfl(my_e, 0, kWave);
    const float dg0 = __shfl(dg, 0, kWave);
    const float pe = __shfl(p, e, kWave);
    dsv = dg0 * pe * ((lane == e ? 1.f : 0.f) - p);
  }
  if (a.lam != 0.f) {
    const float u = !live ? 0.f
                    : a.lb_mode == BTX_LB_TOKEN_FRAC ? (float)a.counts[lane] / ((float)a.T * (float)a.k)
                                                   : a.gate_sum[lane] / (float)a.T;
    const float up = wave_sum(u * p);
    dsv += a.lam * lbc * p * (u - up);
  }
  if (live) a.ds[(size_t)t * a.E + lane] = dsv;
}

}  // namespace btx
