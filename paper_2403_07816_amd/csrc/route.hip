// Router: logits, softmax, expert selection, gates, load-balancing statistics and
// the stable grouping of (token, slot) pairs by expert (Sec. 3.2 router and Top-k;
// Sec. 3.3 load balancing, Switch and sample-top-1 routing).
//
// Two launches for few tokens (see there), else four; no atomics, no host round trip:
//   (optional) the RMS normalisation in front of the sublayer (the seed model's blocks
//   normalise before their feed-forward, Sec. 4.1) is folded into route_tokens: the raw rows
//   are read once more for their mean square (fp64), the normalised, rounded rows are written
//   out for the expert GEMMs and are what the logits are computed from.
//   0. transpose_wr   W_router [d,E] -> [E,d] in the workspace: a lane then reads its 8 columns of
//                     an expert as 32 contiguous bytes and a wavefront's load covers 2 KB in one
//                     piece, where the [d,E] form costs one cache line per lane and load.  (For the matrix cores
//                     wr_fragments, the order of their loads.)
//   1. route_tokens   one wavefront handles a few tokens at a time: fp32 dot
//                     products of the token row with W_router (lanes split the row,
//                     butterfly reduction; with more than 8 experts fp32 matrix instructions
//                     on 16 tokens x 16 experts instead), then softmax / selection / gates
//                     with one lane per expert.  Each workgroup owns kTokPerBlock consecutive
//                     tokens and writes its per-expert counts and gate/prob sums.
//   2. route_scan     one workgroup per expert: exclusive scan of its block counts (fixed
//                     order) and its finished statistics.
//   3. route_scatter  every wavefront rebuilds the expert offsets from the counts (one lane per
//                     expert); one wavefront per block re-reads its indices and writes perm and
//                     inv_pos; ranks inside a block come from wavefront ballots, so the
//                     order inside every expert group is the (token, slot) order.  The first
//                     wavefront also writes offsets and lb_loss.
#include <type_traits>

#include "common.h"

namespace btx {
namespace {

constexpr int kTokPerBlock = 16;                            // consecutive tokens per workgroup
constexpr int kWavesPerBlock = 4;                           // of the scatter kernel, and of route_tokens with many tokens
constexpr int kScanThreads = 1024;
// blocks of kTokPerBlock tokens per workgroup when the logits run on the matrix cores: they share each
// load of W_router (1: 130 us, 2: 112 us, 4: 204 us for 16384 tokens x 32 experts; with 4 the launch has
// one wavefront per SIMD left)
constexpr int kMatrixGroups = 2;

// normalised value, rounded once to the row's storage type; `back` is that value again as float
template <typename XT> struct NormRound;
template <> struct NormRound<bf16_t> {
  static __device__ __forceinline__ bf16_t rnd(double v, float& back) {
    const bf16_t h = f64_to_bf16(v);
    back = bf16_to_f32(h);
    return h;
  }
  static __device__ __forceinline__ void st8(bf16_t* p, const bf16_t* h) {
    *reinterpret_cast<u32x4*>(p) = u32x4{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                                         (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
  }
};
template <> struct NormRound<float> {
  static __device__ __forceinline__ float rnd(double v, float& back) { return back = (float)v; }
  static __device__ __forceinline__ void st8(float* p, const float* h) {
    *reinterpret_cast<f32x4*>(p) = f32x4{h[0], h[1], h[2], h[3]};
    *reinterpret_cast<f32x4*>(p + 4) = f32x4{h[4], h[5], h[6], h[7]};
  }
};
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);   // every lane ends with the same bits
  return v;
}

struct Best { float v; int i; };
// larger value wins; equal values: lower index wins
__device__ __forceinline__ Best best_of(Best a, Best b) {
  return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}
template <int CTRL> __device__ __forceinline__ Best dpp_best(Best x) {
  return best_of(x, Best{dpp_f32<CTRL>(x.v), dpp_i32<CTRL>(x.i)});
}
__device__ __forceinline__ Best lane_best(Best x, int lane) {
  return Best{lane_f32(x.v, lane), __builtin_amdgcn_readlane(x.i, lane)};
}
// (value, index) arg-max over the wavefront; the same DPP scheme as wave_sum
__device__ __forceinline__ Best wave_best(Best x) {
  x = dpp_best<kDppXor1>(x);
  x = dpp_best<kDppXor2>(x);
  x = dpp_best<kDppRor4>(x);
  x = dpp_best<kDppRor8>(x);
  return best_of(best_of(lane_best(x, 0), lane_best(x, 16)), best_of(lane_best(x, 32), lane_best(x, 48)));
}
__device__ __forceinline__ float wave_incl_scan(float v, int lane) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const float u = __shfl_up(v, o, kWave);
    if (lane >= o) v += u;
  }
  return v;
}

// 8 consecutive elements of a row as they are loaded (the conversion to float waits until they are used,
// so that loads issued ahead stay in flight)
template <typename XT> struct Raw8;
template <> struct Raw8<bf16_t> {
  u32x4 r;
  __device__ __forceinline__ void load(const bf16_t* p) { r = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ float get(int i) const { return (i & 1) ? bf16hi(r[i >> 1]) : bf16lo(r[i >> 1]); }
};
template <> struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ float get(int i) const { return i < 4 ? a[i] : b[i - 4]; }
};

// Softmax, expert selection and gates of token t by one wavefront; lane e owns expert e, s is its logit.  What the
// token adds to expert e's statistics is added to lane e's psum, gsum and cnt.
__device__ __forceinline__ void select_experts(float s, bool live, int lane, int t, int E, int k, int mode, float inv_tau,
                                               const float* __restrict__ U, int32_t* __restrict__ topk_idx,
                                               float* __restrict__ gates, float* __restrict__ probs, float& psum,
                                               float& gsum, int& cnt) {
  const float smax = wave_max(s);
  const float z = live ? __expf(s - smax) : 0.f;
  const float zsum = wave_sum(z);
  const float p = z / zsum;
  if (live) probs[(size_t)t * E + lane] = p;
  psum += p;
  if (mode == BTX_ROUTE_TOPK_RENORM) {
    // k different experts whatever the logits are, so that every slot is written: a NaN counts as -infinity, and an
    // expert that is taken (or does not exist) comes after every other one of that value
    Best mine = live && s == s ? Best{s, lane} : Best{-INFINITY, live ? lane : lane + kWave};
    int my_slot = -1;
    for (int j = 0; j < k; ++j) {
      if (wave_best(mine).i == lane) { my_slot = j; mine = Best{-INFINITY, lane + kWave}; }
    }
    const float zsel = wave_sum(my_slot >= 0 ? z : 0.f);
    if (my_slot >= 0) {
      const float g = z / zsel;
      topk_idx[(size_t)t * k + my_slot] = lane;
      gates[(size_t)t * k + my_slot] = g;
      gsum += g;
      cnt += 1;
    }
    return;
  }
  int chosen;
  float g = p;
  if (mode == BTX_ROUTE_SWITCH_TOP1) {
    chosen = wave_best(Best{s, lane}).i;
  } else if (mode == BTX_ROUTE_GUMBEL_TOP1) {
    // soft sample softmax((logits + noise) / tau); its largest entry is 1 / sum of the
    // others' ratios to it, and that entry alone is kept
    const float noisy = live ? s + U[(size_t)t * E + lane] : -INFINITY;
    const Best b = wave_best(Best{noisy, lane});
    chosen = b.i;
    g = 1.f / wave_sum(live ? __expf((noisy - b.v) * inv_tau) : 0.f);
  } else {
    const float c = wave_incl_scan(p, lane);
    const unsigned long long m = __ballot(live && c > U[t]);
    chosen = m ? (__ffsll((long long)m) - 1) : (E - 1);
  }
  if (lane == chosen) {
    topk_idx[t] = lane;
    gates[t] = g;
    gsum += g;
    cnt += 1;
  }
}

// ---- few tokens: two launches ----------------------------------------------------------------------------------
// A decoding step or a prompt is latency: the kernels below gave it one wavefront per 4 tokens, which walked its rows
// twice, and three more launches (16 tokens of 4096 columns with the normalisation: 66 us).  Here every token has a
// workgroup whose threads share its columns and read W_router as it lies, and one workgroup does the grouping:
// 16 tokens of 4096 columns with the normalisation 11 us, 301 tokens 15, 512 tokens 16.  From there on it depends, see
// route_is_small().
constexpr int kSmallTokens = 512, kSmallPairs = 4096;
constexpr int64_t kSmallTraffic = (int64_t)1 << 25;     // T * d * E: every token reads the whole W_router (128 MB in all)
constexpr int kSmallThreads = 256, kGroupThreads = 1024;

// AHEAD: pieces of a thread, 8 columns of the token, the first experts' weights and the gain, that are requested at once, in front of the
// mean square's sum instead of behind it: none or two (see launch_route_small()).
template <typename XT, int EC, bool NORM, int AHEAD>
__global__ __launch_bounds__(kSmallThreads) void route_small_tokens_kernel(
    const XT* __restrict__ x, const float* __restrict__ Wr, const float* __restrict__ br, const float* __restrict__ U,
    int d, int E, int k, int mode, float inv_tau, int32_t* __restrict__ topk_idx, float* __restrict__ gates,
    float* __restrict__ probs, const float* __restrict__ gain, float eps, XT* __restrict__ xn,
    float* __restrict__ rstd_out) {
  typedef f32x4 __attribute__((aligned(4))) f32x4_any;  // W_router need only be aligned to its elements
  __shared__ float s_part[kSmallThreads / kWave][kMaxExperts];
  __shared__ double s_ss[kSmallThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, t = blockIdx.x;
  const XT* row = x + (size_t)t * d;
  struct Piece { Raw8<XT> x; float w[8][EC], g[NORM ? 8 : 1]; };
  constexpr int STEP = kSmallThreads * 8;
  auto load_w = [&](float (&w)[8][EC], int c0, int e0) {
    const float* w0 = Wr + (size_t)c0 * E + e0;
    if (EC % 4 == 0 && e0 + EC <= E) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < EC; j += 4) {
          const f32x4_any q = *reinterpret_cast<const f32x4_any*>(w0 + (size_t)i * E + j);
#pragma unroll
          for (int y = 0; y < 4 && j + y < EC; ++y) w[i][j + y] = q[y];
        }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < EC; ++j) w[i][j] = e0 + j < E ? w0[(size_t)i * E + j] : 0.f;
    }
  };
  auto load = [&](Piece& p, int c0, int e0) {
    p.x.load(row + c0);
    load_w(p.w, c0, e0);
    if constexpr (NORM) RowVec<float, 8>::ld(gain + c0, p.g);
  };
  Piece first[AHEAD ? AHEAD : 1];
#pragma unroll
  for (int q = 0; q < AHEAD; ++q)
    if (const int c0 = threadIdx.x * 8 + q * STEP; c0 < d) load(first[q], c0, 0);
  double rs = 0.0;
  if (NORM) {                                           // in fp64, for the reason given at route_tokens_kernel
    double ss = 0.0;
    auto square = [&](const Raw8<XT>& v) {
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += (double)v.get(i) * (double)v.get(i);
    };
#pragma unroll
    for (int q = 0; q < AHEAD; ++q)
      if (threadIdx.x * 8 + q * STEP < d) square(first[q].x);
    for (int c0 = threadIdx.x * 8 + AHEAD * STEP; c0 < d; c0 += STEP) {
      Raw8<XT> v;
      v.load(row + c0);
      square(v);
    }
    ss = wave_sum_f64(ss);
    if (lane == 0) s_ss[wave] = ss;
    __syncthreads();
    rs = 1.0 / sqrt(((s_ss[0] + s_ss[1]) + (s_ss[2] + s_ss[3])) / (double)d + (double)eps);
    if (threadIdx.x == 0) rstd_out[t] = (float)rs;
  }
  for (int e0 = 0; e0 < E; e0 += EC) {
    float acc[EC] = {};
    auto add = [&](const Piece& p, int c0) {
      float xv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) xv[i] = p.x.get(i);
      if constexpr (NORM) {
        XT h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) h[i] = NormRound<XT>::rnd((double)xv[i] * rs * (double)p.g[i], xv[i]);
        if (e0 == 0) NormRound<XT>::st8(xn + (size_t)t * d + c0, h);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < EC; ++j) acc[j] = fmaf(xv[i], p.w[i][j], acc[j]);
    };
    int c0 = threadIdx.x * 8;
    if (e0 == 0) {
#pragma unroll
      for (int q = 0; q < AHEAD; ++q, c0 += STEP)
        if (c0 < d) add(first[q], c0);
    }
    for (; c0 < d; c0 += STEP) {
      Piece p;
      load(p, c0, e0);
      add(p, c0);
    }
#pragma unroll
    for (int j = 0; j < EC; ++j) {
      const float sum = wave_sum(acc[j]);
      if (lane == 0 && e0 + j < E) s_part[wave][e0 + j] = sum;
    }
  }
  __syncthreads();
  if (wave != 0) return;
  const bool live = lane < E;
  float s = -INFINITY, psum = 0.f, gsum = 0.f;
  int cnt = 0;
  if (live) s = ((s_part[0][lane] + s_part[1][lane]) + (s_part[2][lane] + s_part[3][lane])) + (br ? br[lane] : 0.f);
  select_experts(s, live, lane, t, E, k, mode, inv_tau, U, topk_idx, gates, probs, psum, gsum, cnt);
}

// One workgroup: statistics, offsets and lb_loss, and the stable grouping of the pairs.  Latency is all it costs: what the
// token kernel left is requested at once (up to four pairs a thread), ranks stay in registers, and a wavefront finds the
// lanes of the same expert with a ballot for every bit of the index.  With a ballot per expert, three barriers for every 1024
// pairs and ranks that waited in inv_pos: 512 tokens, 4 experts, top-2
// 12.4 us, now 6; 64 experts, top-8 38, now 16.
// ROUNDS: pairs a thread can have; PIECE: floats of [token][expert] that LDS holds of gates and of probabilities.  (The large
// form's code alone costs a decoding step 0.9 us.)
template <int ROUNDS, int PIECE> __global__ __launch_bounds__(kGroupThreads) void route_small_group_kernel(
    int T, int E, int k, int cap, int lb_mode, float lb_alpha, const int32_t* __restrict__ topk_idx,
    const float* __restrict__ gates, const float* __restrict__ probs, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv_pos,
    float* __restrict__ gate_sum, float* __restrict__ prob_sum, float* __restrict__ lb_loss) {
  constexpr int kWaves = kGroupThreads / kWave, kLoads = PIECE / kGroupThreads;
  static_assert(PIECE % kGroupThreads == 0 && PIECE / kMaxExperts >= kWaves, "a piece holds kWaves tokens of any number of experts");
  __shared__ int s_cnt[ROUNDS * kWaves][kMaxExperts], s_first[kMaxExperts], s_kept;
  __shared__ float s_gate[PIECE], s_prob[PIECE], s_sum[2][kWaves][kMaxExperts];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, R = T * k;

  int e[ROUNDS], local[ROUNDS];
  float gate[ROUNDS];
#pragma unroll
  for (int j = 0; j < ROUNDS; ++j) {
    const int i = j * kGroupThreads + threadIdx.x;
    e[j] = i < R ? topk_idx[i] : -1;
    gate[j] = i < R ? gates[i] : 0.f;
    if (j * kGroupThreads < R) s_cnt[j * kWaves + wave][lane] = 0;
  }

  // ---- gate and probability sums: thread (expert lane, group wave) adds every kWaves-th token, groups in order.  The
  // gates are laid out [token][expert] first, as many tokens at a time as the LDS pieces hold.
  float g = 0.f, p = 0.f;
  const int span = min(T, PIECE / E / kWaves * kWaves);
  for (int t0 = 0; t0 < T; t0 += span) {
    const int n = min(span, T - t0);
    float v[kLoads];
#pragma unroll
    for (int x = 0; x < kLoads; ++x) {
      const int i = x * kGroupThreads + threadIdx.x;
      v[x] = i < n * E ? probs[(size_t)t0 * E + i] : 0.f;
    }
#pragma unroll
    for (int x = 0; x < kLoads; ++x)
      if (x * kGroupThreads < n * E) s_gate[x * kGroupThreads + threadIdx.x] = 0.f;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kLoads; ++x)
      if (x * kGroupThreads < n * E) s_prob[x * kGroupThreads + threadIdx.x] = v[x];
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
      const int i = j * kGroupThreads + threadIdx.x - t0 * k;      // pair of the span
      if (e[j] >= 0 && i >= 0 && i < n * k) s_gate[i / k * E + e[j]] = gate[j];
    }
    if (t0 == 0) {                                      // ranks inside a wavefront's 64 pairs, and how many each expert has of them
#pragma unroll
      for (int j = 0; j < ROUNDS; ++j) {
        local[j] = 0;
        if (j * kGroupThreads >= R) continue;
        unsigned long long same = __ballot(e[j] >= 0);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
          const unsigned long long ones = __ballot((e[j] >> b) & 1);
          same &= (e[j] >> b) & 1 ? ones : ~ones;
        }
        local[j] = __popcll(same & ((1ull << lane) - 1ull));
        if (e[j] >= 0 && local[j] == 0) s_cnt[j * kWaves + wave][e[j]] = __popcll(same);
      }
    }
    __syncthreads();
    if (lane < E) {
#pragma unroll 8
      for (int q = wave; q < n; q += kWaves) {
        g += s_gate[q * E + lane];
        p += s_prob[q * E + lane];
      }
    }
    if (t0 + span < T) __syncthreads();
  }
  s_sum[0][wave][lane] = g;
  s_sum[1][wave][lane] = p;
  __syncthreads();

  // ---- what every expert ends with
  if (wave == 0) {
    int running = 0;                                    // lane e: pairs of expert e so far
    for (int w0 = 0; w0 * kWave < R; w0 += kWaves) {
      int c[kWaves];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) c[w] = s_cnt[w0 + w][lane];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        s_cnt[w0 + w][lane] = running;
        running += c[w];
      }
    }
    const int kept = cap > 0 ? min(running, cap) : running;
    const int incl = wave_incl_scan_i32(kept, lane);
    float gs = 0.f, ps = 0.f, term = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { gs += s_sum[0][w][lane]; ps += s_sum[1][w][lane]; }
    s_first[lane] = incl - kept;
    if (lane == kWave - 1) { s_kept = incl; offsets[E] = incl; }
    if (lane < E) {
      counts[lane] = running;
      offsets[lane] = incl - kept;
      gate_sum[lane] = gs;
      prob_sum[lane] = ps;
      const float u = lb_mode == BTX_LB_TOKEN_FRAC ? (float)running / ((float)T * (float)k) : gs / (float)T;
      term = u * (ps / (float)T);
    }
    float loss = 0.f;
    for (int x = 0; x < E; ++x) loss += lane_f32(term, x);         // expert order
    if (lane == 0) *lb_loss = lb_alpha * (float)E * loss;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ROUNDS; ++j) {
    const int i = j * kGroupThreads + threadIdx.x;
    if (e[j] < 0) continue;
    const int rank = s_cnt[j * kWaves + wave][e[j]] + local[j];
    if (cap > 0 && rank >= cap) {
      inv_pos[i] = -1;                                  // beyond the expert's capacity: dropped
    } else {
      const int pos = s_first[e[j]] + rank;
      perm[pos] = i;
      inv_pos[i] = pos;
    }
  }
  for (int r = s_kept + threadIdx.x; r < R; r += kGroupThreads) perm[r] = 0;   // no such rows: any valid pair
}

// Two launches win up to kSmallTokens tokens; above, route_small_tokens and the one grouping workgroup lose ground to four launches with
// every token.  us, four launches / two:
//   whole vector loads of W_router (4, 8, 16 experts; 9, where one column is left over): 1024 tokens of 1024 columns, 4 experts, top-2
//     14.3 / 13.3, of 2048 15.5 / 15.2, of 4096 17.7 / 19; top-3 853 of 1024 14.8 / 14.0, top-4 1024 of 2048 16.7 / 17.6; 640 of 1024, 8
//     experts 16.5 / 14.2, of 2336 19.4 / 17.8; 9 experts, 640 of 1024 17.0 / 14.3, of 1600 17.3 / 16.9; 16 experts, top-4, 640 of 392
//     17.0 / 16.2, of 776 17.3 / 17.9, of 1024 20.3 / 18.9, of 1072 18.6 / 20.5 (with the normalisation 26.4 / 20.2 for 776)
//   other numbers of experts, whose last columns are loaded one by one: 1024 of 256, 2 experts 11.8 / 9.6, of 384 12.6 / 12.6, of 4096
//     15.7 / 25; 3 experts of 512 13.6 / 14.0; 640 of 256, 7 experts 15.2 / 14.2, of 448 15.3 / 15.8; 5 experts 640 of 512 14.4 / 13.8, 520
//     of 4096 19.5 / 42; 640 of 256, 13 experts 17.7 / 16.6, 12 of 1024 19.3 / 20.7
//   64 experts, top-4, of 512 columns: 512 tokens 31 / 31, 600 31 / 34
// The normalisation is not asked, though it gains more (1024 of 2048, 4 experts 20.9 / 17.3): a logit's sum has another order in two
// launches than in four, and routing with it is routing without it on the rows it writes, bit for bit.
bool route_is_small(const RouteArgs& a) {
  const int64_t traffic = (int64_t)a.T * a.d * a.E, pairs = (int64_t)a.T * a.k;
  if (pairs > kSmallPairs || traffic > kSmallTraffic) return false;
  if (a.T <= kSmallTokens) return true;
  if (a.E <= 8)
    return a.T <= (a.E <= 4 ? 1024 : 640) && (a.E > 4 || pairs <= 2560) &&
           traffic <= (a.E % 4 == 0 ? 12000000 : a.E < 4 ? 800000 : 1300000);
  return a.E <= 16 && a.T <= 640 && traffic <= (a.E == 9 || (a.E == 16 && a.d <= 1024) ? 10500000 : 2500000);
}

int launch_route_small(const RouteArgs& a, hipStream_t s) {
  auto tokens = [&](auto tag, auto ec, auto norm) {
    using XT = decltype(tag);
    constexpr int EC = decltype(ec)::value;
    constexpr bool NORM = decltype(norm)::value;
    // Two pieces ahead where that was measured to gain: us, the whole routing, none / two: bf16, 4096 columns, 16 tokens, 4 experts 10.7 / 10.0,
    // 8 12.9 / 12.2, 16 20.5 / 19.8; 512 tokens, 8 experts 19.1 / 18.5, 16 34.1 / 32.3; fp32, 16 tokens, 4 experts 9.8 / 9.3, 512, 8 18.9 / 18.7.  Up
    // to 2048 columns a thread has no second piece; the fourth and fifth wait as long as they did, beside more registers; of up to 4 bf16 experts
    // other workgroups cover the wait of more than 256 tokens; a second set of experts that is not whole loses (12, 256 tokens of 3072: bf16 19.6 / 22.7,
    // fp32 18.3 / 21.3).  Of 810 calls of 1024 to 16384 columns, 2 to 32 experts, 16 to 512 tokens it takes 204, which gain 3.9 % on average, four of them
    // lose 1.2 to 1.8 %.
    const bool ahead = NORM && a.d > 2048 && (sizeof(XT) == 4 ? a.d <= 4096 && a.E <= 8
                                                              : a.E <= 4 ? a.d <= 6144 && a.T <= 256 : a.d <= 8192 && (a.E <= 8 || a.E == 16));
    const auto kernel = ahead ? route_small_tokens_kernel<XT, EC, NORM, NORM ? 2 : 0> : route_small_tokens_kernel<XT, EC, NORM, 0>;
    kernel<<<a.T, kSmallThreads, 0, s>>>(
        static_cast<const XT*>(a.x), a.W_router, a.b_router, a.U, a.d, a.E, a.k, a.route_mode, 1.f / a.tau, a.topk_idx,
        a.gates, a.probs, a.gain, a.eps, static_cast<XT*>(a.xn), a.rstd);
  };
  auto by_experts = [&](auto tag, auto norm) {
    if (a.E <= 2) tokens(tag, std::integral_constant<int, 2>{}, norm);
    else if (a.E <= 4) tokens(tag, std::integral_constant<int, 4>{}, norm);
    else tokens(tag, std::integral_constant<int, 8>{}, norm);
  };
  auto by_norm = [&](auto tag) {
    if (a.gain) by_experts(tag, std::true_type{});
    else by_experts(tag, std::false_type{});
  };
  if (a.x_dtype == BTX_BF16) by_norm(bf16_t{});
  else by_norm(float{});
  BTX_LAUNCH_CHECK();
  auto group = [&](auto rounds, auto piece) {
    route_small_group_kernel<decltype(rounds)::value, decltype(piece)::value><<<1, kGroupThreads, 0, s>>>(
        a.T, a.E, a.k, a.cap, a.lb_mode, a.lb_alpha, a.topk_idx, a.gates, a.probs, a.counts, a.offsets, a.perm, a.inv_pos,
        a.gate_sum, a.prob_sum, a.lb_loss);
  };
  const std::integral_constant<int, 1> one_round;
  if (a.T * a.k <= kGroupThreads && a.T * a.E <= kGroupThreads) group(one_round, std::integral_constant<int, kGroupThreads>{});
  else if (a.T * a.k <= kGroupThreads) group(one_round, std::integral_constant<int, 4 * kGroupThreads>{});
  else group(std::integral_constant<int, kSmallPairs / kGroupThreads>{}, std::integral_constant<int, 4 * kGroupThreads>{});
  BTX_LAUNCH_CHECK();
  return BTX_OK;
}

// ---- many tokens ---------------------------------------------------------------------------------------------
// EC experts are accumulated per pass over the row; the 16 / NW tokens of a wavefront share each
// load of the (transposed) W_router.
// NW: wavefronts of a workgroup, see token_waves().
template <typename XT, int EC, bool NORM, int NW, int MG = 1, int NS = 1>
__global__ __launch_bounds__(NW* kWave, NW == 8 && EC > 0 ? 4 : 1)   // 8: two workgroups on a compute unit
void route_tokens_kernel(
    const XT* __restrict__ x, const float* __restrict__ WrT, const float* __restrict__ br,
    const float* __restrict__ U, int T, int d, int E, int k, int mode, float inv_tau, int32_t* __restrict__ topk_idx,
    float* __restrict__ gates, float* __restrict__ probs, int32_t* __restrict__ blk_counts,
    float* __restrict__ blk_gsum, float* __restrict__ blk_psum, const float* __restrict__ gain, float eps,
    XT* __restrict__ xn, float* __restrict__ rstd_out) {
  constexpr bool MATRIX = EC == 0;                      // logits on the matrix cores (many experts)
  static_assert(!(MATRIX && NORM), "the matrix-core logits take the rows as they are");
  // the matrix variant covers G blocks of kTokPerBlock tokens per workgroup (they share every load of
  // W_router); the statistics stay per block of kTokPerBlock tokens either way
  constexpr int G = MATRIX ? MG : 1;
  constexpr int kTokPerWave = kTokPerBlock / NW;
  constexpr int kGroup = kTokPerBlock / kWavesPerBlock, kTokPerSlot = kTokPerWave == kGroup ? kGroup : 1, kSlots = kTokPerBlock / kTokPerSlot;
  __shared__ float s_logit[NW][kTokPerWave][kMaxExperts];
  __shared__ float s_stat[kSlots][3][kMaxExperts];
  extern __shared__ float s_part[];                     // MATRIX: [wavefront][G * kTokPerBlock tokens][16 NS experts]
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int n_blk = (T + kTokPerBlock - 1) / kTokPerBlock;
  const int pitch = 16 * NS;                            // MATRIX: NS = ceil(E / 16) sets of 16 experts
  int t0 = blockIdx.x * G * kTokPerBlock + wave * kTokPerWave;

  // ---- row factors of the normalisation -------------------------------------
  // fp64 throughout: the rounded rows then agree with a host fp64 evaluation except where the
  // exact value lies within 1e-16 (relative) of a rounding tie, and so do the routing decisions.
  double rs[kTokPerWave];
  if (NORM) {
    double ss[kTokPerWave] = {};
    for (int c0 = lane * 8; c0 < d; c0 += kWave * 8) {
#pragma unroll
      for (int q = 0; q < kTokPerWave; ++q) {
        float v[8];
        RowVec<XT, 8>::ld(x + (size_t)min(t0 + q, T - 1) * d + c0, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) ss[q] += (double)v[i] * (double)v[i];
      }
    }
#pragma unroll
    for (int q = 0; q < kTokPerWave; ++q) {
      rs[q] = 1.0 / sqrt(wave_sum_f64(ss[q]) / (double)d + (double)eps);
      if (lane == 0 && t0 + q < T) rstd_out[t0 + q] = (float)rs[q];
    }
  }

  // ---- logits -------------------------------------------------------------
  if constexpr (MATRIX) {
    // fp32 16x16x4 matrix products: the workgroup's 16 tokens are the rows, 16 experts at a time the
    // columns; wavefront w takes the 32-column pieces w, w + NW, ... of the rows and the NW partial
    // sums are added in that order below.  A lane supplies A[token = lane % 16][k] and
    // B[k][expert = lane % 16] for the 8 columns k = 32 piece + 8 (lane / 16) + i, one product per i,
    // and receives the sums of expert lane % 16 for the tokens 4 (lane / 16) + v.
    const int row = lane & 15, kc = lane >> 4;
    const XT* xrow[G];
    f32x4 acc[G][NS];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      xrow[g] = x + (size_t)min((blockIdx.x * G + g) * kTokPerBlock + row, T - 1) * d;   // clamped rows are dropped later
#pragma unroll
      for (int u = 0; u < NS; ++u) acc[g][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // experts of a set, and the one of this lane (past E: expert E - 1 again, whose sums are never looked at)
    auto of_set = [&](int u) { return u + 1 < NS ? 16 : E - 16 * (NS - 1); };
    // Trip `it` of this wavefront covers columns 32 (wave + NW it) ... + 31.  The loads of kAhead trips are
    // in flight ahead of the products, and nothing in the loop is conditional (the matrix instructions
    // take all 64 lanes, and a branch would make the compiler wait for every load): a trip past the
    // last one repeats the last one's loads, and a lane whose 8 columns lie past the row's end reads the
    // row's first 8; both supply zeros for the tokens.
    // 2 everywhere: 5200 tokens of 5120 columns, 64 experts 81 us for 76; 3: 10000 of 8192, 16 experts 89 for 83, 1921 of 4096, 64 experts 43.8 for 43.1
    constexpr int kAhead = NW == 8 || NS == 1 ? 2 : 3;
    struct Piece { Raw8<XT> xr[G]; Raw8<float> wr[NS]; };
    Piece buf[kAhead];
    const int n_it = max(0, (d - wave * 32 + NW * 32 - 1) / (NW * 32));
    auto col0 = [&](int it, bool& live) {
      const int c = (wave + NW * min(it, max(n_it - 1, 0))) * 32 + kc * 8;
      live = it < n_it && c < d;
      return c < d ? c : 0;
    };
    auto fetch = [&](Piece& pc, int it) {
      bool live;
      const int c0 = col0(it, live);
#pragma unroll
      for (int g = 0; g < G; ++g) pc.xr[g].load(xrow[g] + c0);
      const int p0 = (wave + NW * min(it, max(n_it - 1, 0))) * 32, chunks = max(min((d - p0) / 8, 4), 1);   // see wr_fragments_kernel
      const float* w0 = WrT + (p0 < d ? (size_t)p0 * E : 0);
      const int c = kc < chunks ? kc : 0, half = chunks * 4 * E;
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const float* w = w0 + u * 64 * chunks + (c * of_set(u) + min(row, of_set(u) - 1)) * 4;
        pc.wr[u].a = *reinterpret_cast<const f32x4*>(w);
        pc.wr[u].b = *reinterpret_cast<const f32x4*>(w + half);
      }
    };
    auto multiply = [&](const Piece& pc, int it) {
      bool live;
      col0(it, live);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float xa[G];
#pragma unroll
        for (int g = 0; g < G; ++g) xa[g] = live ? pc.xr[g].get(i) : 0.f;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
          const float wb = pc.wr[u].get(i);
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[g], wb, acc[g][u], 0, 0, 0);
        }
      }
    };
#pragma unroll
    for (int j = 0; j < kAhead - 1; ++j) fetch(buf[j], j);
    int it0 = 0;
    for (; it0 + kAhead <= n_it; it0 += kAhead) {
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        fetch(buf[(j + kAhead - 1) % kAhead], it0 + j + kAhead - 1);
        __builtin_amdgcn_sched_barrier(0);              // keeps the compiler from sinking the loads to their uses
        multiply(buf[j], it0 + j);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // what is left of the trips, their loads are on their way (a whole round instead: 5200 tokens of 2568 columns, 21 trips, 40 experts, fp32
    // 52 us for 48)
#pragma unroll
    for (int j = 0; j < kAhead - 1; ++j)
      if (it0 + j < n_it) multiply(buf[j], it0 + j);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int u = 0; u < NS; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          s_part[((wave * G + g) * kTokPerBlock + 4 * kc + v) * pitch + u * 16 + row] = acc[g][u][v];
  }
  constexpr int ECN = MATRIX ? 1 : EC;                  // (the loop below is not instantiated for MATRIX)
  if constexpr (!MATRIX) for (int e0 = 0; e0 < E; e0 += ECN) {
    float acc[kTokPerWave][ECN];
#pragma unroll
    for (int q = 0; q < kTokPerWave; ++q)
#pragma unroll
      for (int j = 0; j < ECN; ++j) acc[q][j] = 0.f;
    for (int c0 = lane * 8; c0 < d; c0 += kWave * 8) {
      float xv[kTokPerWave][8];
#pragma unroll
      for (int q = 0; q < kTokPerWave; ++q) {
        const int t = min(t0 + q, T - 1);  // clamped rows are computed and then dropped
        RowVec<XT, 8>::ld(x + (size_t)t * d + c0, xv[q]);
      }
      if (NORM) {
        float gv[8];
        RowVec<float, 8>::ld(gain + c0, gv);
#pragma unroll
        for (int q = 0; q < kTokPerWave; ++q) {
          XT h[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) h[i] = NormRound<XT>::rnd((double)xv[q][i] * rs[q] * (double)gv[i], xv[q][i]);
          if (e0 == 0 && t0 + q < T) NormRound<XT>::st8(xn + (size_t)(t0 + q) * d + c0, h);
        }
      }
#pragma unroll
      for (int j = 0; j < ECN; ++j) {
        float w[8] = {};
        if (e0 + j < E) RowVec<float, 8>::ld(WrT + (size_t)(e0 + j) * d + c0, w);
#pragma unroll
        for (int q = 0; q < kTokPerWave; ++q)
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[q][j] = fmaf(xv[q][i], w[i], acc[q][j]);
      }
    }
#pragma unroll
    for (int q = 0; q < kTokPerWave; ++q)
#pragma unroll
      for (int j = 0; j < ECN; ++j) {
        const float s = wave_sum(acc[q][j]);
        if (lane == 0 && e0 + j < E) s_logit[wave][q][e0 + j] = s;
      }
  }
  const bool live = lane < E;
  for (int g = 0; g < G; ++g, t0 += kTokPerBlock) {
    const int blk = blockIdx.x * G + g;                   // block of kTokPerBlock tokens
    if (blk >= n_blk) break;                              // uniform across the workgroup
    __syncthreads();                                      // logits (or partial sums) written; s_stat free again
    if (MATRIX && live) {                                 // the wavefronts' partial sums, in wavefront order
#pragma unroll
      for (int q = 0; q < kTokPerWave; ++q) {
        const int tok = g * kTokPerBlock + wave * kTokPerWave + q;
        float sum = s_part[tok * pitch + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += s_part[(w * G * kTokPerBlock + tok) * pitch + lane];
        s_logit[wave][q][lane] = sum;                     // read back by this lane only
      }
    }

    // ---- per token: softmax, selection, gates; lane e owns expert e ----------
    // the statistics are sums over groups of kGroup tokens, then over the groups, whatever NW is: the same bits as with any
    // other number of wavefronts
#pragma unroll 1
    for (int q0 = 0; q0 < kTokPerWave; q0 += kTokPerSlot) {
      int cnt = 0;
      float gsum = 0.f, psum = 0.f;
      for (int q = q0; q < q0 + kTokPerSlot; ++q) {
        const int t = t0 + q;
        if (t >= T) break;  // uniform across the wave
        const float s = live ? s_logit[wave][q][lane] + (br ? br[lane] : 0.f) : -INFINITY;
        select_experts(s, live, lane, t, E, k, mode, inv_tau, U, topk_idx, gates, probs, psum, gsum, cnt);
      }
      const int slot = (wave * kTokPerWave + q0) / kTokPerSlot;
      s_stat[slot][0][lane] = __int_as_float(cnt);
      s_stat[slot][1][lane] = gsum;
      s_stat[slot][2][lane] = psum;
    }
    __syncthreads();
    if (threadIdx.x < E) {
      const int e = threadIdx.x;
      int c = 0;
      float gs = 0.f, p = 0.f;
#pragma unroll
      for (int w = 0; w < kSlots; w += kGroup / kTokPerSlot) {
        float group_gs = 0.f, group_p = 0.f;
#pragma unroll
        for (int x = w; x < w + kGroup / kTokPerSlot; ++x) {
          c += __float_as_int(s_stat[x][0][e]);
          group_gs += s_stat[x][1][e];
          group_p += s_stat[x][2][e];
        }
        gs += group_gs;
        p += group_p;
      }
      blk_counts[(size_t)blk * E + e] = c;
      blk_gsum[(size_t)blk * E + e] = gs;
      blk_psum[(size_t)blk * E + e] = p;
    }
  }
}

// Exclusive scan of v over the workgroup (kScanThreads threads); returns the
// exclusive prefix and writes the total to `total`.
__device__ __forceinline__ int block_excl_scan(int v, int& total, int* s_wave) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += u;
  }
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  int base = 0, tot = 0;
  for (int w = 0; w < kScanThreads / kWave; ++w) {
    const int c = s_wave[w];
    if (w < wave) base += c;
    tot += c;
  }
  __syncthreads();
  total = tot;
  return base + incl - v;
}

// one workgroup per expert
__global__ __launch_bounds__(kScanThreads) void route_scan_kernel(
    int nblk, int E, const int32_t* __restrict__ blk_counts, const float* __restrict__ blk_gsum,
    const float* __restrict__ blk_psum, int32_t* __restrict__ blk_base, int32_t* __restrict__ counts,
    float* __restrict__ gate_sum, float* __restrict__ prob_sum) {
  __shared__ int s_wave[kScanThreads / kWave];
  __shared__ float s_red[2][kScanThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int e = blockIdx.x;
  int running = 0;
  float g = 0.f, p = 0.f;
  for (int b0 = 0; b0 < nblk; b0 += kScanThreads) {
    const int b = b0 + threadIdx.x;
    const int v = b < nblk ? blk_counts[(size_t)b * E + e] : 0;
    int total;
    const int ex = block_excl_scan(v, total, s_wave);
    if (b < nblk) {
      blk_base[(size_t)b * E + e] = running + ex;
      g += blk_gsum[(size_t)b * E + e];
      p += blk_psum[(size_t)b * E + e];
    }
    running += total;
  }
  // fixed-order reduction of the per-thread partial sums
  g = wave_sum(g);
  p = wave_sum(p);
  if (lane == 0) { s_red[0][wave] = g; s_red[1][wave] = p; }
  __syncthreads();
  if (threadIdx.x == 0) {
    float gs = 0.f, ps = 0.f;
    for (int w = 0; w < kScanThreads / kWave; ++w) { gs += s_red[0][w]; ps += s_red[1][w]; }
    counts[e] = running;
    gate_sum[e] = gs;
    prob_sum[e] = ps;
  }
}

// grid: one wavefront per token block, plus workgroups that only clear perm's tail
__global__ __launch_bounds__(kWavesPerBlock* kWave) void route_scatter_kernel(
    int nblk, int T, int E, int k, int cap, int lb_mode, float lb_alpha, const int32_t* __restrict__ topk_idx,
    const int32_t* __restrict__ blk_base, const int32_t* __restrict__ counts, const float* __restrict__ gate_sum,
    const float* __restrict__ prob_sum, int32_t* __restrict__ offsets, float* __restrict__ lb_loss,
    int32_t* __restrict__ perm, int32_t* __restrict__ inv_pos) {
  const int lane = threadIdx.x & (kWave - 1);
  // lane e: expert e's first grouped row.  capacity: an expert keeps its first `cap` pairs; the
  // statistics see the routing
  const int cnt = lane < E ? counts[lane] : 0;
  const int kept = cap > 0 ? min(cnt, cap) : cnt;
  int incl = kept;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += u;
  }
  const int group0 = incl - kept;
  const int kept_total = __shfl(incl, kWave - 1, kWave);
  if (blockIdx.x == 0 && threadIdx.x < kWave) {
    if (lane < E) offsets[lane] = group0;
    if (lane == 0) offsets[E] = kept_total;
    float term = 0.f;
    if (lane < E) {
      const float u = lb_mode == BTX_LB_TOKEN_FRAC ? (float)cnt / ((float)T * (float)k) : gate_sum[lane] / (float)T;
      term = u * (prob_sum[lane] / (float)T);
    }
    float loss = 0.f;
    for (int e = 0; e < E; ++e) loss += __shfl(term, e, kWave);   // expert order
    if (lane == 0) *lb_loss = lb_alpha * (float)E * loss;
  }
  // grouped rows past the kept ones do not exist; whoever indexes through perm there
  // (kernels that run over all T*k rows) must still find a valid pair
  for (int64_t r = (int64_t)kept_total + blockIdx.x * blockDim.x + threadIdx.x; r < (int64_t)T * k;
       r += (int64_t)gridDim.x * blockDim.x)
    perm[r] = 0;

  const int b = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;  // one wavefront per token block
  if (b >= nblk) return;
  const int first = b * kTokPerBlock * k;
  const int last = min((b + 1) * kTokPerBlock, T) * k;
  // entry e: rank, inside expert e's pairs, of the next pair of this block.  The lanes of the same expert are found with a
  // ballot per index bit and their first one moves the entry on (a wavefront's LDS operations stay in order); with a ballot and
  // two shuffles for every expert the kernel took 15 us for 1501 tokens and 64 experts, top-8, now 6.5.
  __shared__ int s_next[kWavesPerBlock][kMaxExperts];
  volatile int* next = s_next[threadIdx.x / kWave];
  next[lane] = lane < E ? blk_base[(size_t)b * E + lane] : 0;
  for (int i0 = first; i0 < last; i0 += kWave) {
    const int i = i0 + lane;
    const bool valid = i < last;
    const int e = valid ? topk_idx[i] : 0;
    unsigned long long same = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 6; ++bit) {
      const unsigned long long ones = __ballot((e >> bit) & 1);
      same &= (e >> bit) & 1 ? ones : ~ones;
    }
    const int before = __popcll(same & ((1ull << lane) - 1ull)), base = __shfl(group0, e, kWave);
    const int start = next[e], rank = start + before;
    if (valid && before == 0) next[e] = start + __popcll(same);
    if (valid) {
      if (cap > 0 && rank >= cap) {
        inv_pos[i] = -1;               // beyond the expert's capacity: dropped
      } else {
        const int pos = base + rank;
        perm[pos] = i;
        inv_pos[i] = pos;
      }
    }
  }
}

// W_router [d,E] -> [E,d]
__global__ __launch_bounds__(256) void transpose_wr_kernel(const float* __restrict__ Wr, int d, int E,
                                                           float* __restrict__ WrT) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d * E) return;
  const int e = i / d, c = i - e * d;
  WrT[i] = Wr[(size_t)c * E + e];
}
// W_router [d,E] in the order in which the matrix-core logits take it: 32 columns, of these the first four of every 8 and then the
// others, 16 experts, 8 columns, expert, column; the last 32 columns and the last 16 experts are what is left.  A wavefront's load
// is then one piece of 1 KB: from [E,d] it touched 16 lines at 64 places, and those lookups were what the kernel took its time for.
// Routing as a whole, us, [E,d] / like this: 1501 tokens of 4096 columns, 64 experts 67 / 50; 700 of 512 37 / 30; 2000 of 1024, 16 experts 24.8 /
// 22.0; 16384 of 4096, 32 experts 95 / 91; 5000 of 1032, 33 experts 48.6 / 50; fp32 4500 of 4096, 64 experts 87 / 78.
__global__ __launch_bounds__(256) void wr_fragments_kernel(const float* __restrict__ Wr, int d, int E, float* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d * E) return;
  const int p0 = i / (32 * E) * 32, chunks = min((d - p0) / 8, 4);
  int r = i - p0 * E;
  const int half = r / (chunks * 4 * E);
  r -= half * chunks * 4 * E;
  const int set = r / (64 * chunks), of_set = min(E - 16 * set, 16);
  r -= set * 64 * chunks;
  const int chunk = r / (4 * of_set), e = 16 * set + r / 4 % of_set;
  out[i] = Wr[(size_t)(p0 + 8 * chunk + 4 * half + r % 4) * E + e];
}

// Logits of more than 8 experts go to the matrix cores, of rows that are as they are.
bool matrix_logits(const RouteArgs& a) { return a.E > 8 && !a.gain; }

// Wavefronts of a route_tokens workgroup.  4 while the workgroups alone fill the chip (kFewBlocks).  With fewer of them every
// row's latency shows, and 8 or 16 split the same 16 tokens; but every wavefront reads all of W_router, and that traffic
// decides wherever W_router is large or two workgroups share a compute unit.  us with 4 / 8 / 16:
//   plain, up to 256 blocks: bf16 1500 tokens of 4096 columns, 8 experts 32 / 27 / 34, of 8192 41 / 36 / 49; more: 4500 of
//   4096 34 / 38 / 54, of 8192 49 / 56 / 86; fp32 4500 of 2048 31 / 31 / 39, 8000 37 / 33 / 41, 4500 of 8192 60 / 68 / 96
//   normalising, bf16: 4001 of 4096, 4 experts 55 / 43 / 39, 64 experts 281 / 197 / 213; of 512, 64 experts 87 / 64 / 60; 4500
//   of 4096, 4 experts 58 / 49 / 57, 64 experts 303 / 256 / 366
//   normalising, fp32: 1500 of 4096, 64 experts 152 / 136 / 193; of 512 70 / 56 / 55; of 16384, 8 experts 110 / 105 / 142, 4001
//   187 / 208 / 270; 4500 of 512, 64 experts 80 / 71 / 83, of 4096 235 / 263 / 392
// Logits on the matrix cores: 8 wavefronts that share W_router's columns, for one block of tokens instead of kMatrixGroups.
// 4001 tokens of 4096 columns, 64 experts 67 -> 44 us; past one workgroup on a compute unit few experts of few columns 4500 of 1024, 16
// experts 30 -> 24, of 2048, 32 experts 38 -> 33, and wide rows, where 4 wavefronts wait longer for every piece of a row: 4600 of 4608, 16
// experts 43 -> 36, 28 experts 51 -> 47; of 10240 62 -> 54, 78 -> 74; 7000 of 16384, 12 experts 105 -> 90, but 24 experts 114 -> 115; fp32 5000
// of 6144, 12 experts 61 -> 55, 24 experts 64 -> 67, of 16384 119 -> 113, 126 -> 139.  (More than 65536 weights of up to 4096 columns gain as well,
// 4500 tokens, 32 experts 48 -> 44; left as they are.)
constexpr int kFewBlocks = 512, kComputeUnits = 256;
int token_waves(int nblk, int d, int E, bool f32, bool norm) {
  if (nblk >= kFewBlocks) return kWavesPerBlock;
  if (nblk <= kComputeUnits) {
    if (f32 && d > 8192) return kWavesPerBlock;
    return norm && (f32 ? d <= 512 : d <= 1024 || E <= 4) ? 16 : 8;
  }
  return (f32 ? d <= 4096 && d * E <= 32768 : norm) ? 8 : kWavesPerBlock;
}
bool matrix_few(int nblk, int d, int E, bool f32) {
  if (nblk <= kComputeUnits) return true;
  if (nblk >= kFewBlocks || E > 32) return false;
  return d * E <= 65536 || (d > 4096 && (E <= 16 || (!f32 && d <= 10240)));
}

template <typename XT>
void launch_tokens(const RouteArgs& a, const float* WrT, int nblk, int32_t* bc, float* bg, float* bp, hipStream_t s) {
  const XT* x = static_cast<const XT*>(a.x);
  const int waves = token_waves(nblk, a.d, a.E, std::is_same<XT, float>::value, a.gain != nullptr);
#define BTX_ROUTE_LAUNCH(EC)                                      \
  do {                                                            \
    if (waves == 16) BTX_ROUTE_LAUNCH_NW(EC, 16);                 \
    else if (waves == 8) BTX_ROUTE_LAUNCH_NW(EC, 8);              \
    else BTX_ROUTE_LAUNCH_NW(EC, kWavesPerBlock);                 \
  } while (0)
#define BTX_ROUTE_LAUNCH_NW(EC, NW)                                                                                \
  do {                                                                                                             \
    if (a.gain)                                                                                                    \
      route_tokens_kernel<XT, EC, true, NW><<<nblk, NW * kWave, 0, s>>>(                                                    \
          x, WrT, a.b_router, a.U, a.T, a.d, a.E, a.k, a.route_mode, 1.f / a.tau, a.topk_idx, a.gates, a.probs, bc,  \
          bg, bp, a.gain, a.eps, static_cast<XT*>(a.xn), a.rstd);                                                   \
    else                                                                                                           \
      route_tokens_kernel<XT, EC, false, NW><<<nblk, NW * kWave, 0, s>>>(                                                \
          x, WrT, a.b_router, a.U, a.T, a.d, a.E, a.k, a.route_mode, 1.f / a.tau, a.topk_idx, a.gates, a.probs, bc,  \
          bg, bp, nullptr, 0.f, nullptr, nullptr);                                                                  \
  } while (0)
  if (matrix_logits(a)) {
    // many experts: the dot products go to the matrix cores (fp32 16x16x4, 1024 multiply-adds per
    // instruction).  On the vector unit they took 172 us for 16384 tokens x 32 experts (64 M vector
    // instructions); the kernel now takes 79 us
    auto go_nw = [&](auto nw, auto mg, auto ns) {
      constexpr int NW = decltype(nw)::value, MG = decltype(mg)::value, NS = decltype(ns)::value;
      const size_t lds = (size_t)NW * MG * kTokPerBlock * 16 * NS * sizeof(float);
      route_tokens_kernel<XT, 0, false, NW, MG, NS><<<ceil_div(nblk, MG), NW * kWave, lds, s>>>(
          x, WrT, a.b_router, a.U, a.T, a.d, a.E, a.k, a.route_mode, 1.f / a.tau, a.topk_idx, a.gates, a.probs, bc,
          bg, bp, nullptr, 0.f, nullptr, nullptr);
    };
    using std::integral_constant;
    auto go = [&](auto ns) {
      if (matrix_few(nblk, a.d, a.E, std::is_same<XT, float>::value)) go_nw(integral_constant<int, 8>{}, integral_constant<int, 1>{}, ns);
      else go_nw(integral_constant<int, kWavesPerBlock>{}, integral_constant<int, kMatrixGroups>{}, ns);
    };
    if (a.E <= 16) go(integral_constant<int, 1>{});
    else if (a.E <= 32) go(integral_constant<int, 2>{});
    else if (a.E <= 48) go(integral_constant<int, 3>{});
    else go(integral_constant<int, 4>{});
    return;
  }
  if (a.E <= 1) BTX_ROUTE_LAUNCH(1);
  else if (a.E <= 2) BTX_ROUTE_LAUNCH(2);
  else if (a.E <= 4) BTX_ROUTE_LAUNCH(4);
  else BTX_ROUTE_LAUNCH(8);   // 16 per pass was measured no faster at E = 32
#undef BTX_ROUTE_LAUNCH
#undef BTX_ROUTE_LAUNCH_NW
}

}  // namespace

// WrT: what route_tokens reads, [E,d] or fragments
static int launch_transpose_wr(const RouteArgs& a, float* WrT, hipStream_t s) {
  const int d = a.d, E = a.E;
  if ((int64_t)d * E >= (int64_t)1 << 31) return BTX_ERR_UNSUPPORTED;   // the kernels index W_router with 32 bits
  if (matrix_logits(a)) wr_fragments_kernel<<<ceil_div(d * E, 256), 256, 0, s>>>(a.W_router, d, E, WrT);
  else transpose_wr_kernel<<<ceil_div(d * E, 256), 256, 0, s>>>(a.W_router, d, E, WrT);
  BTX_LAUNCH_CHECK();
  return BTX_OK;
}

static int num_blocks(int T) { return ceil_div(T, kTokPerBlock); }
static size_t block_stats_bytes(int T, int E) {
  // block counts, block bases (int32) and block gate/prob sums (fp32)
  return align_up((size_t)num_blocks(T) * E * 4 * sizeof(int32_t), 256);
}

size_t route_workspace_bytes(int T, int d, int E, int /*k*/) {
  return block_stats_bytes(T, E) + align_up((size_t)E * d * sizeof(float), 256);   // + W_router transposed
}

int launch_route(const RouteArgs& a, hipStream_t s) {
  if (route_is_small(a)) return launch_route_small(a, s);
  const int nblk = num_blocks(a.T);
  const size_t n = (size_t)nblk * a.E;
  int32_t* bc = static_cast<int32_t*>(a.workspace);
  int32_t* bb = bc + n;
  float* bg = reinterpret_cast<float*>(bb + n);
  float* bp = bg + n;
  float* WrT = reinterpret_cast<float*>(static_cast<char*>(a.workspace) + block_stats_bytes(a.T, a.E));
  if (int rc = launch_transpose_wr(a, WrT, s)) return rc;
  if (a.x_dtype == BTX_BF16) launch_tokens<bf16_t>(a, WrT, nblk, bc, bg, bp, s);
  else launch_tokens<float>(a, WrT, nblk, bc, bg, bp, s);
  BTX_LAUNCH_CHECK();
  route_scan_kernel<<<a.E, kScanThreads, 0, s>>>(nblk, a.E, bc, bg, bp, bb, a.counts, a.gate_sum, a.prob_sum);
  BTX_LAUNCH_CHECK();
  route_scatter_kernel<<<ceil_div(nblk, kWavesPerBlock), kWavesPerBlock * kWave, 0, s>>>(
      nblk, a.T, a.E, a.k, a.cap, a.lb_mode, a.lb_alpha, a.topk_idx, bb, a.counts, a.gate_sum, a.prob_sum, a.offsets,
      a.lb_loss, a.perm, a.inv_pos);
  BTX_LAUNCH_CHECK();
  return BTX_OK;
}

}  // namespace btx
