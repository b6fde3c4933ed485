// Backward of the router and the last step of dX (chain rule on the routing function of
// Sec. 3.2 / 3.3 with the expert selection held fixed, plus the gradient of the
// load-balancing loss of Sec. 3.3).  All reductions run in a fixed order; no atomics.
//
//   router_ds       one wavefront per token, lane e = expert e: dg (summed partials of
//                   <dY, expert output>), gate Jacobian, load-balancing term -> ds[T,E]; in batches that are not
//                   large part of the weight gradients' launch (see router_ds_rides())
//   dwr_partial     dW_router = x^T ds as per-token-chunk partial sums
//   dx_finish       dX[t] = sum_j dxs[inv_pos[t,j]] + ds[t] W_router^T, W_router slice kept in registers; in batches that are not
//                   large one launch with dwr_partial (dx_and_dwr)
//   dwr_reduce      fixed-order sum of the partials (and of db_router)
// The rows these kernels stream (x, dxs, dX) are touched once per kernel and go past the caches.
// dwr_partial and dx_finish work expert-major (partials [chunk][E][d], W_router as [E,d]): a
// lane's 8 columns of one expert are then 32 contiguous bytes instead of 8 pieces E floats apart.
#include "common.h"
#include "router_ds.h"

namespace btx {
namespace {

constexpr int kColsPerThread = 8;

__global__ __launch_bounds__(256) void router_ds_kernel(RouterDs a) { router_ds(a, blockIdx.x); }

// grid: (token chunks of CHUNK, column blocks of 256*8, expert passes of KEC).  The partial sums
// are stored expert-major ([chunk][E][d]): a thread's 8 columns of an expert are 32 contiguous bytes.
template <typename XT, int KEC, int CHUNK>
__global__ __launch_bounds__(256) void dwr_partial_kernel(const XT* __restrict__ x, const float* __restrict__ ds, int T,
                                                          int d, int E, float* __restrict__ part,
                                                          float* __restrict__ db_part) {
  __shared__ float s_ds[CHUNK][KEC];
  const int t0 = blockIdx.x * CHUNK, e0 = blockIdx.z * KEC;
  const int nt = min(CHUNK, T - t0);
  for (int i = threadIdx.x; i < CHUNK * KEC; i += 256) {
    const int q = i / KEC, j = i % KEC;
    s_ds[q][j] = (q < nt && e0 + j < E) ? ds[(size_t)(t0 + q) * E + e0 + j] : 0.f;
  }
  __syncthreads();
  const int c0 = (blockIdx.y * 256 + threadIdx.x) * kColsPerThread;
  if (c0 < d) {
    float acc[KEC][kColsPerThread] = {};
    // 4 token rows in flight; rows past the chunk's end are read from a clamped address and
    // meet the zeros of s_ds
    for (int q = 0; q < nt; q += 4) {
      float xv[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) RowVec<XT, 8>::ld_stream(x + (size_t)min(t0 + q + u, T - 1) * d + c0, xv[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < KEC; ++j) {
          const float w = s_ds[q + u][j];
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[j][i] = fmaf(xv[u][i], w, acc[j][i]);
        }
    }
#pragma unroll
    for (int j = 0; j < KEC; ++j)
      if (e0 + j < E) RowVec<float, 8>::st(part + ((size_t)blockIdx.x * E + e0 + j) * d + c0, acc[j]);
  }
  if (blockIdx.y == 0 && threadIdx.x < KEC && e0 + threadIdx.x < E) {
    float a = 0.f;
    for (int q = 0; q < nt; ++q) a += s_ds[q][threadIdx.x];
    db_part[(size_t)blockIdx.x * E + e0 + threadIdx.x] = a;
  }
}

// The same sums with the WAVES wavefronts of a workgroup on the same 512 columns and their share of the chunk's tokens each,
// added in wavefront order: as many times the rows in flight and the workgroups, for batches whose (chunk, column
// block, expert pass) grid would leave the chip idle (fewer than kFewBlocks: 1501 tokens of 4096 columns, 64 experts 65 ->
// 27 us; 4001 of 2048, 8 experts 29 -> 12).
constexpr int kFewBlocks = 512;
template <int KEC, int CHUNK> constexpr int dwr_few_lds_bytes() { return (CHUNK * KEC + KEC * 8 * kWave) * (int)sizeof(float); }
template <typename XT, int KEC, int CHUNK, int WAVES>
__device__ __forceinline__ void dwr_partial_few(const XT* __restrict__ x, const float* __restrict__ ds, int T, int d, int E,
                                                float* __restrict__ part, float* __restrict__ db_part, float* __restrict__ dWr,
                                                float* __restrict__ db, int chunk, int cols, int pass, float* smem) {
  float (*s_ds)[KEC] = reinterpret_cast<float (*)[KEC]>(smem);                  // [CHUNK][KEC]
  f32x4 (*s_acc)[kWave] = reinterpret_cast<f32x4 (*)[kWave]>(smem + CHUNK * KEC);    // [KEC * 2][kWave]
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int t0 = chunk * CHUNK, e0 = pass * KEC;
  const int nt = min(CHUNK, T - t0);
  for (int i = threadIdx.x; i < CHUNK * KEC; i += WAVES * kWave) {
    const int q = i / KEC, j = i % KEC;
    s_ds[q][j] = (q < nt && e0 + j < E) ? ds[(size_t)(t0 + q) * E + e0 + j] : 0.f;
  }
  __syncthreads();
  const int c0 = (cols * kWave + lane) * kColsPerThread, cc = min(c0, d - kColsPerThread);
  float acc[KEC][kColsPerThread] = {};
  constexpr int U = WAVES == 4 ? 4 : 2;                 // rows in flight: more do not fit the registers of 16 wavefronts
  const int share = (nt + 4 * WAVES - 1) / (4 * WAVES) * 4;               // of the tokens there are, whole groups of four
  for (int q = wave * share; q < min(nt, (wave + 1) * share); q += U) {   // rows past the end meet the zeros of s_ds
    float xv[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) RowVec<XT, 8>::ld_stream(x + (size_t)min(t0 + q + u, T - 1) * d + cc, xv[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < KEC; ++j) {
        const float w = s_ds[q + u][j];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[j][i] = fmaf(xv[u][i], w, acc[j][i]);
      }
  }
  for (int w = 1; w < WAVES; ++w) {
    if (wave == w) {
#pragma unroll
      for (int j = 0; j < KEC; ++j) {
        s_acc[2 * j][lane] = f32x4{acc[j][0], acc[j][1], acc[j][2], acc[j][3]};
        s_acc[2 * j + 1][lane] = f32x4{acc[j][4], acc[j][5], acc[j][6], acc[j][7]};
      }
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int j = 0; j < KEC; ++j) {
        const f32x4 u = s_acc[2 * j][lane], v = s_acc[2 * j + 1][lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) { acc[j][i] += u[i]; acc[j][4 + i] += v[i]; }
      }
    }
    __syncthreads();
  }
  if (wave == 0 && c0 < d) {
#pragma unroll
    for (int j = 0; j < KEC; ++j) {
      if (e0 + j >= E) continue;
      if (dWr) {                                        // the only chunk: its sums are the result
#pragma unroll
        for (int i = 0; i < 8; ++i) dWr[(size_t)(c0 + i) * E + e0 + j] = acc[j][i];
      } else {
        RowVec<float, 8>::st(part + ((size_t)chunk * E + e0 + j) * d + c0, acc[j]);
      }
    }
  }
  if (cols == 0 && threadIdx.x < KEC && e0 + threadIdx.x < E) {
    float b = 0.f;
    for (int q = 0; q < nt; ++q) b += s_ds[q][threadIdx.x];
    if (dWr) {
      if (db) db[e0 + threadIdx.x] = b;
    } else {
      db_part[(size_t)chunk * E + e0 + threadIdx.x] = b;
    }
  }
}

template <typename XT, int KEC, int CHUNK>
__global__ __launch_bounds__(256) void dwr_partial_few_kernel(const XT* __restrict__ x, const float* __restrict__ ds, int T, int d, int E,
                                                              float* __restrict__ part, float* __restrict__ db_part,
                                                              float* __restrict__ dWr, float* __restrict__ db) {
  __shared__ __attribute__((aligned(16))) float smem[dwr_few_lds_bytes<KEC, CHUNK>() / sizeof(float)];
  dwr_partial_few<XT, KEC, CHUNK, 4>(x, ds, T, d, E, part, db_part, dWr, db, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}

// 64 sums per block, taken in the partials' expert-major order (coalesced reads) and written to
// dW_router's [d,E] place; 16 thread groups each add every 16th partial, then the 16 sums are
// added in group order (a fixed order, like everything else here).
constexpr int kRedGroups = 16;
__global__ __launch_bounds__(64 * kRedGroups) void dwr_reduce_kernel(const float* __restrict__ part,
                                                                      const float* __restrict__ db_part, int nchunk,
                                                                      int d, int E, float* __restrict__ dWr,
                                                                      float* __restrict__ db) {
  __shared__ float s_sum[kRedGroups][64];
  const int o = threadIdx.x % 64, grp = threadIdx.x / 64;
  const int dE = d * E;
  const int i = blockIdx.x * 64 + o;
  s_sum[grp][o] = i < dE ? strided_row_sum(part, dE, i, grp, kRedGroups, nchunk) : 0.f;
  __syncthreads();
  if (grp == 0 && i < dE) {
    float a = 0.f;
#pragma unroll
    for (int g = 0; g < kRedGroups; ++g) a += s_sum[g][o];
    const int e = i / d, c = i - e * d;
    dWr[(size_t)c * E + e] = a;
  }
  if (db && blockIdx.x == 0 && threadIdx.x < E) {
    float b = 0.f;
    for (int c = 0; c < nchunk; ++c) b += db_part[(size_t)c * E + threadIdx.x];
    db[threadIdx.x] = b;
  }
}

// dX[t] = sum_j dxs[inv_pos[t,j]] + ds[t] W_router^T.  A wavefront owns 512 columns (8 per lane)
// for TOK tokens, 4 of them in flight at a time; its slice of W_router (read from the [E,d]
// copy, E <= EC) stays in registers, so the kernel streams dxs and dX and little else.
template <typename XT, int EC, int TOK>
__device__ __forceinline__ void dx_finish(const XT* __restrict__ dxs, const int32_t* __restrict__ inv_pos, const float* __restrict__ ds,
                                          const float* __restrict__ WrT, int T, int d, int E, int k, XT* __restrict__ dX, int tokens, int cols) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int c0 = ((cols * 4 + wave) * kWave + lane) * 8;
  const int t0 = tokens * TOK;
  if (c0 >= d) return;                      // no cross-lane traffic below
  float wr[EC][8];
#pragma unroll
  for (int j = 0; j < EC; ++j) {
    if (j < E) {
      RowVec<float, 8>::ld(WrT + (size_t)j * d + c0, wr[j]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) wr[j][i] = 0.f;
    }
  }
  for (int tq = 0; tq < TOK; tq += 4) {
    float acc[4][8] = {};
    // slot by slot, the four tokens' rows in flight together; a dropped pair (or a token past
    // the end) reads row 0 and adds zero
#pragma unroll 2
    for (int j = 0; j < k; ++j) {
      float v[4][8];
      bool have[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = t0 + tq + q;
        const int r = t < T ? inv_pos[(size_t)t * k + j] : -1;
        have[q] = r >= 0;
        RowVec<XT, 8>::ld_stream(dxs + (size_t)max(r, 0) * d + c0, v[q]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[q][i] += have[q] ? v[q][i] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + tq + q;
      if (t >= T) break;
#pragma unroll
      for (int j = 0; j < EC; ++j) {
        const float w = j < E ? ds[(size_t)t * E + j] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[q][i] = fmaf(w, wr[j][i], acc[q][i]);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (t0 + tq + q < T) RowVec<XT, 8>::st_stream(dX + (size_t)(t0 + tq + q) * d + c0, acc[q]);
  }
}

// The same for more than 8 experts, where the slice of W_router no longer fits the registers and reloading it
// per 4 tokens (from the caches) cost 110 of the kernel's 337 us at 32 experts: the 8 wavefronts of a
// workgroup share one slice of kDxCols columns, staged once in LDS ([expert][half][lane] 16-byte
// pieces, so that consecutive lanes read consecutive pieces), and split the workgroup's tokens, 4 in flight per
// wavefront.  More than kDxLdsE experts take turns in the same 64 KB, for one pass of 32 tokens per workgroup.  1501
// tokens of 4096 columns, 64 experts, 8 slots: 152 us reloading, 44 now.
constexpr int kDxLdsE = 32;                             // 32 experts x 512 columns x 4 bytes = 64 KB
constexpr int kDxCols = kWave * 8;                      // columns of a workgroup: 8 per lane
constexpr int kDxWaves = 8;
template <typename XT>
__device__ __forceinline__ void dx_finish_lds(const XT* __restrict__ dxs, const int32_t* __restrict__ inv_pos, const float* __restrict__ ds,
                                              const float* __restrict__ WrT, int T, int d, int E, int k, int tok_per_block,
                                              XT* __restrict__ dX, int tokens, int cols, float* smem) {
  f32x4* const s_wr = reinterpret_cast<f32x4*>(smem);   // [min(E, kDxLdsE)][2][kWave]
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int cb = cols * kDxCols, c0 = cb + lane * 8, cc = min(c0, d - 8);
  auto stage = [&](int e0) {
    for (int i = threadIdx.x; i < min(E - e0, kDxLdsE) * (kDxCols / 4); i += kDxWaves * kWave) {
      const int e = i / (kDxCols / 4), c4 = i % (kDxCols / 4);    // 16-byte piece c4 of expert e0 + e's slice
      f32x4 w{0.f, 0.f, 0.f, 0.f};
      if (cb + 4 * c4 < d) w = *reinterpret_cast<const f32x4*>(WrT + (size_t)(e0 + e) * d + cb + 4 * c4);
      s_wr[(e * 2 + (c4 & 1)) * kWave + (c4 >> 1)] = w;
    }
    __syncthreads();
  };
  stage(0);
  const int t_first = tokens * tok_per_block, t_end = min(T, t_first + tok_per_block);
  // every wavefront makes every trip (there are barriers below); tokens past the end and columns past d are not stored
  for (int tb = t_first; tb < t_end; tb += kDxWaves * 4) {
    const int t0 = tb + wave * 4;
    float acc[4][8] = {};
    // slot by slot, the four tokens' rows in flight together; a dropped pair (or a token past
    // the end) reads row 0 and adds zero
#pragma unroll 2
    for (int j = 0; j < k; ++j) {
      float v[4][8];
      bool have[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = t0 + q;
        const int r = t < t_end ? inv_pos[(size_t)t * k + j] : -1;
        have[q] = r >= 0;
        RowVec<XT, 8>::ld_stream(dxs + (size_t)max(r, 0) * d + cc, v[q]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[q][i] += have[q] ? v[q][i] : 0.f;
    }
    for (int e0 = 0; e0 < E; e0 += kDxLdsE) {
      if (e0 > 0) {                                     // only with one trip per workgroup (tok_per_block = 32)
        __syncthreads();                                // everybody is done with the slice in place
        stage(e0);
      }
      for (int e = 0; e < min(E - e0, kDxLdsE); ++e) {
        const f32x4 wa = s_wr[(e * 2) * kWave + lane], wb = s_wr[(e * 2 + 1) * kWave + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float w = ds[(size_t)min(t0 + q, T - 1) * E + e0 + e];   // uniform across the wavefront
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[q][i] = fmaf(w, wa[i], acc[q][i]);
            acc[q][4 + i] = fmaf(w, wb[i], acc[q][4 + i]);
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (t0 + q < t_end && c0 < d) RowVec<XT, 8>::st_stream(dX + (size_t)(t0 + q) * d + c0, acc[q]);
  }
}

// Both read ds and nothing of each other: one launch, whose first dx_blocks workgroups finish dX (dx_x of them to a column block) and
// whose others sum dW_router's partials (chunks x column blocks x expert passes of them; none where a kernel of its own does).
// In two launches one waited for the other's last workgroups, and small ones for their launch.  The router's whole backward pass,
// us, two launches / one: 500 tokens of 512, 4 experts 22.4 / 17.7; 100 of 1000, 16 experts 38.4 / 21.2; 300 of 4096, 4 experts 26.8
// / 17.8; 1501 of 4096, 64 experts 87 / 78; 4001 of 2048, 8 experts 46.9 / 36.2.
template <typename XT, int EC, int TOK>
__global__ __launch_bounds__(256) void dx_and_dwr_kernel(
    const XT* __restrict__ dxs, const int32_t* __restrict__ inv_pos, const float* __restrict__ ds, const float* __restrict__ WrT, int T,
    int d, int E, int k, XT* __restrict__ dX, int dx_blocks, int dx_x, const XT* __restrict__ x, float* __restrict__ part,
    float* __restrict__ db_part, float* __restrict__ dWr, float* __restrict__ db, int chunks) {
  __shared__ __attribute__((aligned(16))) float smem[dwr_few_lds_bytes<8, 64>() / sizeof(float)];
  const int b = blockIdx.x, p = b - dx_blocks;
  if (b < dx_blocks) dx_finish<XT, EC, TOK>(dxs, inv_pos, ds, WrT, T, d, E, k, dX, b % dx_x, b / dx_x);
  else dwr_partial_few<XT, 8, 64, 4>(x, ds, T, d, E, part, db_part, dWr, db, p % chunks, p / chunks, 0, smem);
}
// dX alone, of large batches: 126 registers in bf16 up to 4 experts, so 4 wavefronts on a SIMD, where the other has 133 and 18 KB of LDS
// (16384 tokens of 4096, 4 experts: the router's backward pass 144.3 us with that one, 141.3 with this; Switch 122.5 / 120.7).
template <typename XT, int EC, int TOK>
__global__ __launch_bounds__(256) void dx_finish_kernel(const XT* __restrict__ dxs, const int32_t* __restrict__ inv_pos,
                                                        const float* __restrict__ ds, const float* __restrict__ WrT, int T, int d, int E,
                                                        int k, XT* __restrict__ dX, int dx_x) {
  dx_finish<XT, EC, TOK>(dxs, inv_pos, ds, WrT, T, d, E, k, dX, blockIdx.x % dx_x, blockIdx.x / dx_x);
}
template <typename XT>
__global__ __launch_bounds__(kDxWaves* kWave) void dx_finish_lds_kernel(
    const XT* __restrict__ dxs, const int32_t* __restrict__ inv_pos, const float* __restrict__ ds, const float* __restrict__ WrT, int T,
    int d, int E, int k, int tok_per_block, XT* __restrict__ dX, int dx_x) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  dx_finish_lds<XT>(dxs, inv_pos, ds, WrT, T, d, E, k, tok_per_block, dX, blockIdx.x % dx_x, blockIdx.x / dx_x, lds);
}
template <typename XT>
__global__ __launch_bounds__(kDxWaves* kWave, 4) void dx_and_dwr_lds_kernel(
    const XT* __restrict__ dxs, const int32_t* __restrict__ inv_pos, const float* __restrict__ ds, const float* __restrict__ WrT, int T,
    int d, int E, int k, int tok_per_block, XT* __restrict__ dX, int dx_blocks, int dx_x, const XT* __restrict__ x,
    float* __restrict__ part, float* __restrict__ db_part, float* __restrict__ dWr, float* __restrict__ db, int chunks, int cols) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int b = blockIdx.x, p = b - dx_blocks;
  if (b < dx_blocks) dx_finish_lds<XT>(dxs, inv_pos, ds, WrT, T, d, E, k, tok_per_block, dX, b % dx_x, b / dx_x, lds);
  else dwr_partial_few<XT, 8, 128, kDxWaves>(x, ds, T, d, E, part, db_part, dWr, db, p % chunks, p / chunks % cols, p / (chunks * cols), lds);
}

}  // namespace

// token chunk of the dW_router partial sums: longer chunks for many experts keep the partials
// (chunks * d * E floats) small next to x
static int tok_chunk(int E) { return E <= 8 ? 64 : 128; }
static int n_chunks(int T, int E) { return ceil_div(T, tok_chunk(E)); }

size_t router_bwd_workspace_bytes(int T, int d, int E) {
  const size_t ds = align_up((size_t)T * E * sizeof(float), 256);
  const size_t part = align_up((size_t)n_chunks(T, E) * d * E * sizeof(float), 256);
  const size_t dbp = align_up((size_t)n_chunks(T, E) * E * sizeof(float), 256);
  const size_t wrt = align_up((size_t)E * d * sizeof(float), 256);
  return ds + part + dbp + wrt;
}

namespace {
struct Parts { float *ds, *part, *dbp, *WrT; };
Parts parts_of(const RouterBwdArgs& a) {
  const int nch = n_chunks(a.T, a.E);
  char* w = static_cast<char*>(a.workspace);
  Parts p;
  p.ds = reinterpret_cast<float*>(w);
  w += align_up((size_t)a.T * a.E * sizeof(float), 256);
  p.part = reinterpret_cast<float*>(w);
  w += align_up((size_t)nch * a.d * a.E * sizeof(float), 256);
  p.dbp = reinterpret_cast<float*>(w);
  w += align_up((size_t)nch * a.E * sizeof(float), 256);
  p.WrT = reinterpret_cast<float*>(w);
  return p;
}
}  // namespace

// More than 8 experts: the partial sums beside dX, or in a launch of their own with 16 experts to a pass?  Beside it they read x once
// for every 8 experts, and fill what dX's last round of workgroups (two on a compute unit) leaves idle.  What is read again costs more
// than that from about 84 MB of fp32 rows or 144 MB of bf16 ones on, and a long launch gains nothing where that round is nearly full by
// itself.  Of 232 shapes (9 to 64 experts, 64 to 4096 columns) this leaves 0.2 % on average to the better form, 7 % at most; always beside: 2.4
// and 28 %.  The router's backward pass, us, a launch of its own / beside:
//   4096 columns: 609 tokens fp32, 33 experts 48 / 27; 1410, 48 experts 65 / 57; 2013, 64 experts (504 workgroups) 71 / 75, 2069 (520) 118 / 94
//   3072: 3122 tokens, 64 experts 104 / 89;  2048: 6563, 12 experts 57 / 48; fp32 3200, 64 experts (105 MB) 88 / 94; 10701, 32 (175 MB) 127 / 154
//   1032: 13616 tokens, 24 experts (1278) 122 / 106;  256: 19822, 32 experts 104 / 95; 65408, 12 experts (2044) 153 / 159
constexpr int kDxRound = 512, kDxNearlyFull = 470, kShortBlocks = 1536;
static bool dwr_beside_dx(const RouterBwdArgs& a, int64_t dx_blocks, int64_t blocks) {
  const bool f32 = a.dtype == BTX_F32;
  const int64_t last = dx_blocks % kDxRound, again = (int64_t)a.T * a.d * (f32 ? 4 : 2) * (ceil_div(a.E, 8) - ceil_div(a.E, 16));
  return again <= (f32 ? 84000000 : 144000000) && (blocks <= kShortBlocks || (last > 0 && last <= kDxNearlyFull));
}

RouterDs router_ds_args(const RouterBwdArgs& a) {
  const Parts p = parts_of(a);
  int slots_log2 = 0;                                   // a power of two of lanes for a token's slots
  while ((1 << slots_log2) < a.k) ++slots_log2;
  return RouterDs{a.W_router, a.d, p.WrT, a.T, a.E, a.k, a.route_mode, a.lb_mode, a.lb_alpha, a.lb_grad_scale, a.flags, a.noise,
                  a.noise ? 1.f / a.tau : 1.f, a.topk_idx, a.gates, a.probs, a.inv_pos, a.gate_sum, a.prob_sum, a.counts, a.dg_part,
                  a.n_part, slots_log2, p.ds};
}

int launch_router_bwd(const RouterBwdArgs& a, bool ds_done, hipStream_t s) {
  const int nch = n_chunks(a.T, a.E);
  const Parts w = parts_of(a);
  float *const ds = w.ds, *const part = w.part, *const dbp = w.dbp, *const WrT = w.WrT;

  if ((int64_t)a.d * a.E >= (int64_t)1 << 31) return BTX_ERR_UNSUPPORTED;   // the kernels index W_router with 32 bits
  if (!ds_done) {
    const RouterDs rd = router_ds_args(a);
    router_ds_kernel<<<router_ds_blocks(rd), 256, 0, s>>>(rd);
    BTX_LAUNCH_CHECK();
  }
  const int passes = ceil_div(a.E, a.E <= 8 ? 8 : 16);
  const bool few = (int64_t)nch * ceil_div(a.d, 256 * kColsPerThread) * passes < kFewBlocks;
  const bool reduce = nch > 1 || !few;                  // a single chunk's sums need no further kernel
  float *const dWr = reduce ? nullptr : a.dW_router, *const db = reduce ? nullptr : a.db_router;
  const int few_cols = ceil_div(a.d, kWave * kColsPerThread), dwr_blocks = few ? nch * few_cols * ceil_div(a.E, 8) : 0;   // beside dX
  auto typed = [&](auto tag) -> int {
    using XT = decltype(tag);
    const XT *const x = static_cast<const XT*>(a.x), *const dxs = static_cast<const XT*>(a.dxs);
    XT* const dX = static_cast<XT*>(a.dX);
    if (!few) {
      const dim3 grid(nch, ceil_div(a.d, 256 * kColsPerThread), passes);
      if (a.E <= 8) dwr_partial_kernel<XT, 8, 64><<<grid, 256, 0, s>>>(x, ds, a.T, a.d, a.E, part, dbp);
      else dwr_partial_kernel<XT, 16, 128><<<grid, 256, 0, s>>>(x, ds, a.T, a.d, a.E, part, dbp);
      BTX_LAUNCH_CHECK();
    }
    if (a.E <= 8) {
      const int cols = ceil_div(a.d, 4 * kWave * 8);
      const int tok = ceil_div(a.T, 16) * cols < kFewBlocks ? 4 : 16;     // tokens of a wavefront
      const int dx_x = ceil_div(a.T, tok);
      const int64_t blocks = (int64_t)dx_x * cols + dwr_blocks;
      if (!grid_fits(blocks, 256)) return BTX_ERR_UNSUPPORTED;
#define BTX_DX_AND_DWR(EC, TOK) dx_and_dwr_kernel<XT, EC, TOK><<<(unsigned)blocks, 256, 0, s>>>(dxs, a.inv_pos, ds, WrT, a.T, a.d, a.E, a.k, dX, dx_x * cols, dx_x, x, part, dbp, dWr, db, nch)
#define BTX_DX(EC) dx_finish_kernel<XT, EC, 16><<<(unsigned)blocks, 256, 0, s>>>(dxs, a.inv_pos, ds, WrT, a.T, a.d, a.E, a.k, dX, dx_x)
      if (!few) { if (a.E <= 4) BTX_DX(4); else BTX_DX(8); }             // as many blocks of x: 16 tokens of a wavefront
      else if (a.E <= 4) { if (tok == 4) BTX_DX_AND_DWR(4, 4); else BTX_DX_AND_DWR(4, 16); }
      else { if (tok == 4) BTX_DX_AND_DWR(8, 4); else BTX_DX_AND_DWR(8, 16); }
#undef BTX_DX
#undef BTX_DX_AND_DWR
    } else {
      // tokens per workgroup, for which the slice is staged once: fewer where the chip would be left idle
      const int cols = ceil_div(a.d, kDxCols);
      const int tok = a.E <= kDxLdsE && ceil_div(a.T, 128) * cols >= kFewBlocks ? 128 : 32;
      const int dx_x = ceil_div(a.T, tok);
      const int64_t dx_blocks = (int64_t)dx_x * cols, blocks = dx_blocks + dwr_blocks;
      if (!grid_fits(blocks, kDxWaves * kWave)) return BTX_ERR_UNSUPPORTED;
      const int lds = std::min(a.E, kDxLdsE) * kDxCols * (int)sizeof(float);
      const bool beside = few && dwr_beside_dx(a, dx_blocks, blocks);
      if (few && !beside) {
        dwr_partial_few_kernel<XT, 16, 128><<<dim3(nch, few_cols, passes), 256, 0, s>>>(x, ds, a.T, a.d, a.E, part, dbp, dWr, db);
        BTX_LAUNCH_CHECK();
      }
      if (beside)
        dx_and_dwr_lds_kernel<XT><<<(unsigned)blocks, kDxWaves * kWave, std::max(lds, dwr_few_lds_bytes<8, 128>()), s>>>(
            dxs, a.inv_pos, ds, WrT, a.T, a.d, a.E, a.k, tok, dX, dx_x * cols, dx_x, x, part, dbp, dWr, db, nch, few_cols);
      else
        dx_finish_lds_kernel<XT><<<(unsigned)dx_blocks, kDxWaves * kWave, lds, s>>>(dxs, a.inv_pos, ds, WrT, a.T, a.d, a.E, a.k, tok, dX, dx_x);
    }
    BTX_LAUNCH_CHECK();
    return BTX_OK;
  };
  if (int rc = a.dtype == BTX_BF16 ? typed(bf16_t{}) : typed(float{})) return rc;
  if (reduce) {
    dwr_reduce_kernel<<<ceil_div(a.d * a.E, 64), 64 * kRedGroups, 0, s>>>(part, dbp, nch, a.d, a.E, a.dW_router,
                                                                         a.db_router);
    BTX_LAUNCH_CHECK();
  }
  return BTX_OK;
}

}  // namespace btx
