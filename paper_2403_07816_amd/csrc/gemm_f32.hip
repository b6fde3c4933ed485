// fp32 grouped GEMMs of the expert FFNs (SwiGLU feed-forward of the seed model, Sec. 4.1, inside the
// layer equation of Sec. 3.2) and of their backward: the same six products as gemm_mfma.hip with fp32
// operands, fp32 matrix instructions (v_mfma_f32_16x16x4_f32: exact products, fp32 sums) and fp32 storage.
//
// The matrix pipe bounds it: 256 FLOP per clock and compute unit, a sixteenth of bf16, while a fragment
// feeds as many output tiles, so LDS and L2 have room to spare.  The tiles are therefore kept simple:
//   * 64 x 64 x 32, 4 wavefronts as 2 x 2, operands global -> registers -> LDS, two LDS stages, the loads of the
//     next two k tiles in flight during a k tile's products, one barrier per k tile; four workgroups per compute unit
//     cover each other's barriers.
//   * within 16 consecutive k a lane of k group g supplies k = 4 g + i to instruction i (the order of k inside
//     a sum is free as long as both operands agree), so that an operand whose k is contiguous in memory is kept
//     as [row][BK] and read 16 bytes at a time; an operand whose k is strided (the weights in UP and DOWN,
//     everything in the dW products) stays as it lies in memory, [BK][columns], and a wavefront's fragments are
//     interleaved columns, one read for all of them.  Pitches of BK + 4 and columns + 8 floats against bank conflicts.
//   * addresses are pointers that move on by a k tile; only a last, partial k tile is masked.
//   * the operands' roles are swapped, so that a lane ends up with 4 consecutive columns of one row.
//   * token rows (x, dY) are read through perm wherever they are an operand, the SwiGLU and its backward are
//     epilogues on the accumulators: nothing is gathered, and no product is stored only to be read again.
// Measured, fwd + bwd of 2003 tokens through 8 experts of 512 x 1376, top-2 (the products 51 GFLOP): with plain FMA
// tiles, gathered operands and separate elementwise kernels 1.64 ms, now 0.60; the products run at 70 to 94 of the
// 153 TFLOP/s this instruction sustains (matrix pipe busy 46 - 66 %): UP 120 us, DOWN 81, BWD_ACT 72, BWD_DX 131 + 5,
// DW13 123, DW2 67.  What is left is ragged rounds of 64 x 64 tiles and the operands' way through registers into LDS.
#include "gemm_f32.h"

#include <algorithm>
#include <type_traits>

namespace btx {
namespace {

enum Mode { UP = 0, DOWN = 1, BWD_ACT = 2, BWD_DX = 3, DW13 = 4, DW2 = 5 };

struct FArgs {
  const float* A0; const float* A1;      // A1: second K pass (BWD_DX)
  const float* B0; const float* B1;      // B1: second panel (UP), second product (DW13), second K pass (BWD_DX)
  float* C0; float* C1; float* C2;       // UP: h1, h3 (NULL: not kept), act; BWD_ACT: dh1, dh3, ga; DW13: dW1, dW3
  const float* H1; const float* H3; const float* gates; float* dg_part; int n_part;   // BWD_ACT
  const int32_t* perm; uint32_t div_mul, div_shift;   // gathered operand: row r is token perm[r] / k
  const int32_t* perm_pairs;             // BWD_ACT: perm, for the gates
  const int32_t* offsets; int E;
  int M, N, K;                           // row-grouped: M unused; grouped along K: K unused
  int lda, ldb, ldc;
  int64_t strideB_e, strideC_e;
  int slices; float* sums; int R;        // DOWN, BWD_DX: K ranges of every tile; their sums [slice][R][N] (slices > 1)
  int tiles_n, tiles_m;                  // column tiles of one product; row tiles of an expert (grouped along K)
  // p / k for 0 <= p < 2^31 without a division (which would cost a third of the vector work of a dW tile):
  // with s = 31 + ceil(log2 k) and div_mul = ceil(2^s / k) < 2^32 the product is off by less than one in 2^31
  __device__ __forceinline__ int token(int p) const { return (int)(((uint64_t)(uint32_t)p * div_mul) >> div_shift); }
  void gather(const RowSource& r) {
    perm = r.perm;
    int l = 0;
    while ((1 << l) < r.k) ++l;
    div_shift = 31 + l;
    div_mul = (uint32_t)((((uint64_t)1 << div_shift) + r.k - 1) / r.k);
  }
};

constexpr int kThreads = 256;
constexpr int kBand = 8;                 // row tiles of a band in the tile order

template <int BM, int BN, int BK, int MODE> struct F32Gemm {
  static constexpr bool GROUP_K = MODE == DW13 || MODE == DW2;
  static constexpr bool A_KC = !GROUP_K, B_KC = MODE == BWD_ACT || MODE == BWD_DX;   // k contiguous in memory
  static constexpr bool A_GATHER = MODE == UP || MODE == BWD_ACT || MODE == DW13, B_GATHER = MODE == DW2;
  static constexpr bool SLICED = MODE == DOWN || MODE == BWD_DX;
  static constexpr bool DUAL = MODE == UP;                       // two B panels side by side in one tile
  static constexpr int BNH = DUAL ? BN / 2 : BN;                 // output columns of a tile
  static constexpr int TM = BM / 32, TN = BN / 32, TNH = DUAL ? TN / 2 : TN;
  static constexpr int A_PITCH = A_KC ? BK + 4 : BM + 8, B_PITCH = B_KC ? BK + 4 : BN + 8;
  static constexpr int A_SIZE = (A_KC ? BM : BK) * A_PITCH, B_SIZE = (B_KC ? BN : BK) * B_PITCH;
  static constexpr int NA = BM * BK / 4 / kThreads, NB = BN * BK / 4 / kThreads;      // 16-byte chunks per thread
  static_assert(NA >= 1 && NB >= 1 && BK % 16 == 0 && (!DUAL || TN % 2 == 0), "tile");

  // One operand of a tile: this thread's chunks of it, fetched to registers and put into LDS.
  // contiguous: chunk (row, 4 k);  strided: chunk (k row, 4 columns).  Rows and columns past the matrix repeat
  // its last ones: their results are never stored.
  template <bool KC, int ROWS_OR_COLS, int PITCH, int NQ, bool GATHER> struct Operand {
    const float* p[NQ];                  // the chunk in the k tile that is fetched next (gathered and strided: its column in row 0)
    int kk[NQ], lds[NQ];                 // k of the chunk inside the tile; its place in LDS
    int src[NQ];                         // gathered and strided: token row of the k row that is fetched next
    f32x4 v[2][NQ];                      // two k tiles in flight
    // the k tile in register set S, of which n_k k exist (the rest becomes zeros), to LDS
    template <int S> __device__ __forceinline__ void put(float* tile, int n_k) {
      if (n_k < BK) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int x = 0; x < 4; ++x) v[S][q][x] = kk[q] < n_k ? v[S][q][x] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) *reinterpret_cast<f32x4*>(tile + lds[q]) = v[S][q];
    }
    static __device__ __forceinline__ void coords(int q, int& major, int& minor) {
      constexpr int PER = (KC ? BK : ROWS_OR_COLS) / 4;
      const int c = threadIdx.x + q * kThreads;
      major = c / PER;
      minor = 4 * (c % PER);
    }
    // rows row0 .. of an operand whose k is contiguous, from k0 on
    __device__ __forceinline__ void rows(const float* base, int row0, int row_end, int ld, const FArgs& g) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        int major, minor;
        coords(q, major, minor);
        const int r = min(row0 + major, row_end - 1);
        p[q] = base + (int64_t)(GATHER ? g.token(g.perm[r]) : r) * ld + minor;
        kk[q] = minor;
        lds[q] = major * PITCH + minor;
      }
    }
    // columns col0 .. of an operand whose k is strided, from row k0 on; DUAL: the second half of them is base2's
    __device__ __forceinline__ void cols(const float* base, const float* base2, int col0, int n, int ld, int k0) {
      constexpr int PANEL = DUAL ? ROWS_OR_COLS / 2 : ROWS_OR_COLS;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        int major, minor;
        coords(q, major, minor);
        const bool second = minor >= PANEL;
        p[q] = (second ? base2 : base) + (GATHER ? (int64_t)0 : (int64_t)(k0 + major) * ld) +
               min(col0 + minor - (second ? PANEL : 0), n - 4);
        kk[q] = major;
        lds[q] = major * PITCH + minor;
      }
    }
    // gathered and strided: look up the token rows of the k tile that is fetched next
    __device__ __forceinline__ void look_up(const FArgs& g, int k0, int k_end) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) src[q] = g.token(g.perm[min(k0 + kk[q], k_end - 1)]);
    }
    // request the next k tile, of which n_k k exist, and move on to the one after it
    template <int S> __device__ __forceinline__ void fetch(int ld, int n_k) {
      if (n_k < BK && !(!KC && GATHER)) {          // the last one of a pass: what lies past its end repeats its first k
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (kk[q] >= n_k) p[q] -= KC ? (int64_t)kk[q] : (int64_t)kk[q] * ld;
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        v[S][q] = *reinterpret_cast<const f32x4*>(p[q] + (!KC && GATHER ? (int64_t)src[q] * ld : (int64_t)0));
      if (!(!KC && GATHER)) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) p[q] += KC ? (int64_t)BK : (int64_t)BK * ld;
      }
    }
  };

  // Fragments of 16 rows (columns) x 16 k: element x of f[i] feeds instruction x, k = 16 s + 4 (lane / 16) + x.
  // contiguous: fragment i is rows base + 16 i + lane % 16; strided: rows base + N (lane % 16) + i, so that one read
  // of N consecutive floats serves all N fragments.
  template <bool KC, int PITCH, int N>
  static __device__ __forceinline__ void frags(const float* tile, int base, int s, int lane, f32x4* f) {
    const int r = lane & 15, k = 16 * s + 4 * (lane >> 4);
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < N; ++i) f[i] = *reinterpret_cast<const f32x4*>(tile + (base + 16 * i + r) * PITCH + k);
    } else {
      typedef float __attribute__((ext_vector_type(N))) vec;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const vec w = *reinterpret_cast<const vec*>(tile + (k + x) * PITCH + base + N * r);
#pragma unroll
        for (int i = 0; i < N; ++i) f[i][x] = w[i];
      }
    }
  }
  // row of fragment i (A) that this lane's results belong to, relative to the wavefront's first
  static __device__ __forceinline__ int out_row(int i, int lane) {
    return A_KC ? 16 * i + (lane & 15) : TM * (lane & 15) + i;
  }
  // group q (of TNH) of 4 consecutive output columns of a panel: the first one, relative to the wavefront's first ...
  static __device__ __forceinline__ int out_col(int q, int lane) {
    return B_KC ? 16 * q + 4 * (lane >> 4) : 4 * (TNH * (lane >> 4) + q);
  }
  // ... and the four results of one fragment row
  static __device__ __forceinline__ f32x4 out4(const f32x4* acc, int q) {
    if constexpr (B_KC) return acc[q];
    f32x4 r;
#pragma unroll
    for (int x = 0; x < 4; ++x) r[x] = acc[(4 * q + x) % TNH][(4 * q + x) / TNH];
    return r;
  }

  static __device__ void run(const FArgs& g, float* smem) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    // Workgroups go round-robin to the 8 XCDs: each XCD takes one eighth of the tiles, one after another, and they run
    // through bands of kBand row tiles of an expert, row tile by row tile within a column: what an XCD has in flight is
    // about as high as it is wide, its L2 keeps the band's rows, and the columns of the weights pass through it once.
    int e = 0, row0, row_end, k_begin = 0, k_end = g.K;
    const int nx = MODE == DW13 ? 2 * g.tiles_n : g.tiles_n;
    RowTiles row_tiles(g.offsets, GROUP_K ? 1 : g.E, BM, lane);
    const int per_row_tile = SLICED ? nx * g.slices : nx;
    const int total = GROUP_K ? g.E * g.tiles_m * nx : row_tiles.count() * per_row_tile;
    const int share = (total + 7) / 8, id = (int)(blockIdx.x % 8) * share + (int)(blockIdx.x / 8);
    if ((int)(blockIdx.x / 8) >= share || id >= total) return;
    int tile_m, tile_n, n_rows, slice = 0;
    bool second_product = false;
    if (GROUP_K) {
      e = id / (g.tiles_m * nx);
      n_rows = g.tiles_m;
      tile_m = id - e * n_rows * nx;
    } else {
      row_tiles.expert_of(id, per_row_tile, e, n_rows, tile_m);
      if (SLICED) {
        slice = tile_m / (nx * n_rows);
        tile_m -= slice * nx * n_rows;
      }
    }
    const int band = tile_m / (kBand * nx), in_band = tile_m - band * kBand * nx, h = min(kBand, n_rows - band * kBand);
    tile_m = band * kBand + in_band % h;
    tile_n = in_band / h;
    if (GROUP_K) {
      row0 = tile_m * BM;
      row_end = g.M;
      k_begin = g.offsets[e];
      k_end = g.offsets[e + 1];
      if (MODE == DW13 && tile_n >= g.tiles_n) { tile_n -= g.tiles_n; second_product = true; }
    } else {
      row_tiles.rows_of(e, tile_m, row0, row_end);
    }
    const int col0 = tile_n * BNH;
    const float* A0 = g.A0;
    const float* B0 = second_product ? g.B1 : g.B0;
    const float* B1 = g.B1;
    bool two_passes = MODE == BWD_DX;
    if (SLICED && g.slices > 1) {                        // k tiles s nk / n .. (s + 1) nk / n of this slice's pass
      int n = g.slices;
      if (MODE == BWD_DX) {
        two_passes = false;
        n /= 2;
        if (slice >= n) { A0 = g.A1; B0 = g.B1; }
      }
      const int s = slice % n, nk = (g.K + BK - 1) / BK;
      k_begin = s * nk / n * BK;
      k_end = min((s + 1) * nk / n * BK, g.K);
    }
    if (!GROUP_K) { B0 += e * g.strideB_e; if (B1) B1 += e * g.strideB_e; }

    Operand<A_KC, BM, A_PITCH, NA, A_GATHER> a;
    Operand<B_KC, BN, B_PITCH, NB, B_GATHER> b;
    if constexpr (A_KC) a.rows(A0 + k_begin, row0, row_end, g.lda, g);
    else a.cols(g.A0, nullptr, row0, g.M, g.lda, k_begin);
    if constexpr (B_KC) b.rows(B0 + k_begin, col0, g.N, g.ldb, g);
    else b.cols(B0, B1, col0, g.N, g.ldb, k_begin);

    const int nk1 = (k_end - k_begin + BK - 1) / BK, nk = two_passes ? 2 * nk1 : nk1;
    auto look_up = [&](int kt) {
      if constexpr (!A_KC && A_GATHER) a.look_up(g, k_begin + kt * BK, k_end);
      if constexpr (!B_KC && B_GATHER) b.look_up(g, k_begin + kt * BK, k_end);
    };
    auto k_left = [&](int kt) { return k_end - k_begin - (two_passes && kt >= nk1 ? kt - nk1 : kt) * BK; };
    auto fetch = [&](auto set, int kt) {
      if (two_passes && kt == nk1) {                 // second K pass
        a.rows(g.A1, row0, row_end, g.lda, g);
        b.rows(B1, col0, g.N, g.ldb, g);
      }
      a.template fetch<decltype(set)::value>(g.lda, k_left(kt));
      b.template fetch<decltype(set)::value>(g.ldb, k_left(kt));
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    float* const As = smem;                              // two stages of A, then two of B
    float* const Bs = smem + 2 * A_SIZE;
    auto put = [&](auto set, int kt) {
      a.template put<decltype(set)::value>(As + (kt & 1) * A_SIZE, k_left(kt));
      b.template put<decltype(set)::value>(Bs + (kt & 1) * B_SIZE, k_left(kt));
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;
    if (nk > 0) {
      look_up(0);
      fetch(set0, 0);
      if (nk > 1) { look_up(1); fetch(set1, 1); }
      if (nk > 2) look_up(2);
      put(set0, 0);
      __syncthreads();
    }
    // k tile kt: request tile kt + 2, multiply, put tile kt + 1 into the other stage.  More than three tiles from the end
    // (MORE) no load is conditional: behind a branch that may have issued loads the compiler can only wait for all of
    // them, and every k tile waited for the one requested in it (4096 rows, one expert of 512 x 1376: DOWN 65 -> 60 us, DW13 196 -> 167, DW2 157 -> 115).
    auto step = [&](auto more, auto mine, auto other, int kt) {
      constexpr bool MORE = decltype(more)::value;
      if (MORE || kt + 2 < nk) {
        fetch(mine, kt + 2);
        if (MORE || kt + 3 < nk) look_up(kt + 3);
      }
      const float* At = As + (kt & 1) * A_SIZE;
      const float* Bt = Bs + (kt & 1) * B_SIZE;
#pragma unroll
      for (int s = 0; s < BK / 16; ++s) {
        f32x4 af[TM], bf[TN];
        frags<A_KC, A_PITCH, TM>(At, wm * (BM / 2), s, lane, af);
#pragma unroll
        for (int h = 0; h < TN / TNH; ++h)
          frags<B_KC, B_PITCH, TNH>(Bt, h * BNH + wn * (BNH / 2), s, lane, bf + h * TNH);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[j][x], af[i][x], acc[i][j], 0, 0, 0);
      }
      if (MORE || kt + 1 < nk) put(other, kt + 1);
      __syncthreads();
    };
    int kt = 0;
    for (; kt + 3 < nk; kt += 2) {
      step(std::true_type{}, set0, set1, kt);
      step(std::true_type{}, set1, set0, kt + 1);
    }
    for (; kt < nk; kt += 2) {
      step(std::false_type{}, set0, set1, kt);
      if (kt + 1 < nk) step(std::false_type{}, set1, set0, kt + 1);
    }

    const int m_wave = row0 + wm * (BM / 2), n_wave = col0 + wn * (BNH / 2);
    float* C = second_product ? g.C1 : g.C0;
    if (GROUP_K) C += e * g.strideC_e;
    if (SLICED && g.slices > 1) C = g.sums + (int64_t)slice * g.R * g.ldc;
    float dot[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m_wave + out_row(i, lane);
      dot[i] = 0.f;
      const float gate = MODE == BWD_ACT ? g.gates[g.perm_pairs[min(m, row_end - 1)]] : 0.f;
      if (m < row_end) {
#pragma unroll
        for (int q = 0; q < TNH; ++q) {
          const int n = n_wave + out_col(q, lane);
          if (n >= g.N) continue;
          const int64_t at = (int64_t)m * g.ldc + n;
          if constexpr (MODE == UP) {
            const f32x4 h1 = out4(acc[i], q), h3 = out4(acc[i] + TNH, q);
            f32x4 act;
#pragma unroll
            for (int x = 0; x < 4; ++x) act[x] = silu_f(h1[x]) * h3[x];
            if (g.C0) {
              *reinterpret_cast<f32x4*>(g.C0 + at) = h1;
              *reinterpret_cast<f32x4*>(g.C1 + at) = h3;
            }
            *reinterpret_cast<f32x4*>(g.C2 + at) = act;
          } else if constexpr (MODE == BWD_ACT) {
            const f32x4 z = *reinterpret_cast<const f32x4*>(g.H1 + at), h3 = *reinterpret_cast<const f32x4*>(g.H3 + at);
            const f32x4 D = out4(acc[i], q);
            f32x4 d1, d3, ga;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const float dd = D[x], sg = sigmoid_f(z[x]), sl = z[x] * sg, act = sl * h3[x], da = gate * dd;
              dot[i] = fmaf(dd, act, dot[i]);
              d1[x] = da * h3[x] * (sg * (1.f + z[x] * (1.f - sg)));
              d3[x] = da * sl;
              ga[x] = gate * act;
            }
            *reinterpret_cast<f32x4*>(g.C0 + at) = d1;
            *reinterpret_cast<f32x4*>(g.C1 + at) = d3;
            if (g.C2) *reinterpret_cast<f32x4*>(g.C2 + at) = ga;
          } else {
            *reinterpret_cast<f32x4*>(C + at) = out4(acc[i], q);
          }
        }
      }
    }
    if constexpr (MODE == BWD_ACT) {                     // dg partial of this column tile, summed in a fixed order
      float* red = smem;                                 // [2][BM]; the operand stages are dead
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float s = dot[i] + __shfl_xor(dot[i], 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (lane < 16) red[wn * BM + wm * (BM / 2) + 16 * i + lane] = s;
      }
      __syncthreads();
      for (int r = threadIdx.x; r < BM; r += kThreads)
        if (row0 + r < row_end) g.dg_part[(size_t)(row0 + r) * g.n_part + tile_n] = red[r] + red[BM + r];
    }
  }
};

template <int BM, int BN, int BK, int MODE> __global__ __launch_bounds__(kThreads) void f32_gemm_kernel(FArgs g) {
  using G = F32Gemm<BM, BN, BK, MODE>;
  __shared__ __attribute__((aligned(16))) float smem[2 * (G::A_SIZE + G::B_SIZE)];
  G::run(g, smem);
}

// 128 x 128 and 128 x 64 tiles of the same form (half the operand traffic per product, half the workgroups) were
// slower on this library's fp32 shapes: with 4006 rows, d = 512, f = 1376 DOWN 115 / 111 us against 84, DW13 151 / 142
// against 138 (of the loads then; 123 now).
constexpr int kTile = 64, kTileK = 32, kMaxSlices = 8;
// floats that the slices' sums of a product may take (128 MB): the cut pays while tiles are few, and the scratch has a bound of
// its own
constexpr int64_t kMaxSums = (int64_t)1 << 25;

// The K slices of a product added in slice order, 4 columns of a row per thread.
__global__ __launch_bounds__(kThreads) void f32_slices_finish_kernel(const float* __restrict__ sums, int slices, int R, int N,
                                                                     const int32_t* __restrict__ offsets, int E,
                                                                     float* __restrict__ C) {
  const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4, all = (int64_t)R * N;
  if (i >= (int64_t)offsets[E] * N) return;              // rows past the kept ones do not exist
  f32x4 a = *reinterpret_cast<const f32x4*>(sums + i);
  for (int s = 1; s < slices; ++s) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(sums + s * all + i);
#pragma unroll
    for (int x = 0; x < 4; ++x) a[x] += b[x];
  }
  *reinterpret_cast<f32x4*>(C + i) = a;
}

// K slices of DOWN and BWD_DX.  Few tiles of many k tiles leave compute units idle, or some with a tile more than others.
// Measured on 64 x 64 tiles of 32 k: with r tiles on a compute unit a k tile takes about 0.35 us for every four of them and
// 0.55 us each; the slices' sums pass through memory once more, BWD_DX's in a launch of its own.  (DOWN's are added by the combine where
// combine_most_slices() allows it; the launch that this saves is charged all the same.)  64 tokens, 8 experts of 512 x 1376, top-2:
// DOWN 35 -> 17 us, BWD_DX 66 -> 26.  most: see most_slices().
int f32_slices(int R, int E, int N, int K, bool two_passes, int most) {
  const int busy = std::max(std::min(E, R), 1);
  const int64_t tiles = (int64_t)busy * ceil_div(ceil_div(R, busy), kTile) * ceil_div(N, kTile);
  const double nk = ceil_div(K, kTileK) * (two_passes ? 2.0 : 1.0);
  int best = 1;
  double best_us = 0;
  for (int n = 1; n <= most; ++n) {
    if (n > 1 && ((two_passes && n % 2) || n > nk / 2 || (int64_t)n * R * N > kMaxSums)) continue;
    const double r = (double)ceil_div(tiles * n, 256), per_k = 0.35 * std::ceil(r / 4) + 0.55 * r;
    const double us = per_k * (nk / n + 1) + (n > 1 ? 5.0 + 8e-6 / 4 * n * (double)R * N : 0.0);
    if (n == 1 || us < best_us) { best = n; best_us = us; }
  }
  return best;
}

// No more scratch than two rows of d and three of f per grouped row.
int most_slices(const FfShapes& sh, bool two_passes) {
  const int by_k = ceil_div(sh.f, kTileK) * (two_passes ? 2 : 1) / 2, by_scratch = two_passes ? 2 + sh.f / sh.d : 1 + 2 * sh.f / sh.d;
  return std::min({kMaxSlices, by_k, by_scratch});
}
// Scratch of the sums for up to sh.R rows: what any number of rows up to that asks for, so that a workspace of a large batch
// serves every smaller one (fewer rows may be cut into more slices).
size_t sums_bytes(const FfShapes& sh, bool two_passes) {
  const int most = most_slices(sh, two_passes);
  return most < 2 ? 0 : std::min((size_t)most * sh.R * sh.d, (size_t)kMaxSums) * sizeof(float);
}
int slices_of(const FfShapes& sh, bool two_passes) {
  return f32_slices(sh.R, sh.E, sh.d, sh.f, two_passes, most_slices(sh, two_passes));
}

// left (may be NULL): in, K slices that the caller can add himself; out, those whose sums he finds in g.sums (1: none)
template <int MODE> int launch(FArgs g, int R, hipStream_t s, int* left = nullptr) {
  constexpr int BM = kTile, BN = kTile, BK = kTileK;
  using G = F32Gemm<BM, BN, BK, MODE>;
  g.tiles_n = ceil_div(g.N, G::BNH);
  g.tiles_m = ceil_div(g.M, BM);
  if (!G::SLICED) g.slices = 1;
  g.R = R;
  const int64_t tiles = (int64_t)(MODE == DW13 ? 2 * g.tiles_n : g.tiles_n) * g.slices *
                        (G::GROUP_K ? (int64_t)g.E * g.tiles_m : (int64_t)ceil_div(R, BM) + g.E);   // at most this many
  if (!grid_fits(tiles + 7, kThreads)) return BTX_ERR_UNSUPPORTED;
  const unsigned grid = (unsigned)align_up((size_t)tiles, 8);
  f32_gemm_kernel<BM, BN, BK, MODE><<<grid, kThreads, 0, s>>>(g);
  BTX_LAUNCH_CHECK();
  const bool leave = left && g.slices <= *left;
  if (left) *left = leave ? g.slices : 1;
  if (g.slices > 1 && !leave) {
    f32_slices_finish_kernel<<<ceil_div((int64_t)R * g.N / 4, kThreads), kThreads, 0, s>>>(g.sums, g.slices, R, g.N, g.offsets,
                                                                                         g.E, g.C0);
    BTX_LAUNCH_CHECK();
  }
  return BTX_OK;
}

}  // namespace

bool f32_rows_ok(int R, int E) { return ceil_div(R, 64) + E <= 65535; }
int f32_bwd_act_partials(int f) { return ceil_div(f, kTile); }
size_t f32_down_sums_bytes(const FfShapes& sh) { return sums_bytes(sh, false); }
size_t f32_bwd_dx_sums_bytes(const FfShapes& sh) { return sums_bytes(sh, true); }

int f32_up_swiglu(const RowSource& xs, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh, void* h1,
                  void* h3, void* act, hipStream_t s) {
  FArgs g{};
  g.A0 = (const float*)xs.base; g.gather(xs); g.B0 = (const float*)W1; g.B1 = (const float*)W3;
  g.C0 = (float*)h1; g.C1 = (float*)h3; g.C2 = (float*)act;
  g.offsets = off; g.E = sh.E; g.N = sh.f; g.K = sh.d; g.lda = sh.d; g.ldb = sh.f; g.ldc = sh.f; g.strideB_e = sh.s13;
  return launch<UP>(g, sh.R, s);
}
int f32_down(const void* act, const void* W2, const int32_t* off, const FfShapes& sh, void* y, void* sums, int* slices, hipStream_t s) {
  FArgs g{};
  g.slices = slices_of(sh, false); g.sums = (float*)sums;
  g.A0 = (const float*)act; g.B0 = (const float*)W2; g.C0 = (float*)y;
  g.offsets = off; g.E = sh.E; g.N = sh.d; g.K = sh.f; g.lda = sh.f; g.ldb = sh.d; g.ldc = sh.d; g.strideB_e = sh.s2;
  return launch<DOWN>(g, sh.R, s, slices);
}
int f32_bwd_act(const RowSource& dys, const void* W2, const void* h1, const void* h3, const float* gates,
                const int32_t* perm, const int32_t* off, const FfShapes& sh, void* dh1, void* dh3, void* ga,
                float* dg_part, hipStream_t s) {
  FArgs g{};
  g.A0 = (const float*)dys.base; g.gather(dys); g.B0 = (const float*)W2;
  g.C0 = (float*)dh1; g.C1 = (float*)dh3; g.C2 = (float*)ga;
  g.H1 = (const float*)h1; g.H3 = (const float*)h3; g.gates = gates; g.perm_pairs = perm; g.dg_part = dg_part;
  g.n_part = f32_bwd_act_partials(sh.f);
  g.offsets = off; g.E = sh.E; g.N = sh.f; g.K = sh.d; g.lda = sh.d; g.ldb = sh.d; g.ldc = sh.f; g.strideB_e = sh.s2;
  return launch<BWD_ACT>(g, sh.R, s);
}
int f32_bwd_dx(const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh,
               void* dxs, void* sums, hipStream_t s) {
  FArgs g{};
  g.slices = slices_of(sh, true); g.sums = (float*)sums;
  g.A0 = (const float*)dh1; g.A1 = (const float*)dh3; g.B0 = (const float*)W1; g.B1 = (const float*)W3; g.C0 = (float*)dxs;
  g.offsets = off; g.E = sh.E; g.N = sh.d; g.K = sh.f; g.lda = sh.f; g.ldb = sh.f; g.ldc = sh.d; g.strideB_e = sh.s13;
  return launch<BWD_DX>(g, sh.R, s);
}
int f32_bwd_dw13(const RowSource& xs, const void* dh1, const void* dh3, const int32_t* off, const FfShapes& sh, void* dW1,
                 void* dW3, hipStream_t s) {
  FArgs g{};
  g.A0 = (const float*)xs.base; g.gather(xs); g.B0 = (const float*)dh1; g.B1 = (const float*)dh3;
  g.C0 = (float*)dW1; g.C1 = (float*)dW3;
  g.offsets = off; g.E = sh.E; g.M = sh.d; g.N = sh.f; g.lda = sh.d; g.ldb = sh.f; g.ldc = sh.f; g.strideC_e = sh.s13;
  return launch<DW13>(g, sh.R, s);
}
int f32_bwd_dw2(const void* ga, const RowSource& dys, const int32_t* off, const FfShapes& sh, void* dW2, hipStream_t s) {
  FArgs g{};
  g.A0 = (const float*)ga; g.B0 = (const float*)dys.base; g.gather(dys); g.C0 = (float*)dW2;
  g.offsets = off; g.E = sh.E; g.M = sh.f; g.N = sh.d; g.lda = sh.f; g.ldb = sh.d; g.ldc = sh.d; g.strideC_e = sh.s2;
  return launch<DW2>(g, sh.R, s);
}

}  // namespace btx
