// fp32 grouped GEMMs of the expert FFNs (SwiGLU feed-forward of the seed model, Sec. 4.1, inside the
// layer equation of Sec. 3.2) and of their backward: the same six products as gemm_mfma.hip with fp32
// operands, fp32 matrix instructions (v_mfma_f32_16x16x4_f32: exact products, fp32 sums) and fp32 storage.
//
// The matrix pipe bounds it: 256 FLOP per clock and compute unit, a sixteenth of bf16, while a fragment
// feeds as many output tiles, so LDS and L2 have room to spare.  What keeps the pipe from being busy is the other
// instructions: each vector or scalar one costs it 2 to 4 clocks, whichever wavefront of the SIMD issues it.  So the tiles are
// kept simple and the loop short:
//   * 64 x 64 x 32, 4 wavefronts as 2 x 2, two LDS stages, one barrier per k tile; five workgroups per compute unit cover
//     each other's barriers and memory latency (three stages and three workgroups: 4 % slower, 9 % with four and two;
//     where one or two tiles are all that a unit gets, see weights_from_memory()).
//   * operands go straight from global memory to LDS, four copies per wavefront and k tile in one block: one setting of m0,
//     bases in scalar registers, 32-bit lane offsets that stay the same from k tile to k tile.  With copies from 64-bit addresses in
//     vector registers the compute unit's other wavefronts lose the matrix pipe to them: 4096 rows, one expert of 1024 x 4096: DOWN
//     319 us, 249 like this.  Those only serve operands that 32 bits do not reach (wide_offsets()).
//   * within 16 consecutive k a lane of k group g supplies k = 4 g + i to instruction i (the order of k inside
//     a sum is free as long as both operands agree), so that an operand whose k is contiguous in memory is kept
//     as rows of k and read 16 bytes at a time; an operand whose k is strided (the weights in UP and DOWN,
//     everything in the dW products) stays as it lies in memory, and a wavefront's fragments are interleaved columns, one
//     read for all of them.
//   * only a last, partial k tile is masked; a branch leads there.
//   * the operands' roles are swapped, so that a lane ends up with 4 consecutive columns of one row.
//   * token rows (x, dY) are read through perm wherever they are an operand (the weight gradients: by byte offsets that BWD_ACT
//     leaves behind, found through the scalar cache), the SwiGLU and its backward are epilogues on the accumulators: nothing is
//     gathered, and no product is stored only to be read again.
// Measured, fwd + bwd of 2003 tokens through 8 experts of 512 x 1376, top-2 (the products 51 GFLOP), operands through registers and
// every product by itself / now: 600 / 522 us (16 of it the router's backward pass): UP 114 / 107 us, DOWN 77 / 61, BWD_ACT 68 / 66, BWD_DX 127, DW13 114 and DW2 64 / 263
// in one launch, at 82 to 107 of the 153 TFLOP/s this instruction sustains; 4096 rows, one expert of 1024 x 4096: 2598 / 2404, at 115
// to 137.  What is left is ragged rounds of 64 x 64 tiles and what starting and storing a tile takes.
#include "gemm_f32.h"
#include "router_ds.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace btx {
namespace {

enum Mode { UP = 0, DOWN = 1, BWD_ACT = 2, BWD_DX = 3, DW13 = 4, DW2 = 5 };

struct FArgs {
  const float* A0; const float* A1;      // A1: second K pass (BWD_DX)
  const float* B0; const float* B1;      // B1: second panel (UP), second product (DW13), second K pass (BWD_DX)
  float* C0; float* C1; float* C2;       // UP: h1, h3 (NULL: not kept), act; BWD_ACT: dh1, dh3, ga; DW13: dW1, dW3; DOWN: y, and cut()
  const float* H1; const float* H3; const float* gates; float* dg_part; int n_part;   // BWD_ACT
  const int32_t* perm; uint32_t div_mul, div_shift; int k;   // gathered operand: row r is token perm[r] / k
  uint32_t* row_bytes;                   // byte offset of every grouped row's token row: BWD_ACT writes it for the weight gradients (NULL: none wanted)
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
  // DOWN: the last round's tiles in K slices (see Cut); their sums, [slot][64][64] (NULL: whole).  In the place of a pointer that DOWN does
  // without: with one of its own in front of tiles_n every product waited longer for its arguments, the backward pass of 2204 tokens, 4
  // experts of 64 x 64, top-4 79.6 us, now 77.8; 3284 of 256 x 192, top-2 90.7, now 89.3.
  __host__ __device__ float* cut() const { return C2; }
  void gather(const RowSource& r) {
    perm = r.perm;
    k = r.k;
    int l = 0;
    while ((1 << l) < r.k) ++l;
    div_shift = 31 + l;
    div_mul = (uint32_t)((((uint64_t)1 << div_shift) + r.k - 1) / r.k);
  }
};

constexpr int kThreads = 256;
constexpr int kTile = 64, kTileK = 32;   // rows and columns of a tile, and k of a k tile
constexpr int kBand = 8;                 // row tiles of a band in the tile order

// Four copies of 1 KB, 16 bytes per lane, from global memory straight into LDS, to lds, lds + 1024, ... : copies 0 and 1 from
// a + off, 2 from b0 + off, 3 from b1 + off.  The offset of the instruction counts in memory as in LDS, so the lanes' offsets make up
// for it (Operand::kBias), and all four share one setting of m0.  Inline assembly, so that the compiler does not wait for the
// copies in flight before every LDS read; wait_vmcnt() awaits them.
__device__ __forceinline__ void copy_to_lds(uint32_t lds, const float* a, const float* b0, const float* b1, const uint32_t* oa, const uint32_t* ob) {
  const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5\n\tglobal_load_lds_dwordx4 %2, %5 offset:1024\n\t"
               "global_load_lds_dwordx4 %3, %6 offset:2048\n\tglobal_load_lds_dwordx4 %4, %7 offset:3072"
               :
               : "s"(at), "v"(oa[0]), "v"(oa[1]), "v"(ob[0]), "v"(ob[1]), "s"(uniform64(a)), "s"(uniform64(b0)), "s"(uniform64(b1))
               : "memory");
}
__device__ __forceinline__ void copy_to_lds(uint32_t lds, const float* a, const float* b0, const float* b1, const uint64_t* oa, const uint64_t* ob) {
  const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);
  const uint64_t A = reinterpret_cast<uint64_t>(a), B0 = reinterpret_cast<uint64_t>(b0), B1 = reinterpret_cast<uint64_t>(b1);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\tglobal_load_lds_dwordx4 %2, off offset:1024\n\t"
               "global_load_lds_dwordx4 %3, off offset:2048\n\tglobal_load_lds_dwordx4 %4, off offset:3072"
               :
               : "s"(at), "v"(A + oa[0]), "v"(A + oa[1]), "v"(B0 + ob[0]), "v"(B1 + ob[1])
               : "memory");
}

// DOWN of few tiles: those of an XCD that its 32 compute units do not get evenly, the last ones of its `share`, are cut along K into as
// many slices as give every unit one, and f32_cut_finish_kernel adds them in slice order.  A unit with one tile more than the others
// held them all up (f32_cut()).
struct Cut {
  static constexpr int UNITS = 32, MOST = 8;
  int whole, left, slices;
  __device__ __forceinline__ explicit Cut(int share) {
    left = share % UNITS;
    slices = left ? min(UNITS / left, MOST) : 1;
    if (slices < 2) left = 0;
    whole = share - left;
  }
};

// WIDE: byte offsets inside an operand need more than 32 bits (wide_offsets()).  STAGES: of LDS, three for weights_from_memory()
template <int MODE, bool WIDE, int STAGES = 2> struct F32Gemm {
  typedef std::conditional_t<WIDE, uint64_t, uint32_t> Off;
  static constexpr bool GROUP_K = MODE == DW13 || MODE == DW2;
  static constexpr bool A_KC = !GROUP_K, B_KC = MODE == BWD_ACT || MODE == BWD_DX;   // k contiguous in memory
  static constexpr bool A_GATHER = MODE == UP || MODE == BWD_ACT || MODE == DW13, B_GATHER = MODE == DW2;
  static constexpr bool SLICED = MODE == DOWN || MODE == BWD_DX;
  static constexpr bool DUAL = MODE == UP;                       // two B panels in one tile
  static constexpr int BNH = DUAL ? kTile / 2 : kTile;           // output columns of a tile
  static constexpr int STAGE = 2 * kTile * kTileK, PIECE = STAGE / 4;   // floats of a stage, and of it those that one wavefront copies

  // LDS: a stage is four pieces of 4 KB, each two copies of A and two of B by one wavefront.  An operand whose k is contiguous: 16
  // rows of 32 k to a piece, 8 chunks of 16 bytes to a row, the chunk index XORed with row / 2.  One whose k is strided: 8 k rows of 64
  // columns, as it lies in memory, the halves of the row exchanged in every other group of four k.  Two panels (UP): 8 k rows
  // of 32 columns of the one, then of the other, there odd and even k rows exchanged, and the halves of the row as above.  All of it
  // makes the reads below free of bank conflicts.  A copy fixes where a lane's 16 bytes land, so a lane chooses which chunk of
  // global memory it fetches.
  static __device__ __forceinline__ int kc_swz(int row) { return (row >> 1) & 7; }
  static __device__ __forceinline__ int tr_swz(bool panels, int k) { return ((k >> 2) & 1) << (panels ? 2 : 3); }

  // One operand of a tile: this lane's chunks of it.  Rows and columns past the matrix repeat its last ones: their results are never
  // stored.  SLOT: its first copy's place in the piece.
  template <bool KC, bool GATHER, bool PANELS, int SLOT> struct Operand {
    static constexpr bool LOOK_UP = !KC && GATHER;
    static constexpr int kBias = 4096;   // bytes that `base` lies ahead of the data (see copy_to_lds())
    const float* base;                   // uniform: first row and k (strided: k row and column) of the k tile that is copied next
    const float* base2;                  // PANELS: the same of the second panel
    Off off[2];                          // bytes from there to this lane's chunk of either copy (LOOK_UP: to its column)
    uint32_t tok[LOOK_UP ? 8 : 1];       // LOOK_UP: byte offsets (WIDE: token rows) of this wavefront's k rows of the k tile that is copied next
    // contiguous: the row, strided: the k row of this lane's chunk of copy q
    static __device__ __forceinline__ int major_of(int q, int wave, int lane) {
      return KC ? 16 * wave + 8 * q + (lane >> 3) : PANELS ? 8 * wave + ((lane >> 3) ^ q) : 8 * wave + 4 * q + (lane >> 4);
    }
    // contiguous: its k, strided: its column
    static __device__ __forceinline__ int minor_of(int q, int wave, int lane) {
      const int m = major_of(q, wave, lane);
      return KC ? 4 * ((lane & 7) ^ kc_swz(m)) : PANELS ? 4 * ((lane & 7) ^ tr_swz(true, m)) : 4 * ((lane & 15) ^ tr_swz(false, m));
    }
    static __device__ __forceinline__ Off bytes(int q, Off floats) { return floats * 4 + (Off)(kBias - 1024 * (SLOT + q)); }
    // rows row0 .. of an operand whose k is contiguous, from `from` on
    __device__ __forceinline__ void rows(const float* from, int row0, int row_end, int ld, int wave, int lane, const FArgs& g) {
      base = from + ((GATHER ? (int64_t)0 : (int64_t)row0 * ld) - kBias / 4);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int r = min(row0 + major_of(q, wave, lane), row_end - 1);
        off[q] = bytes(q, (Off)(GATHER ? g.token(g.perm[r]) : r - row0) * (Off)ld + (Off)minor_of(q, wave, lane));
      }
    }
    // columns col0 .. of an operand whose k is strided, from row k0 on; PANELS: as many of `from2` as well
    __device__ __forceinline__ void cols(const float* from, const float* from2, int col0, int n, int ld, int k0, int wave, int lane) {
      const int64_t first = (GATHER ? (int64_t)0 : (int64_t)k0 * ld) + col0 - kBias / 4;
      base = from + first;
      base2 = PANELS ? from2 + first : base;
#pragma unroll
      for (int q = 0; q < 2; ++q)
        off[q] = bytes(q, (Off)(GATHER ? 0 : major_of(q, wave, lane)) * (Off)ld + (Off)(min(col0 + minor_of(q, wave, lane), n - 4) - col0));
    }
    // LOOK_UP: the token rows of the k tile from k0 on, through the scalar cache (vector loads would be waited for together with
    // the copies behind them); rows past k_end repeat the last one
    __device__ __forceinline__ void look_up(const FArgs& g, int k0, int k_end, int wave) {
      typedef uint32_t u32x8 __attribute__((ext_vector_type(8), aligned(4)));
      typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;
      typedef const __attribute__((address_space(4))) u32x8* scalar_ptr8;
      const scalar_ptr table = (scalar_ptr)(uintptr_t)(WIDE ? reinterpret_cast<const uint32_t*>(g.perm) : g.row_bytes);
      const int k = k0 + 8 * wave;
      if (k + 8 <= k_end) {
        const u32x8 t = *(scalar_ptr8)(table + k);
#pragma unroll
        for (int x = 0; x < 8; ++x) tok[x] = t[x];
      } else {
#pragma unroll
        for (int x = 0; x < 8; ++x) tok[x] = table[min(k + x, k_end - 1)];
      }
    }
    // offsets of the copies of a k tile of which n_k k exist; k that do not exist repeat the tile's first (last) k
    __device__ __forceinline__ void offsets(Off (&o)[2], int ld, int n_k, int wave, int lane, const FArgs& g) const {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        o[q] = off[q];
        if constexpr (LOOK_UP) {
          const int x = lane >> 4;
          const uint32_t lo = x & 1 ? tok[4 * q + 1] : tok[4 * q], hi = x & 1 ? tok[4 * q + 3] : tok[4 * q + 2];
          const uint32_t t = x & 2 ? hi : lo;
          o[q] += WIDE ? (Off)g.token((int)t) * (Off)ld * 4 : (Off)t;
        } else if (n_k < kTileK) {
          const int k = KC ? minor_of(q, wave, lane) : major_of(q, wave, lane);
          o[q] -= KC ? (Off)(k >= n_k ? 4 * k : 0) : (Off)max(k - n_k + 1, 0) * (Off)ld * 4;
        }
      }
    }
    __device__ __forceinline__ void advance(int ld) {
      if (LOOK_UP) return;
      const int64_t step = KC ? (int64_t)kTileK : (int64_t)kTileK * ld;
      base += step;
      base2 += step;
    }
  };

  // Fragments of 16 rows (columns) x 16 k: element x of f[i] feeds instruction x, k = 16 s + 4 (lane / 16) + x.
  // contiguous: fragment i is rows 32 w + 16 i + lane % 16 of the tile; strided: columns 32 w + 2 (lane % 16) + i, one read for both
  // fragments.  PANELS: 16 columns of either panel, two pairs of columns from the first, two of the second, and so on, so that
  // a lane of the result holds both products of its outputs.
  template <bool KC, bool PANELS>
  static __device__ __forceinline__ void frags(const float* tile, int w, int s, int lane, f32x4* f) {
    const int r = lane & 15, g4 = lane >> 4;
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        f[i] = *reinterpret_cast<const f32x4*>(tile + (2 * w + i) * PIECE + r * kTileK + (((4 * s + g4) ^ kc_swz(r)) << 2));
    } else {
      typedef float __attribute__((ext_vector_type(2))) vec;
      const int k = 4 * g4, p = (r >> 1) & 1;            // of 16 s + k + x: piece 2 s + k / 8
      const int col = (PANELS ? 16 * w + 2 * ((r & 1) + 2 * (r >> 2)) : 32 * w + 2 * r) ^ (tr_swz(PANELS, k) << 2);
      const float* at = tile + (2 * s + (k >> 3)) * PIECE + col + (PANELS ? 256 * p : 0);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const vec v = *reinterpret_cast<const vec*>(at + (PANELS ? (((k & 7) + x) ^ p) * 32 : ((k & 7) + x) * 64));
        f[0][x] = v[0];
        f[1][x] = v[1];
      }
    }
  }
  // row of fragment i (A) that this lane's results belong to, relative to the wavefront's first
  static __device__ __forceinline__ int out_row(int i, int lane) {
    return A_KC ? 16 * i + (lane & 15) : 2 * (lane & 15) + i;
  }
  // group q of 4 consecutive output columns (UP: one, of each panel): the first one, relative to the wavefront's first ...
  static __device__ __forceinline__ int out_col(int q, int lane) {
    return DUAL ? 4 * (lane >> 4) : B_KC ? 16 * q + 4 * (lane >> 4) : 4 * (2 * (lane >> 4) + q);
  }
  // ... and the four results of one fragment row (UP: of panel q)
  static __device__ __forceinline__ f32x4 out4(const f32x4* acc, int q) {
    if constexpr (!DUAL && B_KC) return acc[q];
    return f32x4{acc[0][2 * q], acc[1][2 * q], acc[0][2 * q + 1], acc[1][2 * q + 1]};
  }

  // tile `tile` of those of an expert of n_rows row tiles, in bands: its row and column
  static __device__ __forceinline__ void in_bands(int tile, int nx, int n_rows, int& tile_m, int& tile_n) {
    const int band = tile / (kBand * nx), in_band = tile - band * kBand * nx, h = min(kBand, n_rows - band * kBand);
    tile_m = band * kBand + in_band % h;
    tile_n = in_band / h;
  }

  // block: of the `total` ones of this product
  static __device__ void run(const FArgs& g, unsigned block, float* smem) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    // Workgroups go round-robin to the 8 XCDs: each XCD takes one eighth of the tiles, one after another, and they run
    // through bands of kBand row tiles of an expert, row tile by row tile within a column: what an XCD has in flight is
    // about as high as it is wide, its L2 keeps the band's rows, and the columns of the weights pass through it once.
    int e = 0, row0, row_end, k_begin = 0, k_end = g.K;
    const int nx = MODE == DW13 ? 2 * g.tiles_n : g.tiles_n;
    RowTiles row_tiles(g.offsets, GROUP_K ? 1 : g.E, kTile, lane);
    const int per_row_tile = SLICED ? nx * g.slices : nx;
    const int total = GROUP_K ? g.E * g.tiles_m * nx : row_tiles.count() * per_row_tile;
    const int share = (total + 7) / 8, xcd = (int)(block % 8);
    int pos = (int)(block / 8), slice = 0, cut_slices = 1;
    float* cut_sums = nullptr;
    if (MODE == DOWN && g.cut()) {
      const Cut cut(share);
      if (const int p = pos - cut.whole; p >= 0 && cut.left > 0) {
        slice = p / cut.left;
        if (slice >= cut.slices) return;
        cut_slices = cut.slices;
        cut_sums = g.cut() + (int64_t)((xcd * cut.left + p % cut.left) * cut.slices + slice) * (kTile * kTile);
        pos = cut.whole + p % cut.left;
      }
    }
    const int id = xcd * share + pos;
    if (pos >= share || id >= total) return;
    int tile_m, tile_n, n_rows;
    bool second_product = false;
    if (GROUP_K) {
      e = id / (g.tiles_m * nx);
      n_rows = g.tiles_m;
      tile_m = id - e * n_rows * nx;
    } else {
      row_tiles.expert_of(id, per_row_tile, e, n_rows, tile_m);
      if (SLICED && (MODE != DOWN || g.slices > 1)) {    // (DOWN's cut tiles have theirs)
        slice = tile_m / (nx * n_rows);
        tile_m -= slice * nx * n_rows;
      }
    }
    in_bands(tile_m, nx, n_rows, tile_m, tile_n);
    if (GROUP_K) {
      row0 = tile_m * kTile;
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
      const int s = slice % n, nk = (g.K + kTileK - 1) / kTileK;
      k_begin = s * nk / n * kTileK;
      k_end = min((s + 1) * nk / n * kTileK, g.K);
    } else if (MODE == DOWN && cut_slices > 1) {
      const int nk = (g.K + kTileK - 1) / kTileK;
      k_begin = slice * nk / cut_slices * kTileK;
      k_end = min((slice + 1) * nk / cut_slices * kTileK, g.K);
    }
    if (!GROUP_K) { B0 += e * g.strideB_e; if (B1) B1 += e * g.strideB_e; }

    Operand<A_KC, A_GATHER, false, 0> a;
    Operand<B_KC, B_GATHER, DUAL, 2> b;
    if constexpr (A_KC) a.rows(A0 + k_begin, row0, row_end, g.lda, wave, lane, g);
    else a.cols(g.A0, nullptr, row0, g.M, g.lda, k_begin, wave, lane);
    if constexpr (B_KC) b.rows(B0 + k_begin, col0, g.N, g.ldb, wave, lane, g);
    else b.cols(B0, B1, col0, g.N, g.ldb, k_begin, wave, lane);

    const int n_k1 = k_end - k_begin, nk1 = (n_k1 + kTileK - 1) / kTileK, nk = two_passes ? 2 * nk1 : nk1;
    const int k_tail = n_k1 - (nk1 - 1) * kTileK;        // k that exist in the last k tile of a pass
    constexpr bool LOOK_UP = GROUP_K;
    auto look_up = [&](int kt) {
      if constexpr (!A_KC && A_GATHER) a.look_up(g, k_begin + kt * kTileK, k_end, wave);
      if constexpr (!B_KC && B_GATHER) b.look_up(g, k_begin + kt * kTileK, k_end, wave);
    };
    const uint32_t lds = (uint32_t)(uintptr_t)smem + wave * (PIECE * 4);
    int next = 0, last = nk1 - 1;                        // the k tile that is copied next; the last one of its pass
    auto request = [&](int stage, int n_k) {
      Off oa[2], ob[2];
      a.offsets(oa, g.lda, n_k, wave, lane, g);
      b.offsets(ob, g.ldb, n_k, wave, lane, g);
      copy_to_lds(lds + stage * (STAGE * 4), a.base, b.base, DUAL ? b.base2 : b.base, oa, ob);
    };
    auto copy = [&](int stage) {
      if (next != last) {                                // a branch, so that the rare case costs nothing else
        request(stage, kTileK);
      } else {
        request(stage, k_tail);
        last = nk - 1;
      }
      ++next;
      a.advance(g.lda);
      b.advance(g.ldb);
      if (MODE == BWD_DX && next == nk1 && two_passes) { // second K pass
        a.rows(g.A1, row0, row_end, g.lda, wave, lane, g);
        b.rows(B1, col0, g.N, g.ldb, wave, lane, g);
      }
    };

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // k tile kt, in LDS stage `stage`; more: another one follows
    auto step = [&](auto stage_tag, auto more_tag, int kt) {
      const int stage = stage_tag;
      constexpr bool more = decltype(more_tag)::value;
      if (STAGES == 2 || kt + STAGES - 2 >= nk) wait_vmcnt<0>(); else wait_vmcnt<4 * (STAGES - 2)>();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();                      // k tile kt published; everybody is done with the last one
      __builtin_amdgcn_sched_barrier(0);
      if (STAGES == 2 ? more : kt + STAGES - 1 < nk) copy(STAGES == 2 ? stage ^ 1 : stage == 0 ? STAGES - 1 : stage - 1);
      const float* T = smem + stage * STAGE;
      f32x4 af[2][2], bf[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        frags<A_KC, false>(T, wm, s, lane, af[s]);
        frags<B_KC, DUAL>(T + PIECE / 2, wn, s, lane, bf[s]);
      }
      if (more && LOOK_UP) {
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): scalar loads behind the fragments would be waited for with them
        __builtin_amdgcn_sched_barrier(0);
        look_up(kt + 2);
      }
      // k that do not exist repeat others: zeros instead
      if (k_tail < kTileK && (!more || (MODE == BWD_DX && two_passes && kt == nk1 - 1))) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const bool in = 16 * s + 4 * (lane >> 4) + x < k_tail;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              af[s][i][x] = in ? af[s][i][x] : 0.f;
              bf[s][i][x] = in ? bf[s][i][x] : 0.f;
            }
          }
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[s][j][x], af[s][i][x], acc[i][j], 0, 0, 0);
    };
    const std::integral_constant<int, 0> stage0;
    const std::integral_constant<int, 1> stage1;
    if (STAGES > 2 && nk > 0) {                          // STAGES - 1 k tiles on their way
      static_assert(STAGES == 2 || !LOOK_UP, "token rows are looked up one k tile ahead");
      for (int j = 0; j < STAGES - 1; ++j)
        if (j < nk) copy(j);
      int stage = 0;
#pragma unroll 1
      for (int kt = 0; kt < nk - 1; ++kt) {
        step(stage, std::true_type{}, kt);
        stage = stage == STAGES - 1 ? 0 : stage + 1;
      }
      step(stage, std::false_type{}, nk - 1);
    } else if (nk > 0) {
      look_up(0);
      copy(0);
      look_up(1);
      for (int kt = 0;; kt += 2) {
        if (kt + 1 >= nk) { step(stage0, std::false_type{}, kt); break; }
        step(stage0, std::true_type{}, kt);
        if (kt + 2 >= nk) { step(stage1, std::false_type{}, kt + 1); break; }
        step(stage1, std::true_type{}, kt + 1);
      }
    }

    const int m_wave = row0 + wm * 32, n_wave = col0 + wn * (BNH / 2);
    constexpr int GROUPS = DUAL ? 1 : 2;                 // of 4 consecutive columns that a lane holds of a row
    float* C = second_product ? g.C1 : g.C0;
    if (GROUP_K) C += e * g.strideC_e;
    if (SLICED && g.slices > 1) C = g.sums + (int64_t)slice * g.R * g.ldc;
    float dot[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = m_wave + out_row(i, lane);
      dot[i] = 0.f;
      const float gate = MODE == BWD_ACT ? g.gates[g.perm_pairs[min(m, row_end - 1)]] : 0.f;
      if (m < row_end) {
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
          const int n = n_wave + out_col(q, lane);
          if (n >= g.N) continue;
          const int64_t at = (int64_t)m * g.ldc + n;
          if constexpr (MODE == UP) {
            const f32x4 h1 = out4(acc[i], 0), h3 = out4(acc[i], 1);
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
          } else if (MODE == DOWN && cut_sums) {
            *reinterpret_cast<f32x4*>(cut_sums + (m - row0) * kTile + n - col0) = out4(acc[i], q);
          } else {
            *reinterpret_cast<f32x4*>(C + at) = out4(acc[i], q);
          }
        }
      }
    }
    if constexpr (MODE == BWD_ACT) {                     // dg partial of this column tile, summed in a fixed order
      __syncthreads();                                   // everybody is done with the operand stages
      float* red = smem;                                 // [2][kTile]
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float s = dot[i] + __shfl_xor(dot[i], 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (lane < 16) red[wn * kTile + wm * 32 + 16 * i + lane] = s;
      }
      __syncthreads();
      const int r = threadIdx.x, row = row0 + r;
      if (r < kTile && row < row_end) {
        g.dg_part[(size_t)row * g.n_part + tile_n] = red[r] + red[kTile + r];
        if (g.row_bytes && tile_n == 0) g.row_bytes[row] = (uint32_t)g.token(g.perm[row]) * (uint32_t)(g.lda * 4);
      }
    }
  }
};

template <int MODE, bool WIDE, int STAGES> __global__ __launch_bounds__(kThreads, STAGES == 2 ? 5 : 3) void f32_gemm_kernel(FArgs g) {
  using G = F32Gemm<MODE, WIDE, STAGES>;
  __shared__ __attribute__((aligned(1024))) float smem[STAGES * G::STAGE];
  G::run(g, blockIdx.x, smem);
}
// The input's and the weights' gradients need what BWD_ACT has left and nothing of each other: one launch, first the tiles of BWD_DX,
// whose contraction is the longest in small batches (last: 279 us for a whole pass of 700 tokens, first 252), then DW13's, then DW2's;
// each number a multiple of 8, as they are dealt to the XCDs.  A product fills what the one before it leaves idle at its end, and in
// small batches two launches count.  Whole backward products, us, three launches / one: 256 tokens of 256, f = 688, 4 experts 34 / 23;
// 100 of 512, f = 1376, 8 experts 67 / 50; 2003 of them 290 / 263.  BWD_DX uncut there would take 249, but its sums would be longer chains, and not
// those of a pass with frozen experts.
template <bool WIDE>
__global__ __launch_bounds__(kThreads, 5) void f32_dx_dw_kernel(FArgs dx, unsigned dx_blocks, FArgs dw13, unsigned dw13_blocks, FArgs dw2, unsigned dw2_blocks, RouterDs ds) {
  __shared__ __attribute__((aligned(1024))) float smem[2 * F32Gemm<BWD_DX, WIDE>::STAGE];
  const unsigned b = blockIdx.x;
  if (b < dx_blocks) F32Gemm<BWD_DX, WIDE>::run(dx, b, smem);
  else if (b < dx_blocks + dw13_blocks) F32Gemm<DW13, WIDE>::run(dw13, b - dx_blocks, smem);
  else if (b < dx_blocks + dw13_blocks + dw2_blocks) F32Gemm<DW2, WIDE>::run(dw2, b - dx_blocks - dw13_blocks, smem);
  else router_ds(ds, b - dx_blocks - dw13_blocks - dw2_blocks);
}

// Tried: 128 x 128 and 128 x 64 tiles (half the operand traffic per product, half the workgroups): 4006 rows, d = 512, f = 1376, operands
// through registers: DOWN 115 / 111 us against 84, DW13 151 / 142 against 138.  64 x 64 per wavefront, the wavefronts taking turns along
// K, each with stages of its own and no barrier (half the reads from LDS): DOWN 76, DW13 140, and 268 against 249 with long K.  The first two
// k tiles requested at once: UP 2 % slower, DW13 2 % faster.
constexpr int kMaxSlices = 8;
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

// The K slices of the tiles that DOWN has cut (see Cut), four workgroups to a tile, in slice order.
__global__ __launch_bounds__(kThreads) void f32_cut_finish_kernel(FArgs g) {
  const int xcd = blockIdx.x % 8, p = blockIdx.x / 32, quarter = blockIdx.x / 8 % 4;
  const RowTiles rt(g.offsets, g.E, kTile, threadIdx.x & (kWave - 1));
  const int total = rt.count() * g.tiles_n, share = (total + 7) / 8;
  const Cut cut(share);
  const int id = xcd * share + cut.whole + p;
  if (p >= cut.left || id >= total) return;
  int e, n_rows, tile_m, tile_n, row0, row_end;
  rt.expert_of(id, g.tiles_n, e, n_rows, tile_m);
  F32Gemm<DOWN, false>::in_bands(tile_m, g.tiles_n, n_rows, tile_m, tile_n);
  rt.rows_of(e, tile_m, row0, row_end);
  const int row = 16 * quarter + threadIdx.x / 16, col = 4 * (threadIdx.x % 16), m = row0 + row, n = tile_n * kTile + col;
  if (m >= row_end || n >= g.N) return;
  const float* from = g.cut() + (int64_t)((xcd * cut.left + p) * cut.slices) * (kTile * kTile) + row * kTile + col;
  f32x4 v[Cut::MOST];
#pragma unroll
  for (int s = 0; s < Cut::MOST; ++s) v[s] = *reinterpret_cast<const f32x4*>(from + min(s, cut.slices - 1) * (kTile * kTile));
#pragma unroll
  for (int s = 1; s < Cut::MOST; ++s)
#pragma unroll
    for (int x = 0; x < 4; ++x) v[0][x] += s < cut.slices ? v[s][x] : 0.f;
  *reinterpret_cast<f32x4*>(g.C0 + (int64_t)m * g.ldc + n) = v[0];
}

// tiles of N columns (rows of tile_cols) to expect: an expert's last row tile is half full on average
double expected_tiles(int R, int E, int N, int tile_cols) {
  const int busy = std::max(std::min(E, R), 1);
  return busy * std::max((double)R / busy / kTile + 0.5, 1.0) * ceil_div(N, tile_cols);
}

// K slices of DOWN and BWD_DX.  Few tiles of many k tiles leave compute units idle, or some with a tile more than others.
// Measured on 64 x 64 tiles of 32 k (64 to 2003 tokens, 8 experts of 512 x 1376, 1 to 4 slices): with r tiles on a compute unit a k
// tile takes 0.5 us for each of them, 0.7 us for a single one, which waits for memory; the slices' sums pass through memory once
// more, at about 8 TB/s, BWD_DX's in a launch of its own, DOWN's in the combine, to which a cut for less than a seventh is not
// worth it.  (DOWN + combine, us, without slices / as chosen here: 64 tokens 45 /
// 22, 512 45 / 29, 1024 57 / 43, 1536 58 / 58; BWD_DX 66 / 25, 66 / 45, 100 / 68, 104 / 90, 2003 tokens 136 / 112.)  Other layers agree:
// of 40 forward and 32 training passes of 16 to 2003 tokens, 2 to 8 experts of 64 to 512 x 64 to 1376, with every number of slices from 1 to 8,
// DOWN + combine are 1 % from the best on average, 10 % at most (1297 tokens, 2 experts of 392 x 464: 28.3 us, 4 slices 25.8), the joint
// launch of the backward pass 2.4 % and 16 % (750 tokens, 4 experts of 88 x 728: 29.8, 4 slices 25.6).
int f32_slices(int R, int E, int N, int K, bool two_passes, int most) {
  const double tiles = expected_tiles(R, E, N, kTile), nk = ceil_div(K, kTileK) * (two_passes ? 2.0 : 1.0);
  int best = 1;
  double best_us = 0, uncut_us = 0;
  for (int n = 1; n <= most; ++n) {
    if (n > 1 && ((two_passes && n % 2) || n > nk / 2 || (int64_t)n * R * N > kMaxSums)) continue;
    const double per_k = std::max(0.5 * std::ceil(tiles * n / 256), 0.7);
    const double us = per_k * (nk / n + 1) + (n > 1 ? (two_passes ? 5.0 : 1.0) + 5e-7 * n * (double)R * N : 0.0);
    if (n == 1) uncut_us = us;
    else if (!two_passes && us * 1.15 > uncut_us) continue;
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

// Is DOWN's last round worth a cut and the launch that adds it up (5 us)?  A unit that has one tile more than the others takes 0.5 us longer
// for each of its k tiles, a slice's part of that when it is cut.  The number of tiles moves by a row tile's columns with the routing:
// with fewer left than that there may be none.  us, whole / cut, forward call, top-2: 2003 tokens, 8 experts of 512 x 1376 (533 tiles) 159.5
// / 145.3 (DOWN 70 / 55.7 and 4.8 for the sums; training pass 534.5 / 522.4); of 512 x 688 91.6 / 85.8; 4006 of 256 x 1376 (517) 165.0 / 151.1;
// but 4 experts of 512 x 1376, 517 tiles expected and 512 there, 140.9 / 143.0.  Where one expert is favoured the cut is as good, as Cut counts
// the tiles that there are: of 60 calls (these three and 1100 of 1024 x 1376, a bias of 0 to 4 on expert 0) 58 gain 3 to 10 %, two without
// an uneven round lose 1 %.
bool f32_cut(const FfShapes& sh) {
  auto gains = [&](double slices) { return 0.5 * ceil_div(sh.f, kTileK) * (1.0 - 1.0 / slices) > 7.0; };
  if (!gains(Cut::MOST) || sums_bytes(sh, false) < (size_t)8 * Cut::UNITS * kTile * kTile * sizeof(float)) return false;
  const double rows = (double)sh.R / sh.E, spread = std::sqrt(2.0 * rows * (1.0 - 1.0 / sh.E));
  // row tiles of an expert, for rows spread at random: the first ones for certain (erfc(-8) is 2 to the last bit)
  const int sure = (int)(std::max(rows - 8 * spread, 0.0) / kTile);
  double row_tiles = sure;
  for (int j = sure; j < ceil_div(sh.R, kTile) && kTile * j < rows + 8 * spread; ++j)
    row_tiles += spread > 0 ? 0.5 * std::erfc((kTile * j + 0.5 - rows) / spread) : 1.0;
  const double tiles = std::round(row_tiles * sh.E) * ceil_div(sh.d, kTile), rounds = std::floor(tiles / 256), left = tiles - 256 * rounds;
  return rounds >= 1 && left >= ceil_div(sh.d, kTile) && left <= 120 && gains(std::min(std::floor(256 / left), (double)Cut::MOST));
}

// Do byte offsets from a tile's first row (gathered: from token 0) need more than 32 bits?  A tile spans 64 rows.
bool wide_offsets(const FArgs& g, int R) {
  const int64_t rows = g.perm ? std::max(ceil_div(R, g.k), kTile) : kTile;
  return rows * std::max(g.lda, g.ldb) >= ((int64_t)1 << 30) - 4096;
}

// UP with few workgroups on a compute unit and weights that come from memory, not from the memory-side cache (256 MB): one k tile on
// its way is too little.  us, two stages / three (in brackets: through registers, with two k tiles on their way), by the bytes of W1 and W3:
// 12 tokens of 5528, f = 216, 16 experts (153 MB) 141 / 117 (127); 37 of 3984, f = 216, 16 experts (110) 103 / 87 (94); 64 of 4096, f = 2048, 4
// experts (268) 109 / 92 (98); 55 of 4096, f = 344, 8 experts (90) 99 / 91 (96); but 32 of 4448, f = 1104, 2 experts (79) 94 / 99, 94 of 2096, f =
// 4072, 1 expert (68) 50 / 52, and with three workgroups on a unit 443 of 3824, f = 1488, 8 experts (752 tiles) 244 / 255.
bool weights_from_memory(const FArgs& g, int R) {
  return (int64_t)8 * std::min(g.E, R) * g.K * g.N >= 88000000 && expected_tiles(R, g.E, g.N, kTile / 2) <= 512;
}

// Completes the arguments of a product; its workgroups, 0: more than a launch can hold
template <int MODE> unsigned blocks_of(FArgs& g, int R) {
  using G = F32Gemm<MODE, false>;
  g.tiles_n = ceil_div(g.N, G::BNH);
  g.tiles_m = ceil_div(g.M, kTile);
  if (!G::SLICED) g.slices = 1;
  g.R = R;
  const int64_t tiles = (int64_t)(MODE == DW13 ? 2 * g.tiles_n : g.tiles_n) * g.slices *
                        (G::GROUP_K ? (int64_t)g.E * g.tiles_m : (int64_t)ceil_div(R, kTile) + g.E);   // at most this many
  const int64_t slices = MODE == DOWN && g.cut() ? 8 * Cut::UNITS : 0;   // of the tiles that are cut
  return grid_fits(tiles + slices + 7, kThreads) ? (unsigned)align_up((size_t)(tiles + slices), 8) : 0;
}
int finish_slices(const FArgs& g, int R, hipStream_t s) {
  f32_slices_finish_kernel<<<ceil_div((int64_t)R * g.N / 4, kThreads), kThreads, 0, s>>>(g.sums, g.slices, R, g.N, g.offsets, g.E, g.C0);
  BTX_LAUNCH_CHECK();
  return BTX_OK;
}
// left (may be NULL): in, K slices that the caller can add himself; out, those whose sums he finds in g.sums (1: none)
template <int MODE> int launch(FArgs g, int R, hipStream_t s, int* left = nullptr) {
  const unsigned grid = blocks_of<MODE>(g, R);
  if (grid == 0) return BTX_ERR_UNSUPPORTED;
  if (wide_offsets(g, R)) f32_gemm_kernel<MODE, true, 2><<<grid, kThreads, 0, s>>>(g);
  else if (MODE == UP && weights_from_memory(g, R)) f32_gemm_kernel<MODE, false, MODE == UP ? 3 : 2><<<grid, kThreads, 0, s>>>(g);
  else f32_gemm_kernel<MODE, false, 2><<<grid, kThreads, 0, s>>>(g);
  BTX_LAUNCH_CHECK();
  if (MODE == DOWN && g.cut()) {
    f32_cut_finish_kernel<<<8 * 4 * (Cut::UNITS / 2), kThreads, 0, s>>>(g);   // at most half of an XCD's units have a tile that is cut
    BTX_LAUNCH_CHECK();
  }
  const bool leave = left && g.slices <= *left;
  if (left) *left = leave ? g.slices : 1;
  return g.slices > 1 && !leave ? finish_slices(g, R, s) : BTX_OK;
}

// The whole feed-forward of a small layer (f32_ff_slices()) in one launch: UP and DOWN are two launches of about 5 us there, each a
// few k tiles long and bound by its waits for memory.  A workgroup of 4 wavefronts takes 16 grouped rows and 64 of the f columns: its piece
// of act stays in LDS, its products with the same 64 rows of W2 are a slice of y, which the combine adds up as it adds K slices.
// Weights go straight from memory to the registers as each is used once for the 16 rows, all of a piece requested together, W2's
// first while W1's and W3's are on their way; the wavefronts share the k of both products and add up their sums in LDS, in their
// order.  512 tokens of 64 columns, f = 176, 4 experts: the two launches and the combine 10.9 us, with this 7.7.
struct FfArgs {
  const float* x; const float* W1; const float* W3; const float* W2;
  const int32_t* perm; int k;            // row r is token perm[r] / k
  const int32_t* offsets; int E, d, f;
  int64_t s13, s2;                       // expert strides
  float* h1; float* h3;                  // [R, f] (NULL: not kept)
  float* sums; int R, slices;            // [slice][R, d]: of 64 f columns each, whoever reads them adds them up
};
constexpr int kFfRows = 16, kFfCols = 64;

__global__ __launch_bounds__(kThreads, 4) void f32_ff_kernel(FfArgs g) {
  constexpr int PITCH = kFfCols + 4;                     // floats of a row in LDS: 16 lanes of as many rows reach all banks
  __shared__ __attribute__((aligned(16))) float part[2][4][kFfRows * PITCH], act[kFfRows * PITCH];
  const int lane = threadIdx.x & (kWave - 1), r = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // each XCD takes one eighth of the ids: of an expert's 64 columns all row tiles, so that its L2 keeps their weights
  const RowTiles rt(g.offsets, g.E, kFfRows, lane);
  const int total = rt.count() * g.slices, share = (total + 7) / 8, pos = (int)(blockIdx.x / 8), id = (int)(blockIdx.x % 8) * share + pos;
  if (pos >= share || id >= total) return;
  int e, n_rows, local, row0, row_end;
  rt.expert_of(id, g.slices, e, n_rows, local);
  const int slice = local / n_rows, col0 = slice * kFfCols;
  rt.rows_of(e, local - slice * n_rows, row0, row_end);
  auto ld = [](const float* p, bool in) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p);
    return in ? v : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // a lane's 4 columns of 4 k rows: k rows 4 g4 + x and columns 4 r + j go to instruction x of fragment j
  const float* const W2 = g.W2 + e * g.s2;
  const int k2 = col0 + 16 * wave + 4 * g4;              // rows of W2, the wavefronts sharing the 64 out
  f32x4 w2[4];
  auto load_w2 = [&](int c0) {
#pragma unroll
    for (int x = 0; x < 4; ++x) w2[x] = ld(W2 + (int64_t)min(k2 + x, g.f - 1) * g.d + min(c0 + 4 * r, g.d - 4), k2 < g.f);
  };
  load_w2(0);
  const float* const xr = g.x + (int64_t)(g.perm[min(row0 + r, row_end - 1)] / g.k) * g.d;
  const int64_t panel = e * g.s13 + min(col0 + 4 * r, g.f - 4);
  f32x4 acc[2][4];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[p][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int s = wave; 16 * s < g.d; s += 4) {             // 16 k at a time, the wavefronts in turn
    const bool in = 16 * s + 4 * g4 < g.d;
    const int k = in ? 16 * s + 4 * g4 : 0;
    const f32x4 a = ld(xr + k, in);
    f32x4 b[2][4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      b[0][x] = ld(g.W1 + panel + (int64_t)(k + x) * g.f, in);
      b[1][x] = ld(g.W3 + panel + (int64_t)(k + x) * g.f, in);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[p][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[p][x][j], a[x], acc[p][j], 0, 0, 0);
  }
  // this lane's sums of row r: columns 16 g4 + 4 v + j
  auto put = [&](float* to, const f32x4 (&c)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) *reinterpret_cast<f32x4*>(to + r * PITCH + 16 * g4 + 4 * v) = f32x4{c[0][v], c[1][v], c[2][v], c[3][v]};
  };
  const int row = threadIdx.x >> 4, c4 = 4 * (threadIdx.x & 15), m = row0 + row;
  auto sum = [&](const float (&from)[4][kFfRows * PITCH]) {   // the wavefronts' sums, in their order
    f32x4 t = *reinterpret_cast<const f32x4*>(from[0] + row * PITCH + c4);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f32x4 u = *reinterpret_cast<const f32x4*>(from[w] + row * PITCH + c4);
#pragma unroll
      for (int x = 0; x < 4; ++x) t[x] += u[x];
    }
    return t;
  };
  put(part[0][wave], acc[0]);
  put(part[1][wave], acc[1]);
  __syncthreads();
  {
    const f32x4 h1 = sum(part[0]), h3 = sum(part[1]);
    const bool in = col0 + c4 < g.f;
    f32x4 a;
#pragma unroll
    for (int x = 0; x < 4; ++x) a[x] = in ? silu_f(h1[x]) * h3[x] : 0.f;
    *reinterpret_cast<f32x4*>(act + row * PITCH + c4) = a;
    if (g.h1 && in && m < row_end) {
      const int64_t at = (int64_t)m * g.f + col0 + c4;
      *reinterpret_cast<f32x4*>(g.h1 + at) = h1;
      *reinterpret_cast<f32x4*>(g.h3 + at) = h3;
    }
  }
  __syncthreads();
  const f32x4 a = *reinterpret_cast<const f32x4*>(act + r * PITCH + 16 * wave + 4 * g4);
  float* const out = g.sums + ((int64_t)slice * g.R + m) * g.d + c4;
  for (int c0 = 0, buf = 0; c0 < g.d; c0 += kFfCols, buf ^= 1) {
    f32x4 c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[x][j], a[x], c[j], 0, 0, 0);
    if (c0 + kFfCols < g.d) load_w2(c0 + kFfCols);
    put(part[buf][wave], c);
    __syncthreads();                                     // (the other half is free: its sums were read before this barrier)
    const f32x4 y = sum(part[buf]);
    if (m < row_end && c0 + c4 < g.d) *reinterpret_cast<f32x4*>(out + c0) = y;
  }
}

}  // namespace

// Small layers, up to 192 columns and 47 million products (rows x d x f, at least 64 columns of f, which a workgroup takes), by 95 forward
// calls of 16 to 2003 tokens, 2 to 8 experts, on both ways (us, UP and DOWN / joint): 512 tokens of 64, f = 176, 4 experts 10.9 / 7.7; 77 of 64,
// f = 208, 5 11.0 / 7.4; 1000 of 64, f = 128, 8, top-4 13.1 / 9.1; 458 of 96, f = 208, 2 12.2 / 10.0; 249 of 128, f = 664, 4 (42 million) 14.0 /
// 12.9; 69 of 192, f = 192, 5 12.4 / 11.7.  Above, 16 rows to a tile read the weights too often, and wide rows are a chain of passes: 400 of
// 192, f = 320, 5 (49) 14.7 / 14.8; 547 of 232, f = 240, 5 (61) 16.6 / 17.7; 1064 of 144, f = 208, 5 (64) 15.6 / 18.0; 1349 of 168, f = 416, 5
// (189) 26.7 / 31.7; 100 of 504, f = 64, 2 19.2 / 22.7; 13020 of 192, f = 8, 1 21.5 / 26.5.  And up to 16000 rows times pieces of 64 columns: four
// times as many workgroups as tiles of 64 rows make, no more than run at once (1024).  Of narrow rows, by 1875 calls of 16 to 300000 tokens, 1 to
// 64 experts, 8 to 240 x 8 to 2560: 46875 of 16, f = 8, 1 expert 19.0 / 24.2; 183593 of 32, f = 8, 1 58.7 / 89.0; 14687 of 8, f = 200, 1 33.4 / 43.5;
// 10374 of 24, f = 72, 3 14.0 / 15.8.  Of those that the rule takes five are more than 2 % slower, 2148 of 160, f = 16, 32, top-2 the most (13.4 /
// 14.7); on average of all calls it leaves 1 % to the better way.
int f32_ff_slices(const FfShapes& sh, int64_t most) {
  const int slices = ceil_div(sh.f, kFfCols);
  const bool small = (int64_t)sh.R * sh.d * std::max(sh.f, kFfCols) <= 47000000 && (int64_t)sh.R * slices <= 16000;
  return sh.d <= 192 && small && slices <= most ? slices : 0;
}
int f32_ff(const RowSource& xs, const void* W1, const void* W3, const void* W2, const int32_t* off, const FfShapes& sh, void* h1, void* h3,
           void* sums, hipStream_t s) {
  FfArgs g{(const float*)xs.base, (const float*)W1, (const float*)W3, (const float*)W2, xs.perm, xs.k, off, sh.E, sh.d, sh.f, sh.s13, sh.s2,
           (float*)h1, (float*)h3, (float*)sums, sh.R, ceil_div(sh.f, kFfCols)};
  const int64_t blocks = ((int64_t)ceil_div(sh.R, kFfRows) + sh.E) * g.slices;
  if (!grid_fits(blocks + 7, kThreads)) return BTX_ERR_UNSUPPORTED;
  f32_ff_kernel<<<(unsigned)align_up((size_t)blocks, 8), kThreads, 0, s>>>(g);
  BTX_LAUNCH_CHECK();
  return BTX_OK;
}

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
  if (g.slices == 1 && f32_cut(sh)) g.C2 = g.sums;
  g.A0 = (const float*)act; g.B0 = (const float*)W2; g.C0 = (float*)y;
  g.offsets = off; g.E = sh.E; g.N = sh.d; g.K = sh.f; g.lda = sh.f; g.ldb = sh.d; g.ldc = sh.d; g.strideB_e = sh.s2;
  return launch<DOWN>(g, sh.R, s, slices);
}
int f32_bwd_act(const RowSource& dys, const void* W2, const void* h1, const void* h3, const float* gates,
                const int32_t* perm, const int32_t* off, const FfShapes& sh, void* dh1, void* dh3, void* ga,
                uint32_t* row_bytes, float* dg_part, hipStream_t s) {
  FArgs g{};
  g.row_bytes = row_bytes;
  g.A0 = (const float*)dys.base; g.gather(dys); g.B0 = (const float*)W2;
  g.C0 = (float*)dh1; g.C1 = (float*)dh3; g.C2 = (float*)ga;
  g.H1 = (const float*)h1; g.H3 = (const float*)h3; g.gates = gates; g.perm_pairs = perm; g.dg_part = dg_part;
  g.n_part = f32_bwd_act_partials(sh.f);
  g.offsets = off; g.E = sh.E; g.N = sh.f; g.K = sh.d; g.lda = sh.d; g.ldb = sh.d; g.ldc = sh.f; g.strideB_e = sh.s2;
  return launch<BWD_ACT>(g, sh.R, s);
}
namespace {
FArgs bwd_dx_args(const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh, void* dxs,
                  void* sums) {
  FArgs g{};
  g.slices = slices_of(sh, true); g.sums = (float*)sums;
  g.A0 = (const float*)dh1; g.A1 = (const float*)dh3; g.B0 = (const float*)W1; g.B1 = (const float*)W3; g.C0 = (float*)dxs;
  g.offsets = off; g.E = sh.E; g.N = sh.d; g.K = sh.f; g.lda = sh.f; g.ldb = sh.f; g.ldc = sh.d; g.strideB_e = sh.s13;
  return g;
}
}  // namespace
int f32_bwd_dx(const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh,
               void* dxs, void* sums, hipStream_t s) {
  return launch<BWD_DX>(bwd_dx_args(dh1, dh3, W1, W3, off, sh, dxs, sums), sh.R, s);
}
int f32_bwd_dx_dw(const RowSource& xs, const RowSource& dys, const void* dh1, const void* dh3, const void* ga, const void* W1,
                  const void* W3, const int32_t* off, const FfShapes& sh, uint32_t* row_bytes, void* dxs, void* sums, void* dW1,
                  void* dW3, void* dW2, const RouterDs* ds, hipStream_t s) {
  FArgs dx = bwd_dx_args(dh1, dh3, W1, W3, off, sh, dxs, sums), dw13{}, dw2{};
  dw13.row_bytes = dw2.row_bytes = row_bytes;
  dw13.A0 = (const float*)xs.base; dw13.gather(xs); dw13.B0 = (const float*)dh1; dw13.B1 = (const float*)dh3;
  dw13.C0 = (float*)dW1; dw13.C1 = (float*)dW3;
  dw13.offsets = off; dw13.E = sh.E; dw13.M = sh.d; dw13.N = sh.f; dw13.lda = sh.d; dw13.ldb = sh.f; dw13.ldc = sh.f; dw13.strideC_e = sh.s13;
  dw2.A0 = (const float*)ga; dw2.B0 = (const float*)dys.base; dw2.gather(dys); dw2.C0 = (float*)dW2;
  dw2.offsets = off; dw2.E = sh.E; dw2.M = sh.f; dw2.N = sh.d; dw2.lda = sh.f; dw2.ldb = sh.d; dw2.ldc = sh.d; dw2.strideC_e = sh.s2;
  const unsigned n_dx = blocks_of<BWD_DX>(dx, sh.R), n13 = blocks_of<DW13>(dw13, sh.R), n2 = blocks_of<DW2>(dw2, sh.R);
  if (n_dx == 0 || n13 == 0 || n2 == 0) return BTX_ERR_UNSUPPORTED;
  const RouterDs rd = ds ? *ds : RouterDs{};
  const unsigned nds = ds ? router_ds_blocks(rd) : 0;
  const bool wide = wide_offsets(dx, sh.R) || wide_offsets(dw13, sh.R) || wide_offsets(dw2, sh.R);
  auto go = [&](unsigned a, unsigned b, unsigned c, unsigned d) -> int {
    if (a + b + c + d == 0) return BTX_OK;
    if (wide) f32_dx_dw_kernel<true><<<a + b + c + d, kThreads, 0, s>>>(dx, a, dw13, b, dw2, c, rd);
    else f32_dx_dw_kernel<false><<<a + b + c + d, kThreads, 0, s>>>(dx, a, dw13, b, dw2, c, rd);
    BTX_LAUNCH_CHECK();
    return BTX_OK;
  };
  if (grid_fits((int64_t)n_dx + n13 + n2 + nds, kThreads)) {
    if (int rc = go(n_dx, n13, n2, nds)) return rc;
  } else {                                               // one after another: each of them fits
    if (int rc = go(0, 0, 0, nds)) return rc;
    if (int rc = go(n_dx, 0, 0, 0)) return rc;
    if (int rc = go(0, n13, 0, 0)) return rc;
    if (int rc = go(0, 0, n2, 0)) return rc;
  }
  return dx.slices > 1 ? finish_slices(dx, sh.R, s) : BTX_OK;
}

}  // namespace btx
