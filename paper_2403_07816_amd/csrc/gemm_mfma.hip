// bf16 MFMA grouped GEMMs of the expert FFNs (the SwiGLU feed-forward FF_i of the layer
// equation in Sec. 3.2, forward and backward), written for gfx950.
//
// One kernel template covers the six products of the layer:
//   UP      h1 = xs W1_e, h3 = xs W3_e, act = silu(h1)*h3          (two B panels share one A tile)
//   DOWN    y = act W2_e
//   BWD_ACT D = dys W2_e^T with the SwiGLU backward fused into the epilogue
//   BWD_DX  dxs = dh1 W1_e^T + dh3 W3_e^T                           (two K passes, one accumulator)
//   DW13    dW1_e = xs_e^T dh1_e, dW3_e = xs_e^T dh3_e              (K = the expert's ragged row count)
//   DW2     dW2_e = ga_e^T dys_e
//
// Structure of a workgroup (WM x WN wavefronts, BM x BN x BK tile):
//   * global -> LDS copies are direct (global_load_lds, 16 bytes per lane, no VGPR staging),
//     three stages of the A tile and two of the B tile; the two wavefronts of a SIMD alternate
//     between a memory phase and a compute phase (see the main loop);
//   * an operand whose K index is contiguous in memory is stored [row][BK] with a 16-byte
//     chunk XOR swizzle and read with ds_read_b128; an operand whose K index is strided
//     (the weights in UP and DOWN, dh1/dh3 in DW13, token rows of dY in DW2) is stored as it lies in memory,
//     [BK][cols], and read with the transposing ds_read_b64_tr_b16; x, ga and, where mfma_dw2_rows() has it so,
//     dY reach the dW products of many rows per expert transposed and zero-padded (x and dY from a gather
//     kernel, ga written that way by BWD_ACT's epilogue; see DwStrip for few rows).  The swizzles are applied by choosing which
//     global chunk each lane fetches, since a direct copy fixes the LDS position per lane;
//   * v_mfma_f32_16x16x32_bf16 (on this chip it sustains a seventh more than the 32x32x16 form
//     under the same power limit) with the roles of the operands swapped (the N-side fragment
//     is passed first), so that each lane ends up with 4 consecutive output columns of one row
//     and stores 8 bytes at a time;
//   * grouped rows: tiles are enumerated per expert on the device (no host sync); a tile past
//     the last one exits.  Rows beyond a group's end are loaded from a clamped address and
//     never stored.  A last k tile that K fills only partly (K is a multiple of 8) has its copies
//     re-pointed at valid data and the A fragments past K zeroed in registers;
//   * few rows per expert (decoding, prompts, many narrow experts): the products stream the weights from HBM and
//     the matrix cores wait, so the same code runs with smaller tiles and deeper prefetch (see row_tile());
//   * UP, DOWN and BWD_DX: the tiles of a partly filled last round of workgroups are cut along K into
//     up to 8 slices whose fp32 accumulators a second small kernel adds in ascending order and stores
//     (UP: with the SwiGLU applied to the sums), so that the round fills the chip (Gemm::split_plan).
#include "gemm_mfma.h"
#include "router_ds.h"
#include <cmath>
#include <type_traits>

namespace btx {

// fp32 accumulators of the K slices of the last round of UP / DOWN / BWD_DX: at most cus + 8 * 8 (tile, slice) pairs
// of 256 x 256 floats.  Small tiles keep their slices' sums here too, as many as fit (see split_bytes()).
constexpr int kSplitMaxSlices = 8;
constexpr int kSplitMaxCus = 256;   // compute units the K-cut of a last round is laid out for (see Gemm::split_plan)
constexpr size_t kSplitBytes = (size_t)(kSplitMaxCus + 8 * kSplitMaxSlices) * 256 * 256 * sizeof(float);

namespace {

// supertile: row tiles x column tiles that run concurrently chip-wide, and the XCDs along its
// rows (8 / kXcdM along its columns)
constexpr int kSupM = 16, kSupN = 16, kXcdM = 4;
static_assert(kSupM % kXcdM == 0 && 8 % kXcdM == 0 && kSupN % (8 / kXcdM) == 0 && (kSupM * kSupN) % 8 == 0, "supertile");

enum Mode { UP = 0, DOWN = 1, BWD_ACT = 2, BWD_DX = 3, DW13 = 4, DW2 = 5 };

struct MArgs {
  const bf16_t* A0; const bf16_t* A1;   // A1: second K pass (BWD_DX)
  const bf16_t* B0; const bf16_t* B1;   // B1: second panel (UP, DW13) or second K pass (BWD_DX)
  void* C0; void* C1; void* C2;         // UP: h1,h3,act; BWD_ACT: dh1,dh3,ga (or NULL, see T2); DW13: dW1,dW3; else C0
  const bf16_t* H1; const bf16_t* H3;   // BWD_ACT inputs
  bf16_t* T2; int ldt;                  // BWD_ACT: ga transposed [N][ldt], experts' rows padded to 64 (NULL: ga goes to C2, if at all)
  const float* gates; const int32_t* perm; float* dg_part; int n_part;
  const int32_t* a_perm; int a_k;       // UP / BWD_ACT: A row r is row a_perm[r] / a_k of A0 (NULL: row r)
  const int32_t* offsets; int E;
  int M, N, K;                          // grouped-M: M unused; grouped-K: K unused
  int lda, ldb, ldc;                    // leading dimensions in elements
  int ldp;                              // of the rows of f that stay inside the library: UP's act, BWD_ACT's dh1, dh3 and ga (mfma_act_pitch())
  int64_t strideB_e, strideC_e;         // per-expert strides in elements
  int R;                                // total grouped rows
  int tiles_n, tiles_m;                 // tile grid (tiles_m is the worst case for grouped-M)
  int c_is_f32;
  int blocks_per_e;                     // grouped-K: block ids per expert (a multiple of 8)
  int total_ids;                        // tile ids of the launch (a few name no tile: padding of the id space)
  // UP / DOWN / BWD_DX: the tiles of the last, partly filled round are cut along K (see Gemm::split_plan)
  f32x4* partial; int cus;              // fp32 accumulators of the slices (NULL: never cut); compute units
  uint32_t* row_bytes;                  // byte offset of every grouped row's token row: BWD_ACT writes it for the weight gradients
  // small tiles: every tile of the launch is cut into `slices` K ranges; slices > 1: fp32 sums in slice_sums,
  // [slice][panel][R][N]
  int slices; float* slice_sums;
};

// Direct global -> LDS copy of 16 bytes per lane: lane l's data lands at lds_base + 16*l.
// Written as inline assembly so that the compiler does not serialise later LDS reads of
// *other* stages behind it (it cannot tell the stages apart and would wait for vmcnt(0));
// completion is awaited explicitly with wait_vmcnt() before the barrier that publishes a tile.
// `base` and `lds_base` are wave-uniform by construction; readfirstlane states that to the
// compiler where its divergence analysis cannot see it.
// STREAM: past the L1 and marked for early eviction in the L2, for bytes that are read once.
template <bool STREAM = false>
__device__ __forceinline__ void copy16_to_lds(const void* base, uint32_t byte_off, uint32_t lds_base) {
  const uint64_t sp = uniform64(base);
  const uint32_t sl = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_base);
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 sc1 nt"
                 :
                 : "s"(sl), "v"(byte_off), "s"(sp)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(sl), "v"(byte_off), "s"(sp)
                 : "memory");
}

// N copies of 1 KB by one wavefront, to lds, lds + 1024, ... : the offset of the instruction counts in memory as in LDS, so that
// all of them share one setting of m0 and one base, and the lanes' offsets make up for it: copy q of bytes at `off` from the
// operand is given base - copy_bias(N) and copy_off<N>(off, q).  (A setting of m0 and a base of their own took each copy 8 scalar
// instructions, which the other wavefront's products wait for.)
constexpr uint32_t copy_bias(int n) { return 1024u * (n - 1); }
constexpr uint32_t kCopyBias = copy_bias(4);             // of the most copies
template <int N, typename Off> __device__ __forceinline__ constexpr Off copy_off(Off off, int q) { return off + (copy_bias(N) - 1024u * q); }
#define BTX_COPY(q, reg, flags) "\n\tglobal_load_lds_dwordx4 %" #reg ", %1 offset:" #q flags
#define BTX_COPIES(flags)                                                                                                           \
  static_assert(N >= 2 && N <= 4, "copies");                                                                                        \
  if constexpr (N == 2)                                                                                                             \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" BTX_COPY(0, 2, flags) BTX_COPY(1024, 3, flags)                                       \
                 : : "s"(lds), "s"(base), "v"(off[0]), "v"(off[1]) : "memory");                                                     \
  else if constexpr (N == 3)                                                                                                        \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" BTX_COPY(0, 2, flags) BTX_COPY(1024, 3, flags) BTX_COPY(2048, 4, flags)              \
                 : : "s"(lds), "s"(base), "v"(off[0]), "v"(off[1]), "v"(off[2]) : "memory");                                        \
  else                                                                                                                              \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" BTX_COPY(0, 2, flags) BTX_COPY(1024, 3, flags) BTX_COPY(2048, 4, flags)              \
                     BTX_COPY(3072, 5, flags)                                                                                       \
                 : : "s"(lds), "s"(base), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]) : "memory")
template <int N, bool STREAM> __device__ __forceinline__ void copies_to_lds(uint64_t base, const uint32_t* off, uint32_t lds) {
  if constexpr (STREAM) { BTX_COPIES(" sc1 nt"); } else { BTX_COPIES(""); }
}
#undef BTX_COPIES
#undef BTX_COPY
// The same with offsets of 64 bits (wide_offsets())
template <int N, bool STREAM> __device__ __forceinline__ void copies_to_lds(uint64_t base, const uint64_t* off, uint32_t lds) {
  static_assert(!STREAM, "copies");
#pragma unroll
  for (int q = 0; q < N; ++q)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 : : "s"(lds + 1024u * q), "v"(base + off[q] + 1024u * q) : "memory");
}

// Epilogue staging band: 32 rows of ROWB bytes in LDS, 16-byte chunks XOR-swizzled by row so
// that both the piece writes (PIECE bytes per lane, 32 rows at one column) and the
// row-contiguous 16-byte reads are free of bank conflicts.
template <int ROWB, int PIECE>
__device__ __forceinline__ uint32_t stage_off(int r, int chunk) {
  constexpr int CPR = ROWB / 16, RP = ROWB >= 256 ? 1 : 256 / ROWB, STEP = PIECE / 8;
  return (uint32_t)(r * ROWB + ((chunk ^ (((r / RP) * STEP) & (CPR - 1))) << 4));
}

// The 8-byte pieces that the lanes of a fragment write into (and read from) a staged band would
// meet two-way in the banks: rows r and r+1 (128-byte rows) or r and r+2 (64-byte rows) of a band
// put the same chunk in the same banks.  Those rows keep the two halves of every 16-byte chunk
// swapped, so that 16 lanes cover all 32 banks; whoever moves whole chunks swaps them back.
// BWD_ACT does without: its epilogue is bound by its vector arithmetic (about 3000 instructions
// per wavefront), the swaps would add 256 selects to it and its LDS conflicts cost no time.
template <int ROWB, int ES>
__device__ __forceinline__ uint32_t half_flip(int r) {
  return ES == 2 ? (uint32_t)(((r >> (ROWB >= 128 ? 0 : 1)) & 1) << 3) : 0u;
}
__device__ __forceinline__ u32x4 swap_halves(u32x4 v, bool yes) {
  return yes ? u32x4{v[2], v[3], v[0], v[1]} : v;
}

// Epilogue stores.  STREAM: marked non-temporal, so that the written tile does not push the operand panels
// that the other compute units are streaming out of the XCD's L2.  Measured per product: BWD_ACT (three
// tensors out per tile, the lowest L2 hit rate of the six) -5 %, DOWN -0.3 % (-3.7 % with 32 narrow experts);
// BWD_DX +0.6 % / -2 %, UP and DW13 +1 %: those keep plain stores.  DW2: see launch_dw().
template <bool STREAM, typename V> __device__ __forceinline__ void store_out(V* p, V v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// TAIL: see run(); kWideTail: any K, and operands whose rows lie too far apart for 32-bit offsets inside a tile
constexpr int kWideTail = 3;
// STREAM_B: the weights past the caches (stream_weights()); ROWS: DW2 whose B is token rows (mfma_dw2_rows())
template <int BM, int BN, int BK, int WM, int WN, int NSA, int NSB, int MODE, int TAIL = 0, bool STREAM_B = false,
          bool STREAM = MODE == BWD_ACT || MODE == DOWN, bool ROWS = false>
struct Gemm {
  // K index contiguous in memory?  A always is.  In the dW products K is the grouped-row index:
  // x (dW1/dW3) and ga, dY (dW2) arrive here transposed, [columns][padded rows], every expert's rows
  // starting at a multiple of 64 and zero-filled up to the next one; dh1/dh3 stay row-major, and so do the token rows of ROWS.
  static constexpr bool A_KC = true;
  static constexpr bool B_KC = (MODE != UP && MODE != DOWN && MODE != DW13 && !ROWS);
  static_assert(!ROWS || MODE == DW2, "token rows as B");
  static constexpr bool DUAL = (MODE == UP || MODE == DW13);
  static constexpr bool GROUP_K = (MODE == DW13 || MODE == DW2);
  typedef std::conditional_t<TAIL == kWideTail, uint64_t, uint32_t> Off;   // bytes from the base of a tile's copies on
  static_assert(TAIL != kWideTail || (BN == 128 && !STREAM_B), "only small tiles come in this form");
  // 128-column tiles: one pipeline for all wavefronts, two workgroups of four per compute unit; 256: ping-pong
  static constexpr bool SMALL = BN == 128;
  static constexpr int NW = WM * WN, NT = NW * kWave;
  static constexpr int TM = BM / WM / 16;                      // 16-row fragments per wavefront
  static constexpr int TN = BN / WN / 16;
  static constexpr int TNH = DUAL ? TN / 2 : TN;
  static constexpr int BNH = DUAL ? BN / 2 : BN;               // output columns per B panel
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  // LDS: NSA stages of the A tile, then NSB of the B tile
  static constexpr int B_BASE = NSA * A_BYTES;
  static constexpr int LDS_BYTES = NSA * A_BYTES + NSB * B_BYTES;
  static_assert(BK == 64 && (SMALL ? NW == 4 && !GROUP_K && NSB >= NSA && NSA >= 2
                                   : NW == 8 && ((NSA == 3 && NSB == 2) || (NSA == 2 && NSB == 3))),
                "the ping-pong schedule is written for 8 wavefronts, 2 k steps");
  static_assert(LDS_BYTES <= (SMALL ? 80 : 160) * 1024, "LDS");
  static constexpr int A_LOADS = A_BYTES / 1024 / NW, B_LOADS = B_BYTES / 1024 / NW;  // per wavefront per tile
  static constexpr int KSTEPS = BK / 32;                       // k steps (one MFMA deep) per tile
  static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "tile must split into 1 KB wave copies");
  static_assert(TM >= 2 && TM % 2 == 0 && TN >= 1 && (!DUAL || TN % 2 == 0), "bad wave tiling");

  // ---- LDS addressing ----------------------------------------------------
  // K-contiguous tile: [rows][BK], 16-byte chunks XOR-swizzled by row
  static __device__ __forceinline__ int kc_swz(int row) { return (row >> 1) & 7; }
  // strided-K tile: [BK][COLS], 16-byte chunk index XORed with tr_swz(k): bits 2-3 keep the four
  // k rows of one transposing read apart, bit 1 the two 16-lane groups that share a pass
  // (64 columns: the rows are half as long, so that bit 0 of k keeps two rows apart by itself)
  template <int COLS> static __device__ __forceinline__ int tr_swz(int k) {
    return COLS >= 128 ? ((k & 3) << 2) | (((k >> 3) & 1) << 1) : (((k >> 1) & 1) << 2) | (((k >> 3) & 1) << 1);
  }

  // byte offset inside a wave's copy `seg` (1 KB each) -> global element offset, for both layouts
  template <bool KC, int ROWS_OR_COLS>
  static __device__ __forceinline__ void copy_coords(int seg, int lane, int& major, int& minor_elem) {
    const int o = seg * 1024 + lane * 16;
    if (KC) {
      const int row = o / (BK * 2);
      const int phys = (o % (BK * 2)) / 16;
      major = row;                              // row of the tile (M or N index)
      minor_elem = (phys ^ kc_swz(row)) * 8;    // k offset inside the tile
    } else {
      constexpr int PITCH = ROWS_OR_COLS * 2;
      const int k = o / PITCH;
      const int phys = (o % PITCH) / 16;
      major = k;                                // k row of the tile
      minor_elem = (phys ^ tr_swz<ROWS_OR_COLS>(k)) * 8;      // column offset inside the tile
    }
  }

  // fragment of 16 rows x 32 k: lane l holds row l % 16, k = 32 ks + 8 (l / 16) .. + 7
  static __device__ __forceinline__ uint32_t kc_at(int row, int ks, int lane) {
    const int r = row + (lane & 15);
    const int chunk = 4 * ks + (lane >> 4);
    return (uint32_t)(r * (BK * 2) + ((chunk ^ kc_swz(r)) << 4));
  }
  static __device__ __forceinline__ bf16x8 read_kc(const char* tile, int row, int ks, int lane) {
    return *reinterpret_cast<const bf16x8*>(tile + kc_at(row, ks, lane));
  }
  template <int COLS> static __device__ __forceinline__ uint32_t tr_at(int col, int ks, int lane) {
    // a transposing read hands lane 4a+b of a 16-lane group element b of what lanes a, a+4, a+8,
    // a+12 fetched (4 consecutive columns each): lane r fetches k row r/4 at columns 4 (r%4) ..
    const int g = lane >> 4, r = lane & 15;
    const int k = 32 * ks + 8 * g + (r >> 2);
    const int c = col + 4 * (r & 3);
    return (uint32_t)(k * (COLS * 2) + ((((c >> 3) ^ tr_swz<COLS>(k)) << 4) | ((c & 7) << 1)));
  }
  template <int COLS>
  static __device__ __forceinline__ bf16x8 read_tr(const char* tile, int col, int ks, int lane) {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const char* at = tile + tr_at<COLS>(col, ks, lane);
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)at);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(at + 4 * COLS * 2));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }

  // ---- which tile ------------------------------------------------------
  // Workgroups are dealt round-robin to the 8 XCDs (block id mod 8) and start in id order.
  // SM x SN consecutive ids form one supertile of the tile grid, so that the tiles running at
  // any moment share few operand panels chip-wide (little HBM / infinity-cache traffic, short
  // miss latency); inside it XCD x owns a (SM/XM) x (SN/XN) sub-block, so that the panels its
  // CUs stream meet in that XCD's L2.  Only whole supertiles are laid out like this.  The
  // tiles right of and below the last whole supertile form one list (right strip row by row,
  // then the bottom strip column by column) that is cut into 8 equal runs, one per XCD: a
  // ragged edge must not leave some XCDs with fewer tiles than others.  The number of row
  // tiles of the row-grouped products depends on the routing and is counted here.
  struct Tile { int e, row0, row_end, k_begin, k_end, kp_begin, tile_n, exp_row0; };
  // Row-grouped products: the experts' row ranges are looked at by the whole wavefront at once, lane x
  // taking expert x (at most 64): one load and two prefix sums instead of loops of dependent scalar
  // loads over the experts, which with 32 experts took longer than a tenth of a short tile's main loop.
  // (The products grouped along K know their expert from the block id and keep the one short loop.)
  struct Experts {
    int o0, o1, nt, pad, nt_incl, pad_incl, n_rt;
    __device__ __forceinline__ Experts(const MArgs& g, int lane) : o0(0), o1(0), nt(0), pad(0), nt_incl(0), pad_incl(0) {
      n_rt = g.tiles_m;
      if (!GROUP_K) {
        const int xe = min(lane, g.E - 1);
        o0 = g.offsets[xe];
        o1 = g.offsets[xe + 1];
        const int x_n = lane < g.E ? o1 - o0 : 0;
        nt = (x_n + BM - 1) / BM;
        pad = (x_n + 63) & ~63;
        nt_incl = wave_incl_scan_i32(nt, lane);                              // row tiles up to and including expert x
        if (MODE == BWD_ACT) pad_incl = wave_incl_scan_i32(pad, lane);       // padded rows likewise
        n_rt = __builtin_amdgcn_readlane(nt_incl, kWave - 1);
      }
    }
  };
  // tile id -> tile; false: the id names no tile (all 64 lanes must be active)
  static __device__ __forceinline__ bool locate(const MArgs& g, const Experts& x, int id, Tile& t) {
    constexpr int SM = kSupM, SN = kSupN, XM = kXcdM, XN = 8 / XM;
    const int n_rt = x.n_rt;
    const int fr = n_rt / SM, fc = g.tiles_n / SN;     // whole supertile rows / columns
    const int blocks_full = fr * fc * SM * SN;
    int e = 0;
    if (GROUP_K) {
      e = id / g.blocks_per_e;
      id -= e * g.blocks_per_e;
    }
    int tile_m, tile_n;
    if (id < blocks_full) {
      const int sup = id / (SM * SN), r = id % (SM * SN);
      const int xcd = r % 8, slot = r / 8, sub_m = SM / XM, sub_n = SN / XN;
      tile_m = (sup / fc) * SM + (xcd % XM) * sub_m + slot % sub_m;
      tile_n = (sup % fc) * SN + (xcd / XM) * sub_n + slot / sub_m;
    } else {
      const int idl = id - blocks_full;
      const int w = g.tiles_n - fc * SN, h = n_rt - fr * SM;   // strip width / height
      const int n_right = fr * SM * w, n_left = n_right + h * g.tiles_n;
      const int run = (n_left + 7) / 8;
      const int l = (idl % 8) * run + idl / 8;
      if (idl / 8 >= run || l >= n_left) return false;
      if (l < n_right) {
        tile_m = l / w;
        tile_n = fc * SN + l % w;
      } else {
        tile_m = fr * SM + (l - n_right) % h;
        tile_n = (l - n_right) / h;
      }
    }
    t.kp_begin = 0;                                     // first padded row of expert e (transposed operand)
    t.exp_row0 = 0;
    if (GROUP_K) {
      t.row0 = tile_m * BM;
      t.row_end = g.M;
      t.k_begin = g.offsets[e];
      t.k_end = g.offsets[e + 1];
      t.kp_begin = padded_rows_before(g, e, threadIdx.x & (kWave - 1));
    } else {
      // the expert whose row tiles include tile_m: the first lane whose running total exceeds it
      const unsigned long long owners = __ballot(x.nt_incl > tile_m);
      if (owners == 0) return false;                    // past the last row tile of this routing
      e = __ffsll((long long)owners) - 1;
      const int tt = tile_m - (__builtin_amdgcn_readlane(x.nt_incl, e) - __builtin_amdgcn_readlane(x.nt, e));
      t.exp_row0 = __builtin_amdgcn_readlane(x.o0, e);
      t.row0 = t.exp_row0 + tt * BM;
      t.row_end = __builtin_amdgcn_readlane(x.o1, e);
      t.k_begin = 0;
      t.k_end = g.K;
    }
    if (MODE == BWD_ACT)                                // where expert e starts in the transposed, padded output
      t.kp_begin = __builtin_amdgcn_readlane(x.pad_incl, e) - __builtin_amdgcn_readlane(x.pad, e);
    t.e = e;
    t.tile_n = tile_n;
    return true;
  }

  // first padded row of expert e in the transposed operands (all 64 lanes active)
  static __device__ __forceinline__ int padded_rows_before(const MArgs& g, int e, int lane) {
    int p = 0;
    if (g.E <= 8) {                                      // with 64 experts the loop cost DW13 and DW2 7 %
      for (int q = 0; q < e; ++q) p += (g.offsets[q + 1] - g.offsets[q] + 63) & ~63;
    } else {
      p = lane < e ? (g.offsets[lane + 1] - g.offsets[lane] + 63) & ~63 : 0;
      p = __builtin_amdgcn_readlane(wave_incl_scan_i32(p, lane), kWave - 1);
    }
    return p;
  }
  // Small tiles: every XCD takes one eighth of the ids, one after another: K slice by K slice of an expert, its row
  // tiles fastest, so that what an XCD runs at a time reads a piece of the weights from HBM once and long rows of it.
  static __device__ __forceinline__ bool locate_small(const MArgs& g, int lane, Tile& t, int& slice) {
    const RowTiles rt(g.offsets, g.E, BM, lane);
    const int per_row_tile = g.tiles_n * g.slices, total = rt.count() * per_row_tile;
    const int share = (total + 7) / 8, pos = (int)(blockIdx.x / 8), id = (int)(blockIdx.x % 8) * share + pos;
    if (pos >= share || id >= total) return false;
    int n_rows, local;
    rt.expert_of(id, per_row_tile, t.e, n_rows, local);
    slice = local / (g.tiles_n * n_rows);
    local -= slice * g.tiles_n * n_rows;
    t.tile_n = local / n_rows;
    rt.rows_of(t.e, local - t.tile_n * n_rows, t.row0, t.row_end);
    t.exp_row0 = __builtin_amdgcn_readlane(rt.o0, t.e);
    t.k_begin = 0;
    t.k_end = g.K;
    t.kp_begin = MODE == BWD_ACT ? padded_rows_before(g, t.e, lane) : 0;
    return true;
  }

  // DOWN and BWD_DX have few, long tiles (16 column tiles): their last round is often a small fraction of
  // the chip (8.25 rounds for the benchmark's top-2 layer, 4.1 for top-1, 2.25 for one sequence), and a
  // tile cannot be cut smaller; UP has 44.3, 22.2 and 11.4 rounds there.  So the tiles of that round are cut
  // along K instead: slice s of a
  // left-over tile runs k tiles [s nk/S, (s+1) nk/S) in a workgroup of its own and leaves its fp32
  // accumulators in `partial`; a second, small kernel adds the S slices of a tile in slice order and stores
  // the result.  No atomics, and the order of every sum is fixed by the shapes and the number of compute
  // units alone.  ids >= total_ids are the workgroups of the slices 1 .. S-1.
  static constexpr bool SPLIT = !SMALL && (MODE == DOWN || MODE == BWD_DX || MODE == UP);
  static constexpr int kMaxSlices = kSplitMaxSlices, kMinSliceTiles = 16, kIdHoles = 8;   // the id space has up to 8 ids past the last tile
  struct SplitPlan { int id_full, n_left, n_slices; };
  static __device__ __forceinline__ SplitPlan split_plan(const MArgs& g, int n_rt) {
    SplitPlan p{0, 0, 1};
    if (!SPLIT || !g.partial) return p;
    const int n_real = n_rt * g.tiles_n;
    p.id_full = n_real / g.cus * g.cus;                 // ids below this fill whole rounds
    const int left = n_real - p.id_full;
    if (left == 0) return p;
    p.n_left = left + kIdHoles;                         // ids id_full .. id_full + n_left - 1 may name a tile
    // as many slices as fill the chip, at most eight, none shorter than kMinSliceTiles k tiles (a slice pays a
    // tile's fixed costs once more, and its accumulators travel through memory)
    const int nk_all = (g.K + BK - 1) / BK * (MODE == BWD_DX ? 2 : 1);
    p.n_slices = max(1, min(min(kMaxSlices, g.cus / left), nk_all / kMinSliceTiles));
    return p;
  }
  // fp32 accumulators of (left-over tile j, slice s), as the wavefronts hold them: [wave][fragment][lane] x 4
  static __device__ __forceinline__ f32x4* partial_slot(const MArgs& g, const SplitPlan& p, int j, int slice) {
    return g.partial + (size_t)(j * p.n_slices + slice) * (NW * TM * TN * kWave);
  }

  // Second kernel of a K-cut product: TM workgroups per left-over tile (one per fragment row of the
  // wavefronts: a single workgroup per tile left most of the chip idle and took 53 us for 72 MB) add the
  // slices' accumulators in slice order and store the tile (same ownership of the elements as in run():
  // fragment (i, j) of a wavefront, lane l = row l % 16, four columns from 4 (l / 16)).
  static __device__ void finish(const MArgs& g) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave / WN, wn = wave % WN;
    const Experts experts(g, lane);
    const SplitPlan plan = split_plan(g, experts.n_rt);
    const int j = blockIdx.x / TM, i = blockIdx.x % TM;
    if (plan.n_slices <= 1 || j >= plan.n_left) return;
    Tile tile;
    if (!locate(g, experts, plan.id_full + j, tile)) return;
    const int col0 = tile.tile_n * BNH;
    auto put = [&](void* C, size_t idx, const f32x4& v) {
      *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(C) + idx) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    };
    const int m0 = tile.row0 + wm * (TM * 16) + i * 16, m = m0 + (lane & 15);
    if (m0 >= tile.row_end) return;                      // 16 rows that do not exist: the slices left nothing there
    // Latency: all fragments of up to four slices are requested together, and they were stored through the caches, which still hold
    // most of them.  With streamed sums, a load waited for after another, us: 301 tokens, 4 experts of 4096 x 11008, UP (88 tiles of 2
    // slices) 10.0, DOWN (64 of 4) 14.5, now 9.0 and 10.4; 4001 tokens, 8 of 2048 x 5504, DOWN 12.4, BWD_DX 19.0, now 6.4 and 8.0;
    // 1501, 64 of 4096 x 688, UP 21.1, now 14.9; batches of four alone, streamed, 12.8 and 12.5, 9.5 and 9.7, 23.
    f32x4 sum[TN] = {};
    int sl = 0;
    auto add = [&](auto batch) {
      constexpr int B = decltype(batch)::value;
      for (; sl + B <= plan.n_slices; sl += B) {
        f32x4 v[B][TN];
#pragma unroll
        for (int b = 0; b < B; ++b) {
          const f32x4* from = partial_slot(g, plan, j, sl + b) + (size_t)wave * (TM * TN * kWave) + i * TN * kWave + lane;
#pragma unroll
          for (int jj = 0; jj < TN; ++jj) v[b][jj] = from[jj * kWave];
        }
        __builtin_amdgcn_sched_barrier(0);               // no sum in front of a load
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
          for (int jj = 0; jj < TN; ++jj)
#pragma unroll
            for (int x = 0; x < 4; ++x) sum[jj][x] = sl + b == 0 ? v[b][jj][x] : sum[jj][x] + v[b][jj][x];
      }
    };
    add(std::integral_constant<int, 4>{});
    add(std::integral_constant<int, 2>{});
    add(std::integral_constant<int, 1>{});
#pragma unroll
    for (int jj = 0; jj < TNH; ++jj) {
      const int n = col0 + wn * (TNH * 16) + jj * 16 + 4 * (lane >> 4);
      const bool inside = m < tile.row_end && n < g.N;
      const size_t idx = (size_t)m * g.ldc + n, idx_act = (size_t)m * g.ldp + n;
      if constexpr (MODE == UP) {                        // fragment jj holds x W1, fragment jj + TNH x W3 of the same outputs
        const f32x4 h1 = sum[jj], h3 = sum[jj + TNH];
        f32x4 a;
#pragma unroll
        for (int x = 0; x < 4; ++x) a[x] = silu_f(h1[x]) * h3[x];
        if (inside) {
          if (g.C0) { put(g.C0, idx, h1); put(g.C1, idx, h3); }
          put(g.C2, idx_act, a);
        }
      } else {
        if (inside) put(g.C0, idx, sum[jj]);
      }
    }
  }

  static __device__ void run(const MArgs& g, char* smem) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave / WN, wn = wave % WN;

    int id = blockIdx.x, slice = 0;
    SplitPlan plan{0, 0, 1};
    Tile tile;
    bool sliced;
    if constexpr (SMALL) {
      if (!locate_small(g, lane, tile, slice)) return;
      plan.n_slices = g.slices;
      sliced = MODE != BWD_ACT && plan.n_slices > 1;
    } else {
      const Experts experts(g, lane);
      plan = split_plan(g, experts.n_rt);
      if (SPLIT && id >= g.total_ids) {                  // a workgroup for slice 1.. of a left-over tile
        if (plan.n_slices <= 1) return;
        const int w = id - g.total_ids;
        slice = 1 + w / plan.n_left;
        if (slice >= plan.n_slices) return;
        id = plan.id_full + w % plan.n_left;
      }
      sliced = SPLIT && plan.n_slices > 1 && id >= plan.id_full;
      if (!locate(g, experts, id, tile)) return;
    }
    const int e = tile.e, row0 = tile.row0, row_end = tile.row_end, k_begin = tile.k_begin, k_end = tile.k_end;
    const int kp_begin = tile.kp_begin, tile_n = tile.tile_n;
    const int col0 = tile_n * BNH;
    // an expert with more rows than expected reads its weights through the caches, where its row tiles share them: small tiles (320
    // tokens, top-1, 4 experts of 4096 x 11008, the favoured one with more than 128 rows: forward pass 322 us with every weight
    // streamed, 306 with none, 293 like this) and the backward products (backward pass with every weight streamed / like this, top-1
    // with a favoured expert: 480 tokens 655 / 626, 600 tokens 681 / 662, 1200 tokens, 8 experts of 2048 x 5504 403 / 389; even loads the
    // same).  The forward products of larger tiles do not look: it costs their loop 1 % (even loads, 600 tokens 260 / 263, 420
    // tokens, top-2, 294 / 298) and gives as much at times (favoured experts 221 / 218, but 333 / 336).
    const bool read_once = (!SMALL && (MODE == UP || MODE == DOWN)) || row_end - tile.exp_row0 <= BM;

    const bf16_t* Bp0 = g.B0;
    const bf16_t* Bp1 = g.B1;
    if (!GROUP_K) { Bp0 += e * g.strideB_e; if (Bp1) Bp1 += e * g.strideB_e; }

    // ---- per-lane byte offsets of the direct copies, relative to a per-tile uniform base --
    // KC operand:      base = P + row0*ld + k0,  offset = (clamp(row) - row0)*ld + k_in_tile
    // strided operand: base = P + k0*ld,         offset = k_in_tile*ld + clamp(col)
    Off a_off[A_LOADS], b_off[B_LOADS];
    int b_k[B_LOADS], b_c[B_LOADS];                               // strided layout: k row / column
    int a_k[A_LOADS], b_kc[B_LOADS];                              // KC layouts: the chunk's first k inside the tile
#pragma unroll
    for (int q = 0; q < A_LOADS; ++q) {
      int major, minor;
      copy_coords<A_KC, BM>(wave * A_LOADS + q, lane, major, minor);
      const int gr = min(row0 + major, row_end - 1);
      // gathered rows: the offset is taken from the first row of A0 (it fits 32 bits, checked on the host)
      a_off[q] = copy_off<A_LOADS>(g.a_perm ? (Off)(g.a_perm[gr] / g.a_k) * ((Off)g.lda * 2u) + (Off)minor * 2u
                                            : ((Off)(gr - row0) * (Off)g.lda + (Off)minor) * 2u, q);
      a_k[q] = minor;
    }
#pragma unroll
    for (int q = 0; q < B_LOADS; ++q) {
      int major, minor;
      // DUAL: the B tile is two panels [BK][BNH] back to back, and half of the wavefronts copy either
      constexpr int SEGS_PER_PANEL = B_BYTES / 1024 / (DUAL ? 2 : 1);
      static_assert(SEGS_PER_PANEL % B_LOADS == 0, "a wavefront's copies have one base");
      const int seg = wave * B_LOADS + q;
      copy_coords<B_KC, BNH>(seg % SEGS_PER_PANEL, lane, major, minor);
      if (B_KC) {
        // tile rows are output columns (DUAL: BNH of the first panel, then BNH of the second)
        b_off[q] = copy_off<B_LOADS>(((Off)(min(col0 + major, g.N - 1) - col0) * (Off)g.ldb + (Off)minor) * 2u, q);
        b_k[q] = b_c[q] = 0;
        b_kc[q] = minor;
      } else {
        b_kc[q] = 0;
        b_k[q] = major;
        b_c[q] = min(col0 + minor, g.N - 8);
        b_off[q] = copy_off<B_LOADS>(((Off)(ROWS ? 0 : major) * (Off)g.ldb + (Off)b_c[q]) * 2u, q);
      }
    }

    const int k_len = k_end - k_begin;
    const int nk1 = (k_len + BK - 1) / BK;
    const int nk_all = MODE == BWD_DX ? 2 * nk1 : nk1;
    // a slice runs k tiles kb .. kb + nk - 1 of the tile's nk_all; below, kt counts from the slice's first one
    const int kb = sliced ? slice * nk_all / plan.n_slices : 0;
    const int nk = sliced ? (slice + 1) * nk_all / plan.n_slices - kb : nk_all;
    // K is a multiple of 8 (of 64 in the dW products, whose rows are padded): when it is not
    // a multiple of 64 only the first k_tail k of a pass's last k tile exist.  The copies of the
    // 16-byte chunks (rows, where K is strided) past them are re-pointed at the tile's first chunk
    // (last row that exists; any finite data will do) and the A fragments that lie past k_tail are
    // zeroed in registers: a lane's fragment is one such chunk, so it exists whole or not at all.
    // TAIL is a template parameter: 0 the common shapes, which pay nothing for it; 1 K = 32 mod 64, where only the
    // second half of the tile has to be looked at (with 2 in its place the step with 32 split experts, where DOWN and
    // BWD_DX run 21.5 k tiles, lost 0.7 %); 2 any other multiple of 8.  The shapes of 2 ran on plain fp32 FMA kernels
    // before: fwd + bwd of 1501 tokens, 64 experts of 4096 x 688, top-8: 13.9 -> 1.44 ms.
    static_assert(!(TAIL && GROUP_K), "the dW products have no K tail");
    // in the slice's own count of k tiles: where the second K pass begins, and the two possible tail tiles
    const int pass2_at = nk1 - kb, tail1_at = nk1 - 1 - kb, tail2_at = nk_all - 1 - kb;
    const int k_first1 = k_begin + kb * BK, k_first2 = k_begin - pass2_at * BK;
    const int kp_first = kp_begin + kb * BK;
    const int k_tail = TAIL == 1 ? BK / 2 : k_len - (nk1 - 1) * BK;
    auto is_tail = [&](int kt) { return TAIL && (kt == tail1_at || kt == tail2_at); };
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;   // LDS byte address of the dynamic segment

    // Copies of the A / B part of tile kt into LDS stage kt % NSA / kt % NSB.
    auto tile_k0 = [&](int kt, bool kc, bool& pass2) {
      pass2 = MODE == BWD_DX && kt >= pass2_at;
      return (GROUP_K && kc ? kp_first : (pass2 ? k_first2 : k_first1)) + kt * BK;
    };
    // where this wavefront's copies of tile kt come from and go to
    auto sourceA = [&](int kt) {
      bool pass2;
      const int k0 = tile_k0(kt, A_KC, pass2);
      return uniform64((pass2 ? g.A1 : g.A0) + (g.a_perm ? (size_t)0 : (size_t)row0 * g.lda) + k0) - copy_bias(A_LOADS);
    };
    const bool b_second = DUAL && wave >= NW / 2;        // DUAL: whose columns this wavefront copies
    auto sourceB = [&](int kt) {
      bool pass2;
      const int k0 = tile_k0(kt, B_KC, pass2);
      return uniform64(((MODE == BWD_DX ? pass2 : b_second) ? Bp1 : Bp0) + (B_KC ? (size_t)col0 * g.ldb + k0 : (size_t)k0 * g.ldb)) - copy_bias(B_LOADS);
    };
    const uint32_t ldsA = smem_base + wave * (A_LOADS * 1024), ldsB = smem_base + B_BASE + wave * (B_LOADS * 1024);
    auto put_a = [&](uint64_t from, const Off* off, uint32_t to) { copies_to_lds<A_LOADS, false>(from, off, to); };
    auto put_b = [&](uint64_t from, const Off* off, uint32_t to) {
      if (STREAM_B && read_once) copies_to_lds<B_LOADS, STREAM_B>(from, off, to);
      else copies_to_lds<B_LOADS, false>(from, off, to);
    };
    auto issueA = [&](int kt) {
      Off off[A_LOADS];
#pragma unroll
      for (int q = 0; q < A_LOADS; ++q) {
        off[q] = a_off[q];
        if (is_tail(kt) && a_k[q] >= k_tail) off[q] -= (Off)(a_k[q] * 2);
      }
      put_a(sourceA(kt), off, ldsA + (kt % NSA) * A_BYTES);
    };
    // ROWS: the 8 token rows of k tile kt that this wavefront copies, by the byte offsets that BWD_ACT left, through the scalar cache
    // (vector loads would be waited for together with the copies behind them); rows past the expert's last repeat it
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8), aligned(4)));
    typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;
    typedef const __attribute__((address_space(4))) u32x8* scalar_ptr8;
    uint32_t tok[8];
    Off row_off[ROWS ? B_LOADS : 1];                     // of the k tile whose rows are copied next
    auto look_up = [&](int kt) {
      const int k = kt * BK + wave * 8;
      const scalar_ptr table = (scalar_ptr)(uintptr_t)g.row_bytes + k_begin;
      if (k + 8 <= k_len) {
        const u32x8 t = *(scalar_ptr8)(table + k);
#pragma unroll
        for (int x = 0; x < 8; ++x) tok[x] = t[x];
      } else {
#pragma unroll
        for (int x = 0; x < 8; ++x) tok[x] = table[min(k + x, k_len - 1)];
      }
    };
    auto next_rows = [&]() {
#pragma unroll
      for (int q = 0; q < B_LOADS; ++q) row_off[q] = b_off[q] + (lane < 32 ? tok[2 * q] : tok[2 * q + 1]);
    };
    auto issueB = [&](int kt) {
      if constexpr (ROWS) {
        put_b(uniform64(g.B0) - copy_bias(B_LOADS), row_off, ldsB + (kt % NSB) * B_BYTES);
        return;
      }
      bool pass2;
      const int k0 = tile_k0(kt, B_KC, pass2);
      Off off[B_LOADS];
#pragma unroll
      for (int q = 0; q < B_LOADS; ++q) {
        off[q] = b_off[q];
        // grouped-K, strided operand: a k row past the expert's last grouped row is re-pointed at that last
        // row.  It meets the zero fill of the transposed operand, so it must hold finite numbers: the
        // expert's own rows were written by BWD_ACT in this call, whereas the rows behind them belong to
        // the next expert or, past the last kept row when a capacity limit dropped pairs, to nobody
        // (workspace bytes nothing has written, possibly NaN patterns).
        if (GROUP_K && !B_KC) off[q] = copy_off<B_LOADS>(((Off)(min(k0 + b_k[q], k_end - 1) - k0) * (Off)g.ldb + (Off)b_c[q]) * 2u, q);
        if (is_tail(kt)) {
          if (B_KC) { if (b_kc[q] >= k_tail) off[q] -= (Off)(b_kc[q] * 2); }
          else off[q] = copy_off<B_LOADS>(((Off)min(b_k[q], k_tail - 1) * (Off)g.ldb + (Off)b_c[q]) * 2u, q);
        }
      }
      put_b(sourceB(kt), off, ldsB + (kt % NSB) * B_BYTES);
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

    auto load_frags = [&](int kt, int ks, bf16x8 (&af)[TM], bf16x8 (&bfr)[TN]) {
      const char* At = smem + (kt % NSA) * A_BYTES;
      const char* Bt = smem + B_BASE + (kt % NSB) * B_BYTES;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = wm * (TM * 16) + i * 16;
        af[i] = read_kc(At, r, ks, lane);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int c = wn * (TNH * 16) + (j % TNH) * 16;
        bfr[j] = B_KC ? read_kc(Bt, (j / TNH) * BNH + c, ks, lane)
                      : read_tr<BNH>(Bt + (j / TNH) * (BK * BNH * 2), c, ks, lane);
      }
    };
    auto mfma_step = [&](bf16x8 (&af)[TM], bf16x8 (&bfr)[TN]) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
    };
    // the A fragments that lie past K in a pass's last k tile
    auto zero_past = [&](bf16x8 (&af)[TM], int ks) {
      const bool past = TAIL == 1 ? ks == 1 : 32 * ks + 8 * (lane >> 4) >= k_tail;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        u32x4 w = __builtin_bit_cast(u32x4, af[i]);
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = past ? 0u : w[v];
        af[i] = __builtin_bit_cast(bf16x8, w);
      }
    };

    // ROWS: token rows that repeat the expert's last one meet zeros, which an infinity there would not survive
    auto zero_rows_past = [&](bf16x8 (&bfr)[TN], int kt, int ks) {
      const int left = k_len - kt * BK - 32 * ks - 8 * (lane >> 4);
      u32x4 mask;
#pragma unroll
      for (int x = 0; x < 4; ++x) mask[x] = (2 * x < left ? 0xffffu : 0u) | (2 * x + 1 < left ? 0xffff0000u : 0u);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[j] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, bfr[j]) & mask);
    };

    if constexpr (SMALL) {
      // One pipeline for all wavefronts: A tiles are requested NSA - 1 k tiles ahead, B tiles NSB - 1, one barrier
      // per k tile.  A's copies are issued before B's, so that of what may be outstanding when tile kt is needed
      // only the copies behind A's of that tile remain.
      constexpr int kAhead = (NSB > NSA ? B_LOADS : 0) + (NSA - 2) * (A_LOADS + B_LOADS);
#pragma unroll
      for (int j = 1 - NSB; j < 0; ++j) {
        if (j + NSA - 1 >= 0 && j + NSA - 1 < nk) issueA(j + NSA - 1);
        if (j + NSB - 1 < nk) issueB(j + NSB - 1);
      }
#pragma unroll 1
      for (int kt = 0; kt < nk; ++kt) {
        if (kt + NSB - 2 < nk) wait_vmcnt<kAhead>(); else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();                    // tile kt published; everybody is done with tile kt - 1
        __builtin_amdgcn_sched_barrier(0);
        if (kt + NSA - 1 < nk) issueA(kt + NSA - 1);
        if (kt + NSB - 1 < nk) issueB(kt + NSB - 1);
        bf16x8 fa[KSTEPS][TM], fb[KSTEPS][TN];
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) load_frags(kt, ks, fa[ks], fb[ks]);
        if (is_tail(kt)) {
#pragma unroll
          for (int ks = 0; ks < KSTEPS; ++ks) zero_past(fa[ks], ks);
        }
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) mfma_step(fa[ks], fb[ks]);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_barrier();                      // the epilogue reuses the operand stages
      __builtin_amdgcn_sched_barrier(0);
    } else {
      // Ping-pong schedule.  The two wavefronts that share a SIMD (w and w+4) alternate
      // between a memory phase (LDS fragment reads of half a tile + a quarter of the copies
      // of a later tile) and a compute phase (an uninterrupted run of 32 MFMAs), half a period
      // apart and kept in step by a barrier at every phase boundary.  The matrix pipe always
      // has one wavefront feeding it and is never held up behind a wavefront that is stuck
      // issuing copies or waiting for LDS.  Time is counted in phases; tile kt occupies phases
      // 4kt .. 4kt+3 for group 0 and one phase later for group 1:
      //   phase 4kt   : G0 reads half 0 of tile kt, issues its B copies of tile kt+1   | G1 computes
      //   phase 4kt+1 : G0 computes | G1 reads half 0 of tile kt, issues its B copies of tile kt+1
      //   phase 4kt+2 : G0 reads half 1, issues its A copies of tile kt+2             | G1 computes
      //   phase 4kt+3 : G0 computes | G1 reads half 1, issues its A copies of tile kt+2
      // so the address unit sees the same 16 copies in every phase.  B has two LDS stages (its
      // copies have at least 2.5 phases to land), A has three (at least 4 phases).  Every
      // wavefront waits for its copies of tile kt+1 right before the barrier that ends phase
      // 4kt+3; its youngest copies (A of tile kt+2) may stay in flight.
      // NSB == 3: the roles of A and B in the copies are exchanged, for products that wait for the weights to arrive
      // from HBM (UP of 301 tokens, 4 experts of 4096 x 11008, top-2, 192-row tiles: 177 us with three stages of A,
      // 170 with three of B; large products lose up to 10 % with it).
      constexpr int HS = KSTEPS / 2;                 // k steps per half tile
      const int grp = wave / (NW / 2);               // group 1 lags group 0 by one phase
      bf16x8 fa[HS][TM], fb[HS][TN];
      constexpr bool DEEP_B = NSB == 3;
      constexpr int DEEP_LOADS = DEEP_B ? B_LOADS : A_LOADS;
      auto issue_near = [&](int kt) { if constexpr (DEEP_B) issueA(kt); else issueB(kt); };
      auto issue_deep = [&](int kt) { if constexpr (DEEP_B) issueB(kt); else issueA(kt); };
      if (nk > 0) {
        if constexpr (ROWS) {
          look_up(0);
          next_rows();
        }
        issue_deep(0);
        issue_near(0);
        if (nk > 1) issue_deep(1);
        if constexpr (ROWS) {
          look_up(1);
          next_rows();
          look_up(2);
        }
        if (nk > 1) wait_vmcnt<DEEP_LOADS>(); else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();                // tile 0 published
      }
      if (grp == 1 && nk > 0) __builtin_amdgcn_s_barrier();   // idle during group 0's first memory phase
      // One k tile.  fast: not one of the last of a pass, whose copies and fragments need a look: sources, stages and the lanes' LDS
      // addresses move on by additions, made while the second half's fragments are on their way.  In front of its copies and
      // reads a memory phase then issues one setting of m0.  With everything worked out from kt, 90 scalar and vector instructions and
      // 10 branches per k tile, the phase was as long as the products of the other group (fwd + bwd of 16384 tokens, 4 experts
      // of 4096 x 11008, top-2: 19.73 ms / 19.01 like this; 32 of 4096 x 1376, top-8: 12.74 / 12.23; one sequence forward 1.79 / 1.72); with
      // the additions made during the products 19.31, which wait for them.
      constexpr int NRB = B_KC ? KSTEPS : TNH;       // B_KC: an address for each k step, else one for each column of fragments
      struct Moving { uint64_t a, b; uint32_t to_a, to_b, at_a, at_b, ra[KSTEPS], rb[NRB]; } mv{};
      auto read_fast = [&](int ks, bf16x8 (&af)[TM], bf16x8 (&bfr)[TN]) {
        typedef const __attribute__((address_space(3))) bf16x8* ptr8;
        typedef __attribute__((address_space(3))) bf16x4* ptr4;
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = *(ptr8)(uintptr_t)(mv.ra[ks] + i * (16 * BK * 2));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (B_KC) {
            bfr[j] = *(ptr8)(uintptr_t)(mv.rb[ks] + ((j / TNH) * BNH + (j % TNH) * 16) * (BK * 2));
          } else {
            const uint32_t at = mv.rb[j % TNH] + (j / TNH) * (BK * BNH * 2) + ks * (32 * BNH * 2);
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((ptr4)(uintptr_t)at);
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((ptr4)(uintptr_t)(at + 4 * BNH * 2));
            bfr[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          }
        }
      };
      const uint64_t step_b = B_KC ? (uint64_t)(BK * 2) : (uint64_t)g.ldb * (BK * 2);
      auto start_moving = [&](int kt) {
        const int ta = kt + (DEEP_B ? 1 : 2), tb = kt + (DEEP_B ? 2 : 1);
        mv.a = sourceA(ta); mv.b = sourceB(tb);
        mv.to_a = ldsA + (ta % NSA) * A_BYTES; mv.to_b = ldsB + (tb % NSB) * B_BYTES;
        mv.at_a = (kt % NSA) * A_BYTES; mv.at_b = (kt % NSB) * B_BYTES;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) mv.ra[ks] = smem_base + mv.at_a + kc_at(wm * (TM * 16), ks, lane);
#pragma unroll
        for (int x = 0; x < NRB; ++x)
          mv.rb[x] = smem_base + B_BASE + mv.at_b + (B_KC ? kc_at(wn * (TNH * 16), x, lane) : tr_at<BNH>(wn * (TNH * 16) + x * 16, 0, lane));
      };
      auto move_on = [&]() {
        auto next = [](uint32_t x, uint32_t first, uint32_t bytes, int n) { return x == first + (n - 1) * bytes ? first : x + bytes; };
        mv.a += BK * 2;
        mv.b += step_b;
        mv.to_a = next(mv.to_a, ldsA, A_BYTES, NSA);
        mv.to_b = next(mv.to_b, ldsB, B_BYTES, NSB);
        const uint32_t a = next(mv.at_a, 0, A_BYTES, NSA), b = next(mv.at_b, 0, B_BYTES, NSB);
#pragma unroll
        for (int x = 0; x < KSTEPS; ++x) {
          mv.ra[x] += a - mv.at_a;
          asm volatile("" : "+v"(mv.ra[x]));         // here, not where it is used
        }
#pragma unroll
        for (int x = 0; x < NRB; ++x) {
          mv.rb[x] += b - mv.at_b;
          asm volatile("" : "+v"(mv.rb[x]));
        }
        mv.at_a = a;
        mv.at_b = b;
      };
      auto k_tile = [&](auto fast_tag, int kt) {
        constexpr bool fast = decltype(fast_tag)::value;
        auto landed = [&]() {
          if (fast || kt + 2 < nk) wait_vmcnt<DEEP_LOADS>(); else wait_vmcnt<0>();
        };
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          // ---- memory phase: copies first, they take longer
          if constexpr (fast) {
            if ((h == 0) == DEEP_B) put_a(mv.a, a_off, mv.to_a);
            else if constexpr (ROWS) put_b(uniform64(g.B0) - copy_bias(B_LOADS), row_off, mv.to_b);
            else put_b(mv.b, b_off, mv.to_b);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < HS; ++x) read_fast(h * HS + x, fa[x], fb[x]);
            __builtin_amdgcn_sched_barrier(0);
            if (h == 1) move_on();                   // while the reads are on their way
          } else {
#pragma unroll
            for (int x = 0; x < HS; ++x) load_frags(kt, h * HS + x, fa[x], fb[x]);
            if (h == 0 && kt + 1 < nk) issue_near(kt + 1);
            if (h == 1 && kt + 2 < nk) issue_deep(kt + 2);
          }
          __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0): fragments are in registers
          if (!fast && (TAIL == 2 || h == 1) && is_tail(kt)) {   // the part of the last k tile that lies past K
#pragma unroll
            for (int x = 0; x < HS; ++x) zero_past(fa[x], h * HS + x);
          }
          if (ROWS && !fast && (kt + 1) * BK > k_len) {
#pragma unroll
            for (int x = 0; x < HS; ++x) zero_rows_past(fb[x], kt, h * HS + x);
          }
          if (h == 1 && grp == 1) landed();
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
          // ---- compute phase
          if constexpr (ROWS) {                          // looked up half a k tile before, waited for with the fragments
            if (h == 0) next_rows();                     // of k tile kt + 2
            else look_up(kt + 3);
          }
#pragma unroll
          for (int x = 0; x < HS; ++x) mfma_step(fa[x], fb[x]);
          if (h == 1 && grp == 0) landed();
          __builtin_amdgcn_sched_barrier(0);
          if (fast || !(grp == 1 && h == 1 && kt + 1 == nk)) __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      for (int kt = 0; kt < nk;) {
        // the tiles in front of the last two of this pass (three, where the copies of its last one are special)
        const int pass_end = MODE == BWD_DX && kt < pass2_at && pass2_at < nk ? pass2_at : nk;
        if (const int stop = pass_end - (TAIL ? 3 : 2); kt < stop) {
          start_moving(kt);
          // one k tile per trip: unrolled by two (the compiler's choice for some instantiations) the loop ran 2 to
          // 4 % slower
#pragma unroll 1
          do k_tile(std::true_type{}, kt);
          while (++kt < stop);
        }
#pragma unroll 1
        for (; kt < pass_end; ++kt) k_tile(std::false_type{}, kt);
      }
    }

    if (SMALL && sliced) {                               // row-major sums, for slices_finish_kernel
      const size_t panel = (size_t)g.R * g.N;
      float* P = g.slice_sums + (size_t)slice * (DUAL ? 2 : 1) * panel;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int m = row0 + wm * (TM * 16) + i * 16 + (lane & 15);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int n = col0 + wn * (TNH * 16) + (j % TNH) * 16 + 4 * (lane >> 4);
          if (m < row_end && n < g.N) *reinterpret_cast<f32x4*>(P + (j / TNH) * panel + (size_t)m * g.N + n) = acc[i][j];
        }
      }
      return;
    }
    if (SPLIT && sliced) {                               // a slice leaves its accumulators for split_finish
      f32x4* slot = partial_slot(g, plan, id - plan.id_full, slice) + (size_t)wave * (TM * TN * kWave);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (row0 + wm * (TM * 16) + i * 16 >= row_end) break;          // finish() does not look at these rows
#pragma unroll
        for (int j = 0; j < TN; ++j) slot[(i * TN + j) * kWave + lane] = acc[i][j];   // plain: they are read back at once
      }
      return;
    }

    // ---- epilogue ----------------------------------------------------------
    // acc[i][j][v]: row m = row0 + wm*TM*16 + i*16 + lane%16,
    //               col n = col0 + wn*TNH*16 + (j%TNH)*16 + 4*(lane/16) + v
    // In that layout one store instruction would touch 16 rows with 8 to 16 bytes each.  Instead
    // every wavefront turns its results around in a private piece of LDS, one band of 32 rows
    // (two fragment rows) at a time: the lanes write their 4-column pieces, read the band back
    // as 16-byte chunks that follow each other along a row, and store whole row segments (64 to
    // 256 contiguous bytes per row).  BWD_ACT fetches the saved h1/h3 band the same way round.
    // The operand stages are dead by now: in the ping-pong schedule the barrier that ends group
    // 0's last compute phase comes after group 1's last fragment read and after every copy has
    // landed.
    const int lane_m = lane & 15, lane_c = lane >> 4;
    const int wcol0 = col0 + wn * (TNH * 16);         // first output column of this wavefront (per panel)
    constexpr int NB = TM / 2;                         // 32-row bands per wavefront
    // byte offset, inside a band, of this lane's 4-column piece of fragment (i2, j); ES = element size
    auto piece = [&](auto rowb_tag, auto es_tag, int i2, int j) {
      constexpr int ROWB = decltype(rowb_tag)::value, ES = decltype(es_tag)::value;
      const int byte = (j * 16 + 4 * lane_c) * ES;
      const uint32_t flip = MODE == BWD_ACT ? 0u : half_flip<ROWB, ES>(i2 * 16 + lane_m);
      return stage_off<ROWB, 4 * ES>(i2 * 16 + lane_m, byte >> 4) + ((byte & 15) ^ flip);
    };
    float dg_acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) dg_acc[i] = 0.f;

    if constexpr (MODE == BWD_ACT) {
      constexpr int ROWB = TNH * 32;                  // bytes per band row
      constexpr int CPR = ROWB / 16, RPI = 64 / CPR, NI = 32 / RPI;
      static_assert(5 * 32 * ROWB * NW <= LDS_BYTES, "epilogue bands must fit the operand stages");
      char* bufA = smem + wave * (5 * 32 * ROWB);
      char* bufB = bufA + 32 * ROWB;
      char* bufC = bufB + 32 * ROWB;
      char* bufT = bufC + 32 * ROWB;                  // two bands of g * act, transposed: [column][64 rows]
      const int cr = lane / CPR, cc = lane % CPR;     // row (per pass) and chunk of the row-contiguous view
      const int cn = wcol0 + cc * 8;
      u32x4 p1[NI], p3[NI];
      float gate_next[2];
      // band ib of h1/h3 in the row-contiguous view (clamped, always valid addresses)
      auto fetch = [&](int ib) {
        const int mb = row0 + wm * (TM * 16) + ib * 32;
#pragma unroll
        for (int t = 0; t < NI; ++t) {
          const size_t idx = (size_t)min(mb + t * RPI + cr, row_end - 1) * g.ldc + min(cn, g.N - 8);
          // read once by this tile and by nobody else: streamed past the L2 (another 2 % of the kernel)
          p1[t] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(g.H1 + idx));
          p3[t] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(g.H3 + idx));
        }
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2) gate_next[i2] = g.gates[g.perm[min(mb + i2 * 16 + lane_m, row_end - 1)]];
      };
      fetch(0);
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) {
        const int mb = row0 + wm * (TM * 16) + ib * 32;
#pragma unroll
        for (int t = 0; t < NI; ++t) {
          const uint32_t o = stage_off<ROWB, 8>(t * RPI + cr, cc);
          *reinterpret_cast<u32x4*>(bufA + o) = p1[t];
          *reinterpret_cast<u32x4*>(bufB + o) = p3[t];
        }
        const float gate2[2] = {gate_next[0], gate_next[1]};
        if (ib + 1 < NB) fetch(ib + 1);               // in flight during the arithmetic below
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2) {
          const int i = 2 * ib + i2;
          const bool m_ok = mb + i2 * 16 + lane_m < row_end;
          const float gate = m_ok ? gate2[i2] : 0.f;    // rows past the group's end come out as zeros
#pragma unroll
          for (int j = 0; j < TNH; ++j) {
            const uint32_t o = piece(std::integral_constant<int, ROWB>{}, std::integral_constant<int, 2>{}, i2, j);
            const u32x2 a1 = *reinterpret_cast<const u32x2*>(bufA + o);
            const u32x2 a3 = *reinterpret_cast<const u32x2*>(bufB + o);
            const float z[4] = {bf16lo(a1[0]), bf16hi(a1[0]), bf16lo(a1[1]), bf16hi(a1[1])};
            const float v3[4] = {bf16lo(a3[0]), bf16hi(a3[0]), bf16lo(a3[1]), bf16hi(a3[1])};
            float o1[4], o3[4], oa[4], dot = 0.f;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const float dd = acc[i][j][x];
              const float sg = sigmoid_f(z[x]), sl = z[x] * sg;
              const float a = sl * v3[x];
              dot = fmaf(dd, a, dot);
              const float da = gate * dd;
              o1[x] = da * v3[x] * fmaf(sl, 1.f - sg, sg);     // silu'(z) = sg + silu(z) (1 - sg)
              o3[x] = da * sl;
              oa[x] = gate * a;
            }
            if (m_ok && wcol0 + j * 16 + 4 * lane_c < g.N) dg_acc[i] += dot;
            // each lane overwrites exactly the pieces it has just read
            *reinterpret_cast<u32x2*>(bufA + o) = u32x2{pack_bf16x2(o1[0], o1[1]), pack_bf16x2(o1[2], o1[3])};
            *reinterpret_cast<u32x2*>(bufB + o) = u32x2{pack_bf16x2(o3[0], o3[1]), pack_bf16x2(o3[2], o3[3])};
            if (g.T2 || g.C2) *reinterpret_cast<u32x2*>(bufC + o) = u32x2{pack_bf16x2(oa[0], oa[1]), pack_bf16x2(oa[2], oa[3])};
          }
        }
#pragma unroll
        for (int t = 0; t < NI; ++t) {
          const int r = t * RPI + cr;
          const uint32_t o = stage_off<ROWB, 8>(r, cc);
          const u32x4 v1 = *reinterpret_cast<const u32x4*>(bufA + o);
          const u32x4 v3 = *reinterpret_cast<const u32x4*>(bufB + o);
          if (mb + r < row_end && cn < g.N) {
            const size_t idx = (size_t)(mb + r) * g.ldp + cn;
            store_out<STREAM>(reinterpret_cast<u32x4*>(static_cast<bf16_t*>(g.C0) + idx), v1);
            store_out<STREAM>(reinterpret_cast<u32x4*>(static_cast<bf16_t*>(g.C1) + idx), v3);
            if (g.C2) store_out<STREAM>(reinterpret_cast<u32x4*>(static_cast<bf16_t*>(g.C2) + idx), *reinterpret_cast<const u32x4*>(bufC + o));
          }
        }
        if (g.T2) {
          // The same band once more, transposed, for the dW products: [column][padded grouped row].
          // A pair of transposing reads turns 16 columns x 8 rows per 16-lane group around: lane
          // 4a+b of a group receives element b of what lanes a, a+4, a+8, a+12 fetched, so lane r
          // fetches band row 8*group + r/4 (then +4) at columns 4*(r%4).. and ends up with rows
          // 8*group .. +7 of column r: 16 contiguous bytes of the transposed matrix.  Those are
          // collected over two bands as [column][64 rows] (128 bytes per column, chunks swizzled by
          // column) and read back so that eight consecutive lanes hold one column's 128 bytes: whole,
          // aligned cache lines per store (with 64-byte pieces, one band at a time, these stores moved
          // 3.1 TB/s where the row stores of dh1/dh3 move 5.1; scattered 16-byte stores cost the address
          // unit four times as much again).  Rows past the group's end are zeros (see the gate above) and
          // are written up to the 64-row padding.
          typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
          static_assert(NB % 2 == 0, "bands are turned around in pairs");
          const int o_e = tile.exp_row0;
          const int pad_e = (row_end - o_e + 63) & ~63;
          const int fr = 8 * lane_c + (lane_m >> 2), fa4 = lane_m & 3;
          bf16x8 v[TNH];
#pragma unroll
          for (int pr = 0; pr < TNH; ++pr) {
            const uint32_t o_lo = stage_off<ROWB, 8>(fr, 2 * pr + (fa4 >> 1)) + 8 * (fa4 & 1);
            const uint32_t o_hi = stage_off<ROWB, 8>(fr + 4, 2 * pr + (fa4 >> 1)) + 8 * (fa4 & 1);
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(bufC + o_lo));
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(bufC + o_hi));
            v[pr] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          }
#pragma unroll
          for (int pr = 0; pr < TNH; ++pr) {
            const int tc = 16 * pr + lane_m;             // column; chunk = 8 rows: 4 per band
            *reinterpret_cast<bf16x8*>(bufT + tc * 128 + ((((ib & 1) * 4 + lane_c) ^ ((tc >> 1) & 7)) << 4)) = v[pr];
          }
          if (ib & 1) {
            const int qc = lane >> 3, qg = lane & 7;     // read-back view: column within 8, 8-row chunk of the pair
            const int m8 = mb - 32 + 8 * qg - o_e;       // grouped row of that chunk, relative to the expert
#pragma unroll
            for (int pr = 0; pr < 2 * TNH; ++pr) {
              const int tc = 8 * pr + qc;
              const bf16x8 w = *reinterpret_cast<const bf16x8*>(bufT + tc * 128 + ((qg ^ ((tc >> 1) & 7)) << 4));
              const int col = wcol0 + tc;
              if (col < g.N && m8 < pad_e)
                store_out<STREAM>(reinterpret_cast<bf16x8*>(g.T2 + (size_t)col * g.ldt + kp_begin + m8), w);
            }
          }
        }
      }
    } else {
      constexpr int NP = MODE == UP ? 3 : (DUAL ? 2 : 1);            // matrices written
      // ET: element type of the output (bf16 bits or float)
      auto staged = [&](auto tag) {
        using ET = decltype(tag);
        constexpr int ES = sizeof(ET);
        constexpr int ROWB = TNH * 16 * ES;
        constexpr int CPR = ROWB / 16, RPI = 64 / CPR, NI = 32 / RPI;
        static_assert(ROWB == 64 || ROWB == 128 || ROWB == 256 || ROWB == 512, "band row");
        static_assert(NP * 32 * ROWB * NW <= LDS_BYTES, "epilogue bands must fit the operand stages");
        char* wb = smem + wave * (NP * 32 * ROWB);
        const int cr = lane / CPR, cc = lane % CPR;
        const int cn = wcol0 + cc * (16 / ES);
        const bool want_h = MODE != UP || g.C0 != nullptr;
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) {
          const int mb = row0 + wm * (TM * 16) + ib * 32;
#pragma unroll
          for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
            for (int j = 0; j < TNH; ++j) {
              const int i = 2 * ib + i2;
              const uint32_t o = piece(std::integral_constant<int, ROWB>{}, std::integral_constant<int, ES>{}, i2, j);
              float v[NP][4];
#pragma unroll
              for (int x = 0; x < 4; ++x) {
                if constexpr (MODE == UP) {
                  v[0][x] = acc[i][j][x];
                  v[1][x] = acc[i][j + TNH][x];
                  v[2][x] = silu_f(v[0][x]) * v[1][x];
                } else {
#pragma unroll
                  for (int pp = 0; pp < NP; ++pp) v[pp][x] = acc[i][j + pp * TNH][x];
                }
              }
#pragma unroll
              for (int pp = 0; pp < NP; ++pp) {
                if (MODE == UP && pp < 2 && !want_h) continue;
                char* dst = wb + pp * (32 * ROWB) + o;
                if constexpr (ES == 2)
                  *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16x2(v[pp][0], v[pp][1]), pack_bf16x2(v[pp][2], v[pp][3])};
                else
                  *reinterpret_cast<f32x4*>(dst) = f32x4{v[pp][0], v[pp][1], v[pp][2], v[pp][3]};
              }
            }
#pragma unroll
          for (int pp = 0; pp < NP; ++pp) {
            if (MODE == UP && pp < 2 && !want_h) continue;
            ET* C = static_cast<ET*>(pp == 0 ? g.C0 : (pp == 1 ? g.C1 : g.C2)) + (GROUP_K ? (size_t)e * g.strideC_e : 0);
#pragma unroll
            for (int t = 0; t < NI; ++t) {
              const int r = t * RPI + cr;
              const u32x4 val = swap_halves(
                  *reinterpret_cast<const u32x4*>(wb + pp * (32 * ROWB) + stage_off<ROWB, 4 * ES>(r, cc)),
                  half_flip<ROWB, ES>(r) != 0);
              const int ld = MODE == UP && pp == 2 ? g.ldp : g.ldc;
              if (mb + r < row_end && cn < g.N) store_out<STREAM>(reinterpret_cast<u32x4*>(C + (size_t)(mb + r) * ld + cn), val);
            }
          }
        }
      };
      if constexpr (GROUP_K) {                       // only the weight gradients can be asked for in fp32
        if (g.c_is_f32) staged(float{});
        else staged(bf16_t{});
      } else {
        staged(bf16_t{});
      }
    }
    if (MODE == BWD_ACT) {
      // dg partial of this column tile: lanes l, l^16, l^32, l^48 hold the same row; then the WN
      // wavefronts of a row band are summed in fixed order through LDS.
      __syncthreads();  // all waves are done with the operand tiles
      float* red = reinterpret_cast<float*>(smem);   // [WN][BM]
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float s = dg_acc[i] + __shfl_xor(dg_acc[i], 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (lane_c == 0) red[wn * BM + wm * (TM * 16) + i * 16 + lane_m] = s;
      }
      __syncthreads();
      for (int r = threadIdx.x; r < BM; r += NT) {
        const int m = row0 + r;
        if (m < row_end) {
          float s = 0.f;
#pragma unroll
          for (int w = 0; w < WN; ++w) s += red[w * BM + r];
          g.dg_part[(size_t)m * g.n_part + tile_n] = s;
          if (g.row_bytes && tile_n == 0) g.row_bytes[m] = (uint32_t)(g.a_perm[m] / g.a_k) * (uint32_t)(g.lda * 2);
        }
      }
    }
  }
};

template <int BM, int BN, int BK, int WM, int WN, int NSA, int NSB, int MODE, int TAIL, bool STREAM_B, bool STREAM>
__global__ __launch_bounds__(WM* WN* kWave) void mfma_gemm_kernel(MArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  Gemm<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B, STREAM>::run(g, smem);
}
// dW2 from token rows of dY (mfma_dw2_rows())
template <int BM, int BN, int BK, int WM, int WN, int NSA, int NSB, int MODE, int TAIL, bool STREAM_B, bool STREAM>
__global__ __launch_bounds__(WM* WN* kWave) void mfma_gemm_kernel_rows(MArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  Gemm<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B, STREAM, true>::run(g, smem);
}

// small tiles: 4 wavefronts, two workgroups per compute unit
template <int BM, int WM, int WN, int NSA, int NSB, int MODE, int TAIL, bool STREAM_B>
__global__ __launch_bounds__(WM* WN* kWave, 2) void mfma_small_kernel(MArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  Gemm<BM, 128, 64, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B>::run(g, smem);
}

// The K slices of small tiles added in slice order, 8 columns of a row per thread; SWIGLU: [slice][2][R][N], the
// activation (and the two products themselves, unless C0 is NULL) is stored.
template <bool SWIGLU>
__global__ __launch_bounds__(256) void slices_finish_kernel(const float* __restrict__ sums, int slices, int R, int N, int ldp,
                                                            const int32_t* __restrict__ offsets, int E,
                                                            bf16_t* __restrict__ C0, bf16_t* __restrict__ C1,
                                                            bf16_t* __restrict__ C2) {
  const int chunks = N / 8;
  const unsigned i = blockIdx.x * 256 + threadIdx.x;     // R * N floats fit the scratch, so 32 bits do
  const int row = (int)(i / (unsigned)chunks), c = (int)(i - row * (unsigned)chunks) * 8;
  if (row >= offsets[E]) return;                         // at most R rows are kept
  const size_t panel = (size_t)R * N, at = (size_t)row * N + c;
  float h1[8] = {}, h3[8] = {};
  for (int s = 0; s < slices; ++s) {
    const float* P = sums + (size_t)s * (SWIGLU ? 2 : 1) * panel + at;
    float v[8];
    RowVec<float, 8>::ld(P, v);
#pragma unroll
    for (int x = 0; x < 8; ++x) h1[x] += v[x];
    if constexpr (SWIGLU) {
      RowVec<float, 8>::ld(P + panel, v);
#pragma unroll
      for (int x = 0; x < 8; ++x) h3[x] += v[x];
    }
  }
  if constexpr (SWIGLU) {
    if (C0) { RowVec<bf16_t, 8>::st(C0 + at, h1); RowVec<bf16_t, 8>::st(C1 + at, h3); }
#pragma unroll
    for (int x = 0; x < 8; ++x) h1[x] = silu_f(h1[x]) * h3[x];
    RowVec<bf16_t, 8>::st(C2 + (size_t)row * ldp + c, h1);
  } else {
    RowVec<bf16_t, 8>::st(C0 + at, h1);
  }
}

template <int BM, int BN, int BK, int WM, int WN, int NSA, int NSB, int MODE, int TAIL = 0>
__global__ __launch_bounds__(WM* WN* kWave) void mfma_split_finish_kernel(MArgs g) {
  Gemm<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL>::finish(g);
}

// Weight gradients of experts with few rows (dW1, dW3 = xs^T dh1, dh3; dW2 = ga^T dys): a contraction of a few k tiles
// whose result, the size of the weights, has to be written: up to about 64 rows the stores are the bound (64 experts of 4096 x
// 688, 37 rows: 721 MB of dW1 and dW3 in 160 us), above the copies from L2 to LDS (188 rows: 300 us, 209 without them, 270 with
// a quarter of the matrix instructions).  With one 256 x 256 tile per workgroup a tile costs its latencies one after
// another, and the token rows have to be laid out transposed first.  Here
//   * both operands are read as they lie in memory, rows of x, dh1, dh3, ga and dY; the token rows by the byte offsets that
//     BWD_ACT has left in row_bytes.  No transposed copies (188 rows: 95 us), and BWD_ACT writes ga as it writes dh1 and dh3;
//   * a wavefront takes 64 x 128 outputs.  The 64 columns of A are turned around by transposing reads; for the 128 columns
//     of B a lane reads 16 bytes (8 columns) of 8 k rows and pairs them up with v_perm, which puts column 8 r + j into lane r of
//     fragment j: the products of a row then lie in a lane 8 columns at a time, and the tile is stored from the registers
//     in whole segments of 256 bytes without a way through LDS.  fp32 gradients: two times 8 bytes, which makes it columns 4 r + j
//     and 64 + 4 r + j, so that 16 lanes store 256 bytes in a row as well.  With 8 columns to a lane every store left half of each
//     64 bytes out, which is what streamed stores pay for (backward pass with fp32 gradients, transposed tiles / 8 columns /
//     now: 128 tokens, 4 experts of 4096 x 11008 814 / 1410 / 684 us, 1024 tokens, 32 of 4096 x 1376 772 / 1413 / 698);
//   * a workgroup (4 wavefronts, three LDS stages of 32 k) walks down a strip of row tiles, the k tiles of all of them one
//     sequence: a tile is stored while the copies of the next one are in flight, and a second workgroup on the compute
//     unit fills the rest.  Workgroups that run at a time take neighbouring column tiles of the same rows, so that lines which
//     two tiles share meet in L2 (37 rows, f = 688: along the columns 197 us, 160 down the rows);
//   * an expert's strips are the shorter, the more k tiles it has, so that all strips cost about the same, and those of an expert
//     with far more rows than the average go to all XCDs: a routing that has collapsed is shared out over all workgroups (3953 of 4096
//     rows on one of 64 experts of 4096 x 704: backward pass 758 us; 1054 with its strips on one XCD after another).
// us, (dW1, dW3) / dW2 with the transposing launch, before -> now, 64 experts of 4096 x 688, top-8: 37 rows 193 / 102 + 43 ->
// 160 / 73, 188 rows 349 / 167 + 94 -> 300 / 160, 375 rows 461 / 229 + 158 -> 450 / 239; 16 of 1032 x 264, 250 rows 29 / 25 + 8 ->
// 16 / 12.  Tried: one workgroup of 8 wavefronts on 256 x 256 with B's k tiles kept in LDS (188 rows 286 / 155, but 16 of 1032 x
// 264 27 / 15), the same with the ping-pong schedule (316 / 180).
template <int MODE, typename ET, bool STREAM> struct DwStrip {
  using H = Gemm<256, 256, 64, 2, 4, 3, 2, MODE>;       // its LDS layouts
  static constexpr int WM = MODE == DW13 ? 4 : 2, WN = 4 / WM, BM = 64 * WM, BN = 128 * WN, BK = 32;
  static constexpr bool A_GATHER = MODE == DW13;         // the operand of token rows: x (A), or dY (B); 256 columns either way
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES, STAGES = 3;
  static constexpr int LDS_BYTES = STAGES * STAGE;
  static constexpr int A_LOADS = A_BYTES / 4096, B_LOADS = B_BYTES / 4096, LOADS = A_LOADS + B_LOADS;   // of a wavefront, per k tile
  static constexpr int PRODUCTS = MODE == DW13 ? 2 : 1, ES = sizeof(ET);
  static constexpr int STORES = 4 * 4 * (ES / 2);         // of a wavefront, per tile
  static constexpr int LANE_COLS = 16 / ES;               // columns of B in a row that a lane reads and stores: 16 bytes of the result
  // strips to aim at: four for every workgroup that runs at a time; what storing a tile costs, in k tiles
  static constexpr int kStrips = 2048, kStoreCost = 8;
  static constexpr int kXcdStrips = 32;                   // compute units of an XCD
  static constexpr float kLong = 1.15f;                   // a long expert's tiles cost more than so many average ones

  // block: of `blocks`, a multiple of 8
  static __device__ void run(const MArgs& g, unsigned block, unsigned blocks, char* smem) {
    const int lane = threadIdx.x & (kWave - 1);
    const int nx = g.tiles_n * PRODUCTS, xe = min(lane, g.E - 1);
    const int x_cost = kStoreCost + (g.offsets[xe + 1] - g.offsets[xe] + BK - 1) / BK;
    const float costs = wave_sum(lane < g.E ? (float)x_cost : 0.f), all = costs * (float)nx * (float)g.tiles_m;
    const int x_len = min(max((int)(all / ((float)kStrips * (float)x_cost)), 1), g.tiles_m);
    const int x_strips = lane < g.E ? (g.tiles_m + x_len - 1) / x_len : 0, xcd = block % 8;
    // The strips of long experts, then the others', each dealt to the XCDs in eighths: a long expert's cost products, the others'
    // stores, and an XCD that has one sort only leaves the other half of its means idle (experts in order, top-1 with one favoured
    // expert, backward pass: 1016 of 1600 rows on one of 8 experts of 2048 x 5504 660 us, 434 like this, 516 with tiles; 2282 of 6400
    // on one of 32 of 1024 x 2752 757, 530, 582; milder, kLong 1.5 / 1.15: 523 of 1300 rows on one of 4 of 2048 x 5504 392 / 331, tiles
    // 359; 730 of 3600 on one of 8 of 1024 x 2752 268 / 237, 260; 391 of 2400 on one of 8 of 1024 x 1376 141 / 146, 150)
    const bool x_long = lane < g.E && (float)x_cost * (float)g.E > kLong * costs;
    int incl_long = 0, n_long = 0;
    if (__builtin_expect(__ballot(x_long) != 0, 0)) {
      incl_long = wave_incl_scan_i32(x_long ? x_strips : 0, lane);
      n_long = __builtin_amdgcn_readlane(incl_long, kWave - 1) * nx;
    }
    if (n_long <= kXcdStrips) n_long = 0;                // an XCD has a unit for each and reads their rows once (16 of 1024 x 64, one with
                                                         // 8000 of 16000 rows: 424, dealt out 433)
    const int incl_rest = wave_incl_scan_i32(x_long && n_long ? 0 : x_strips, lane);
    const int share_long = (n_long + 7) / 8, shares = share_long + (__builtin_amdgcn_readlane(incl_rest, kWave - 1) * nx + 7) / 8;
    bool again = false;
    for (int pos = block / 8; pos < shares; pos += blocks / 8) {
      const bool in_long = pos < share_long;
      const int i = in_long ? xcd * share_long + pos : xcd * (shares - share_long) + pos - share_long, incl = in_long ? incl_long : incl_rest;
      const unsigned long long owners = __ballot((int64_t)incl * nx > i);
      if (owners == 0) continue;                         // past the last strip of that sort
      const int e = __ffsll((long long)owners) - 1, len = __builtin_amdgcn_readlane(x_len, e);
      const int local = i - (__builtin_amdgcn_readlane(incl, e) - __builtin_amdgcn_readlane(x_strips, e)) * nx;
      const int first = local / nx * len;
      if (again) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();                    // everybody is done with what the first copies overwrite
        __builtin_amdgcn_sched_barrier(0);
      }
      strip(g, smem, e, local % nx, first, min(first + len, g.tiles_m));
      again = true;
    }
  }

  // row tiles first .. last - 1 of column tile ct of expert e's gradient
  static __device__ __forceinline__ void strip(const MArgs& g, char* smem, int e, int ct, int first, int last) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave / WN, wn = wave % WN, lane_m = lane & 15, lane_c = lane >> 4;
    const int k_begin = __builtin_amdgcn_readfirstlane(g.offsets[e]), k_end = __builtin_amdgcn_readfirstlane(g.offsets[e + 1]);
    const int n_k = k_end - k_begin, nk = (n_k + BK - 1) / BK;
    const bool second = PRODUCTS == 2 && ct >= g.tiles_n;
    const int col0 = (ct - (second ? g.tiles_n : 0)) * BN;

    // copies: k row inside the tile and column of this lane's 16 bytes (A swizzled, B as it lies in memory)
    constexpr int ROW_LOADS = A_GATHER ? B_LOADS : A_LOADS;
    int a_k[A_LOADS], a_col[A_LOADS], b_k[B_LOADS], b_col[B_LOADS];
#pragma unroll
    for (int q = 0; q < A_LOADS; ++q) {
      H::template copy_coords<false, BM>(wave * A_LOADS + q, lane, a_k[q], a_col[q]);
    }
#pragma unroll
    for (int q = 0; q < B_LOADS; ++q) {
      const int o = (wave * B_LOADS + q) * 1024 + lane * 16;
      b_k[q] = o / (BN * 2);
      b_col[q] = min(col0 + o % (BN * 2) / 2, g.N - 8) * 2;
    }
    const uint32_t row_pitch = (uint32_t)(A_GATHER ? g.ldb : g.lda) * 2u;
    uint32_t row_off[ROW_LOADS];                         // the operand in row order: k row of the copy, in bytes
#pragma unroll
    for (int q = 0; q < ROW_LOADS; ++q) row_off[q] = (uint32_t)(A_GATHER ? b_k[q] : a_k[q]) * row_pitch;
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    // the 8 token rows of k tile kt that this wavefront copies, read through the scalar cache: vector loads would be
    // waited for together with the copies behind them
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8), aligned(4)));
    typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;
    typedef const __attribute__((address_space(4))) u32x8* scalar_ptr8;
    const scalar_ptr table = (scalar_ptr)(uintptr_t)g.row_bytes + k_begin;
    uint32_t tok[8];
    auto look_up = [&](int kt) {
      const int k = kt * BK + wave * 8;
      if (k + 8 <= n_k) {
        const u32x8 t = *(scalar_ptr8)(table + k);
#pragma unroll
        for (int x = 0; x < 8; ++x) tok[x] = t[x];
      } else {
#pragma unroll
        for (int x = 0; x < 8; ++x) tok[x] = table[min(k + x, n_k - 1)];
      }
    };
    auto tok_off = [&](int q) { return lane < 32 ? tok[2 * q] : tok[2 * q + 1]; };
    const bf16_t* const Bp = second ? g.B1 : g.B0;
    // copies of k tile kt of row tile rt to LDS
    auto issue = [&](int rt, int kt, uint32_t stage) {
      const int k0 = kt * BK;
      const bf16_t* A = A_GATHER ? g.A0 : g.A0 + (size_t)(k_begin + k0) * g.lda;
      const bf16_t* B = A_GATHER ? Bp + (size_t)(k_begin + k0) * g.ldb : Bp;
      uint32_t rows[ROW_LOADS];
#pragma unroll
      for (int q = 0; q < ROW_LOADS; ++q) rows[q] = row_off[q];
      if (k0 + BK > n_k) {                               // k rows that do not exist repeat the last one
#pragma unroll
        for (int q = 0; q < ROW_LOADS; ++q) rows[q] = min(rows[q], (uint32_t)(n_k - 1 - k0) * row_pitch);
      }
#pragma unroll
      for (int q = 0; q < A_LOADS; ++q)
        copy16_to_lds(A, (A_GATHER ? tok_off(q) : rows[A_GATHER ? 0 : q]) + (uint32_t)min(rt * BM + a_col[q], g.M - 8) * 2u,
                      stage + (wave * A_LOADS + q) * 1024);
#pragma unroll
      for (int q = 0; q < B_LOADS; ++q)
        copy16_to_lds(B, (A_GATHER ? rows[A_GATHER ? q : 0] : tok_off(q)) + (uint32_t)b_col[q], stage + A_BYTES + (wave * B_LOADS + q) * 1024);
    };

    f32x4 acc[4][8];
    auto clear = [&]() {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    ET* const C = static_cast<ET*>(second ? g.C1 : g.C0) + (size_t)e * g.strideC_e;
    const int n = col0 + wn * 128 + LANE_COLS * lane_m;
    auto store = [&](int rt) {
      const bool rows_full = (rt + 1) * BM <= g.M;
      const int m0 = rt * BM + wm * 64 + 4 * lane_c;
      if (n < g.N) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = m0 + 16 * i + v;
            ET* p = C + (size_t)m * g.ldc + n;
            if (rows_full || m < g.M) {
              if constexpr (ES == 2) {
                store_out<STREAM>(reinterpret_cast<u32x4*>(p),
                                  u32x4{pack_bf16x2(acc[i][0][v], acc[i][1][v]), pack_bf16x2(acc[i][2][v], acc[i][3][v]),
                                        pack_bf16x2(acc[i][4][v], acc[i][5][v]), pack_bf16x2(acc[i][6][v], acc[i][7][v])});
              } else {
                store_out<STREAM>(reinterpret_cast<f32x4*>(p), f32x4{acc[i][0][v], acc[i][1][v], acc[i][2][v], acc[i][3][v]});
                if (n + 64 < g.N)
                  store_out<STREAM>(reinterpret_cast<f32x4*>(p + 64), f32x4{acc[i][4][v], acc[i][5][v], acc[i][6][v], acc[i][7][v]});
              }
            }
          }
      }
    };

    clear();
    if (nk == 0) {                                       // an expert without rows: zeros
      for (int rt = first; rt < last; ++rt) store(rt);
      return;
    }
    const int n_it = (last - first) * nk;
    int next_rt = first, next_kt = 0;                    // the k tile whose copies come next
    auto advance = [&]() {
      if (++next_kt == nk) { next_kt = 0; ++next_rt; }
    };
    look_up(0);
    issue(next_rt, next_kt, smem_base);
    advance();
    look_up(next_kt);
    if (n_it > 1) {
      issue(next_rt, next_kt, smem_base + STAGE);
      advance();
      look_up(next_kt);
    }
    int it = 0, st = 0, st_next = 2 * STAGE, stored1 = 0, stored2 = 0;     // groups of STORES issued one and two k tiles ago
    for (int rt = first; rt < last; ++rt) {
#pragma unroll 1
      for (int kt = 0; kt < nk; ++kt, ++it) {
        // younger than this k tile's copies: those of the next one, and the stores
        constexpr auto cap = [](int n) { return n < 63 ? n : 63; };
        if (it + 1 == n_it) wait_vmcnt<0>();
        else if (stored1 + stored2 == 0) wait_vmcnt<LOADS>();
        else if (stored1 + stored2 == 1) wait_vmcnt<cap(LOADS + STORES)>();
        else wait_vmcnt<cap(LOADS + 2 * STORES)>();
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): the token rows of the k tile that is copied below
        stored2 = stored1;
        stored1 = 0;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();                    // this k tile published; everybody is done with the last one
        __builtin_amdgcn_sched_barrier(0);
        const char* At = smem + st;
        const char* Bt = At + A_BYTES + (8 * lane_c) * (BN * 2) + (wn * 128 + LANE_COLS * lane_m) * 2;
        bf16x8 fa[4], fb[8];
        u32x4 w[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const char* row = Bt + x * (BN * 2);
          if constexpr (ES == 2) {
            w[x] = *reinterpret_cast<const u32x4*>(row);
          } else {
            const u32x2 lo = *reinterpret_cast<const u32x2*>(row), hi = *reinterpret_cast<const u32x2*>(row + 128);
            w[x] = u32x4{lo[0], lo[1], hi[0], hi[1]};
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[i] = H::template read_tr<BM>(At, wm * 64 + i * 16, 0, lane);
        __builtin_amdgcn_sched_barrier(0);
        if (it + 2 < n_it) {                             // while the fragments are on their way
          issue(next_rt, next_kt, smem_base + st_next);
          advance();
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): fragments are in registers
        __builtin_amdgcn_sched_barrier(0);
        look_up(next_kt);                                // behind that wait: it arrives during the products
        if (kt + 1 == nk && n_k % BK != 0) {             // k rows that do not exist repeat the last one: zeros instead
          const int left = n_k - kt * BK - 8 * lane_c;
          u32x4 mask;
#pragma unroll
          for (int x = 0; x < 4; ++x) mask[x] = (2 * x < left ? 0xffffu : 0u) | (2 * x + 1 < left ? 0xffff0000u : 0u);
#pragma unroll
          for (int i = 0; i < 4; ++i) fa[i] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, fa[i]) & mask);
#pragma unroll
          for (int x = 0; x < 8; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) w[x][y] = x < left ? w[x][y] : 0u;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          u32x4 o;
#pragma unroll
          for (int x = 0; x < 4; ++x)
            o[x] = __builtin_amdgcn_perm(w[2 * x + 1][j >> 1], w[2 * x][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
          fb[j] = __builtin_bit_cast(bf16x8, o);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        st = st == 2 * STAGE ? 0 : st + STAGE;
        st_next = st_next == 2 * STAGE ? 0 : st_next + STAGE;
      }
      __builtin_amdgcn_sched_barrier(0);
      store(rt);
      clear();
      __builtin_amdgcn_sched_barrier(0);
      // only a whole tile is sure to have issued every one of its stores: vmcnt counts instructions in order
      stored1 = (rt + 1) * BM <= g.M && col0 + BN <= g.N ? 1 : 0;
    }
  }
};

// Neither product needs anything of the other: one launch, the workgroups of dW1 and dW3 first.  A launch less in small batches, and
// dW2's stores fill what the others' last strips leave idle.  us, two launches / one, training passes: 64 tokens of 256, f = 688, 4 experts
// 70.4 / 67.1; 500 of 2056, f = 136, 4 experts 99.8 / 89.8; 600 of 4096, f = 5504, 8 experts 878 / 870; 1501 of 4096, f = 688, 64 experts, top-8
// 1294 / 1273; 1200 of 2048, f = 344, 64 experts 405 / 406.
template <typename ET, bool STREAM13, bool STREAM2>
__global__ __launch_bounds__(256, 2) void dw_strip_kernel(MArgs dw13, unsigned blocks13, MArgs dw2, unsigned blocks_ds, RouterDs ds) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if (blockIdx.x < blocks13) DwStrip<DW13, ET, STREAM13>::run(dw13, blockIdx.x, blocks13, smem);
  else if (blockIdx.x < blocks13 + blocks_ds) router_ds(ds, blockIdx.x - blocks13);
  else DwStrip<DW2, ET, STREAM2>::run(dw2, blockIdx.x - blocks13 - blocks_ds, gridDim.x - blocks13 - blocks_ds, smem);
}

// compute units of the current device (looked up once per device)
int compute_units() {
  static int n[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -1;
  if (n[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 8) return -1;
    n[dev] = v;
  }
  return n[dev];
}

// The kernels use more dynamic LDS than the default limit allows: the limit is raised once per
// device and instantiation (idempotent, so a race between threads is harmless).  This must not
// happen inside a stream capture; mfma_prepare() does it for every instantiation up front.
template <auto Kernel, int LDS_BYTES> int raise_lds_limit() {
  static bool attr_set[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return BTX_ERR_HIP;
  if (!attr_set[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) !=
        hipSuccess)
      return BTX_ERR_HIP;
    attr_set[dev] = true;
  }
  return BTX_OK;
}

template <int BM, int BN, int BK, int WM, int WN, int NSA, int NSB, int MODE, int TAIL = 0, bool STREAM_B = false,
          bool STREAM = MODE == BWD_ACT || MODE == DOWN, bool ROWS = false>
int launch(MArgs g, bool prepare_only, hipStream_t s) {
  using G = Gemm<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B, STREAM, ROWS>;
  constexpr auto kernel = [] {
    if constexpr (ROWS) return mfma_gemm_kernel_rows<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B, STREAM>;
    else return mfma_gemm_kernel<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B, STREAM>;
  }();
  if (int rc = raise_lds_limit<kernel, G::LDS_BYTES>()) return rc;
  if (prepare_only) return BTX_OK;
  constexpr int BNH = G::DUAL ? BN / 2 : BN;
  g.tiles_n = ceil_div(g.N, BNH);
  g.tiles_m = G::GROUP_K ? ceil_div(g.M, BM) : ceil_div(g.R, BM) + g.E;
  // every tile has exactly one block id below (number of tiles) + 8; see the tile mapping
  g.blocks_per_e = (int)align_up((size_t)g.tiles_m * g.tiles_n, 8) + 8;
  g.total_ids = G::GROUP_K ? g.E * g.blocks_per_e : g.tiles_m * g.tiles_n + 8;
  int grid = g.total_ids;
  if constexpr (G::SPLIT) {
    // K too short for two slices of the minimum length: split_plan() would never cut
    if (ceil_div(g.K, BK) * (MODE == BWD_DX ? 2 : 1) < 2 * G::kMinSliceTiles) g.partial = nullptr;
    if (g.partial) {                                   // room for the workgroups of slices 1.. of the last round
      g.cus = compute_units();
      if (g.cus <= 0) return BTX_ERR_HIP;
      if (g.cus > kSplitMaxCus) g.partial = nullptr;   // the caller's buffer is sized for that many
      else grid += g.cus + G::kIdHoles * (G::kMaxSlices - 1);   // (left + 8)(S - 1) <= cus + 8 (S - 1) for every left
    }
  } else {
    g.partial = nullptr;
  }
  kernel<<<grid, G::NT, G::LDS_BYTES, s>>>(g);
  BTX_LAUNCH_CHECK();
  if constexpr (G::SPLIT) {
    if (g.partial) {
      mfma_split_finish_kernel<BM, BN, BK, WM, WN, NSA, NSB, MODE, TAIL>
          <<<(g.cus / 2 + G::kIdHoles) * G::TM, G::NT, 0, s>>>(g);
      BTX_LAUNCH_CHECK();
    }
  }
  return BTX_OK;
}

// row tiles of BM rows if the rows were spread evenly over the experts
int even_row_tiles(const MArgs& g, int BM) {
  const int busy = std::max(std::min(g.E, g.R), 1);
  return busy * ceil_div(ceil_div(g.R, busy), BM);
}

// K slices of a product of `tiles` small tiles of nk k tiles: as many as give every compute unit a workgroup, each of
// at least 8 k tiles, and no more than the caller's scratch holds.  DOWN of 16 tokens (4 experts of 11008 x 4096, 128
// tiles): 2 slices 68 us, 4 (two workgroups per unit) 73.
int small_slices(int64_t tiles, int nk, size_t bytes_per_slice) {
  const int64_t fill = kSplitMaxCus / std::max<int64_t>(tiles, 1), fit = (int64_t)(kSplitBytes / bytes_per_slice);
  return (int)std::max<int64_t>(std::min({fill, fit, (int64_t)(nk / 8), (int64_t)kSplitMaxSlices}), 1);
}

// left (may be NULL): in, K slices that the caller can add himself; out, those whose sums he finds in slice_sums (1: none)
template <int BM, int MODE, int TAIL, bool STREAM_B> int launch_small(MArgs g, bool prepare_only, int* left, hipStream_t s) {
  // 64 rows: three stages of both operands (72 KB); 128: two of A and three of B (80 KB, half of a compute unit's LDS)
  constexpr int WM = MODE == BWD_ACT && BM == 64 ? 1 : 2, WN = 4 / WM;
  constexpr int NSA = BM == 64 ? 3 : 2, NSB = 3;
  using G = Gemm<BM, 128, 64, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B>;
  constexpr auto kernel = mfma_small_kernel<BM, WM, WN, NSA, NSB, MODE, TAIL, STREAM_B>;
  if (int rc = raise_lds_limit<kernel, G::LDS_BYTES>()) return rc;
  if (prepare_only) return BTX_OK;
  g.tiles_n = ceil_div(g.N, G::BNH);
  g.tiles_m = ceil_div(g.R, BM) + g.E;
  g.slice_sums = reinterpret_cast<float*>(g.partial);
  g.slices = 1;
  if (MODE != BWD_ACT && g.slice_sums)
    g.slices = small_slices((int64_t)even_row_tiles(g, BM) * g.tiles_n, ceil_div(g.K, 64) * (MODE == BWD_DX ? 2 : 1),
                            (size_t)g.R * g.N * (MODE == UP ? 8 : 4));
  const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * g.slices;
  if (!grid_fits(blocks + 7, 256)) return BTX_ERR_UNSUPPORTED;
  kernel<<<(unsigned)align_up((size_t)blocks, 8), G::NT, G::LDS_BYTES, s>>>(g);
  BTX_LAUNCH_CHECK();
  const bool leave = left && g.slices <= *left;
  if (left) *left = leave ? g.slices : 1;
  if (g.slices > 1 && !leave) {
    slices_finish_kernel<MODE == UP><<<ceil_div((int64_t)g.R * (g.N / 8), 256), 256, 0, s>>>(
        g.slice_sums, g.slices, g.R, g.N, g.ldp, g.offsets, g.E, (bf16_t*)g.C0, (bf16_t*)g.C1, (bf16_t*)g.C2);
    BTX_LAUNCH_CHECK();
  }
  return BTX_OK;
}

// Row tile of a row-grouped product.  With few rows per expert a product streams the weights: what counts is how
// many bytes of them are in flight, and that no rows are computed that do not exist.  us, 4 experts of 4096 x 11008:
//   rows per expert      8 (UP / DOWN)   32          80          150         170         210
//   256                  190 / 104       190 / 107   192 / 110   196 / 115   195 / 117   197 / 121
//   64                   138 /  68       145 /  72   189 / 103
//   128                  144 /  71       150 /  74   154 /  82   222 / 125   227 / 129   235 / 133
//   192 (3 stages of B)                              160 /  90   170 / 101   179 / 104   290 / 148
// (how many rows an expert has is only known on the device: the average decides, and a routing that is far from it pays
// with a second row tile for the experts that have more.  192 rows stop at 168 on average, not where the table crosses: an
// expert that has more than 192 costs a second tile, the jump from 179 to 290, and random routing spreads by sqrt(rows).)
// A product of few 256-row tiles, even when cut along K into pieces of 32 k tiles, leaves compute units idle, and 128-row tiles
// (64 where those are too few as well) may fill them: 480 rows on each of 4 experts of 4096 x 1376: DOWN 33 us with 256 rows,
// 28 with 128; BWD_DX 66, 58; BWD_ACT 83, 43 with 64.  Or need a second round: 200 rows, 2 experts of 4096 x 11008: UP 82 with
// 256 rows, 107 with 128.  There tile_us() decides.
constexpr int kSmallRows = 110;                          // rows per expert up to which a product takes small tiles
constexpr int64_t kEnough = 192;                         // workgroups of three quarters of the compute units: 256-row tiles without question
// row tiles to expect of rows that are spread at random over the experts
double random_row_tiles(const MArgs& g, int BM) {
  const double rows = (double)g.R / g.E, m = std::ceil(rows / BM), spread = std::sqrt(2.0 * rows * (1.0 - 1.0 / g.E));
  if (spread == 0) return g.E * m;
  return g.E * m + std::round(g.E * 0.5 * std::erfc((m * BM - rows) / spread)) -
         (m > 1 ? std::round(g.E * 0.5 * std::erfc((rows - (m - 1) * BM) / spread)) : 0.0);
}
// Rounds of workgroups times what a k tile takes, us: small tiles with one workgroup on a compute unit and with two, large ones
// whole and in a last round that is cut.  Fitted to 741 shapes (1 to 64 experts, 115 to 2300 rows each, 128 x 512 to 8192 x
// 4096).  With "fewer than kEnough: small" a product was more than 5 % slower than with 256 rows at 159 of these 2964 (by up to
// half), now at 30, near a full round where single rows decide; on average 3 % behind the best tile.
template <int MODE> double tile_us(const MArgs& g, int BM) {
  constexpr bool ACT = MODE == BWD_ACT;
  const bool small = BM <= 128;
  const int cols = ceil_div(g.N, (small ? 128 : 256) / (MODE == UP ? 2 : 1)), nk = ceil_div(g.K, 64) * (MODE == BWD_DX ? 2 : 1);
  const int64_t tiles = (int64_t)(random_row_tiles(g, BM) * cols);
  const bool cut = !ACT && g.partial;
  if (small) {
    const double one = BM == 64 ? 0.44 : 0.655, pair = BM == 64 ? 0.66 : 0.95, fixed = (BM == 64 ? 2.5 : 4.0) + (ACT ? 7.0 : 0.0);
    const int slices = cut ? small_slices((int64_t)even_row_tiles(g, BM) * cols, nk, (size_t)g.R * g.N * (MODE == UP ? 8 : 4)) : 1;
    const double k = (double)nk / slices;
    const int64_t wgs = tiles * slices, rest = wgs % (2 * kSplitMaxCus), pairs = wgs / (2 * kSplitMaxCus) + (rest > kSplitMaxCus);
    return pairs * (fixed + k * pair) + (rest > 0 && rest <= kSplitMaxCus ? fixed + k * one : 0.0) + (slices > 1 ? 4.0 : 0.0);
  }
  const double fixed = 9.0 + (ACT ? 20.0 : 0.0);
  const int64_t rounds = tiles / kSplitMaxCus, left = tiles % kSplitMaxCus;
  const int64_t slices = cut && left > 0 ? std::max<int64_t>(std::min<int64_t>({kSplitMaxSlices, kSplitMaxCus / left, nk / 16}), 1) : 1;
  return rounds * (fixed + nk * 1.4) + (left > 0 ? fixed + (double)nk / slices * 1.05 : 0.0) + (slices > 1 ? 4.0 + 0.09 * left * slices : 0.0);
}
// Do byte offsets from a tile's first row (of A, and of B where its K is contiguous) or k row (of B elsewhere) need more than 32 bits?
template <int MODE> bool wide_offsets(const MArgs& g) {
  const int64_t rows = (int64_t)255 * g.K + 64, k_rows = MODE == UP || MODE == DOWN ? (int64_t)64 * g.N : 0;
  return std::max(rows, k_rows) * 2 + kCopyBias > (int64_t)1 << 32;
}
template <int MODE> int row_tile(const MArgs& g) {
  constexpr bool DUAL = MODE == UP;
  if (wide_offsets<MODE>(g)) return 64;
  const int64_t avg = g.R / std::max(g.E, 1);
  if (avg <= 48) return 64;
  if (avg <= kSmallRows) return 128;
  const int64_t tiles = (int64_t)even_row_tiles(g, 256) * ceil_div(g.N, DUAL ? 128 : 256);
  const int64_t pieces = MODE == BWD_ACT || !g.partial ? 1 : ceil_div(g.K, 64) * (MODE == BWD_DX ? 2 : 1) / 32;
  const int large = MODE != BWD_ACT && avg <= 168 ? 192 : 256;
  if (tiles * std::max<int64_t>(std::min(pieces, kSplitMaxCus / std::max<int64_t>(tiles, 1)), 1) >= kEnough) return large;
  const int small = (int64_t)even_row_tiles(g, 128) * ceil_div(g.N, DUAL ? 64 : 128) >= kEnough ? 128 : 64;
  return tile_us<MODE>(g, large) < tile_us<MODE>(g, small) ? large : small;
}

// Scratch for the K slices of a product of up to R rows, or of any smaller number of them.  Small tiles (at most one (tile,
// slice) pair of 128 x 128 sums for a compute unit; small_slices()) may be cut at any number of rows; the last round of larger
// tiles only with rows enough for those and K for two slices (row_tile(), split_plan()).
template <int MODE> size_t split_bytes(int R, int E, int N, int K) {
  const int nk = ceil_div(K, 64) * (MODE == BWD_DX ? 2 : 1), slices = std::min(nk / 8, kSplitMaxSlices);
  if (R / std::max(E, 1) > kSmallRows && nk >= 2 * Gemm<256, 256, 64, 2, 4, 3, 2, MODE>::kMinSliceTiles) return kSplitBytes;
  return slices < 2 ? 0 : std::min((size_t)slices * R * N * (MODE == UP ? 8 : 4), (size_t)kSplitMaxCus * 128 * 128 * sizeof(float));
}

// the instantiation for this row tile, way of reading the weights (stream_weights()) and K (see TAIL)
template <int MODE> int launch_rows(const MArgs& g, int tile, bool stream_b, bool prepare_only, int* left, hipStream_t s) {
  const bool whole = g.K % 64 == 0;
  if (left && tile > 128) *left = 1;                     // large tiles finish their slices themselves
  if (tile == 64 && wide_offsets<MODE>(g)) return launch_small<64, MODE, kWideTail, false>(g, prepare_only, left, s);
  auto go = [&](auto stream) {
    constexpr bool S = decltype(stream)::value;
    if (tile == 64) return launch_small<64, MODE, 0, S>(g, prepare_only, left, s);
    if (tile == 128) return launch_small<128, MODE, 0, S>(g, prepare_only, left, s);
    if constexpr (MODE != BWD_ACT)
      if (tile == 192) return launch<192, 256, 64, 2, 4, 2, 3, MODE, 0, S>(g, prepare_only, s);
    return launch<256, 256, 64, 2, 4, 3, 2, MODE, 0, S>(g, prepare_only, s);
  };
  if (whole) return stream_b ? go(std::true_type{}) : go(std::false_type{});
  if (tile == 64) return launch_small<64, MODE, 2, false>(g, prepare_only, left, s);
  if (tile == 128) return launch_small<128, MODE, 2, false>(g, prepare_only, left, s);
  if constexpr (MODE != BWD_ACT)
    if (tile == 192) return launch<192, 256, 64, 2, 4, 2, 3, MODE, 2>(g, prepare_only, s);
  if (g.K % 64 == 32) return launch<256, 256, 64, 2, 4, 3, 2, MODE, 1>(g, prepare_only, s);
  return launch<256, 256, 64, 2, 4, 3, 2, MODE, 2>(g, prepare_only, s);
}
// Weights streamed past the caches: products of one row tile per expert read them once.  Where the layer's three weights are more than
// the memory-side cache (256 MB) keeps from pass to pass, which shows from 300 MB on (plain / streamed, forward pass, us: 4 experts of 2048
// x 5504, 271 MB, 16 tokens 55 / 55, 60 tokens 56 / 59; 16 of 1024 x 2752, 271 MB, 640 tokens 66 / 69; 3 of 3072 x 5504, 304 MB, 16 tokens 73
// / 70, 120 tokens 96 / 94; 7 of 2048 x 4096, 352 MB, 16 tokens 81 / 72, 280 tokens 94 / 91), with room for experts that have more rows
// than the average (128-row tiles of 32 x 4096 x 1376, 110 rows: 274, 293; see read_once), and where a row of B is whole lines: else
// every line is fetched for two tiles (32 x 4096 x 1376, UP 137, 139).  K is whole k tiles: the forms with a K tail are not built twice.
//   4 x 4096 x 11008: 4 rows 200 / 180, 30 206 / 187, 64 244 / 232, 150 277 / 265;  8 x 2048 x 5504: 16 106 / 93, 64 127 / 122
//   32 x 1024 x 2752: 16 106 / 90, 130 168 / 143, 200 173 / 158;  32 x 2048 x 2752: 30 208 / 186, 200 294 / 283;  backward 30
//   468 / 441, 200 746 / 718
bool stream_weights(const MArgs& g, int tile) {
  const int64_t avg = g.R / std::max(g.E, 1), layer_bytes = (int64_t)6 * g.E * g.N * g.K;
  const uintptr_t at = (uintptr_t)g.B0 | (uintptr_t)g.B1 | (uintptr_t)(g.strideB_e * 2) | (uintptr_t)g.ldb * 2;
  return avg <= (tile == 128 ? 96 : tile == 256 ? 236 : tile) && layer_bytes >= 300000000 && at % 128 == 0 && g.K % 64 == 0;
}
template <int MODE> int launch_rows(const MArgs& g, hipStream_t s, int* left = nullptr) {
  const int tile = row_tile<MODE>(g);
  return launch_rows<MODE>(g, tile, stream_weights(g, tile), false, left, s);
}

template <int MODE> int prepare_rows() {
  MArgs g{};
  for (int tile : {64, 128, 192, 256})
    for (int k : {64, 32, 8, 1 << 30}) {                 // whole k tiles, half a last one, any other, wide_offsets()
      g.K = k;
      if (int rc = launch_rows<MODE>(g, tile, false, true, nullptr, nullptr)) return rc;
      if (k == 64)
        if (int rc = launch_rows<MODE>(g, tile, true, true, nullptr, nullptr)) return rc;
    }
  return BTX_OK;
}

template <typename ET, bool STREAM13, bool STREAM2> int launch_dw_strips(MArgs dw13, MArgs dw2, const RouterDs* ds, bool prepare_only, hipStream_t s) {
  using D13 = DwStrip<DW13, ET, STREAM13>;
  using D2 = DwStrip<DW2, ET, STREAM2>;
  static_assert(D13::LDS_BYTES == D2::LDS_BYTES);
  constexpr auto kernel = dw_strip_kernel<ET, STREAM13, STREAM2>;
  if (int rc = raise_lds_limit<kernel, D2::LDS_BYTES>()) return rc;
  if (prepare_only) return BTX_OK;
  auto blocks = [](MArgs& g, auto tag) {
    using D = decltype(tag);
    g.tiles_n = ceil_div(g.N, D::BN);
    g.tiles_m = ceil_div(g.M, D::BM);
    const int64_t tiles = (int64_t)g.E * g.tiles_m * g.tiles_n * D::PRODUCTS;
    return (unsigned)align_up((size_t)std::min<int64_t>(tiles, D::kStrips), 8);
  };
  const unsigned blocks13 = blocks(dw13, D13{}), blocks2 = blocks(dw2, D2{});
  const unsigned blocks_ds = ds ? (unsigned)align_up(router_ds_blocks(*ds), 8) : 0;   // the strips' are dealt to the XCDs
  kernel<<<blocks13 + blocks_ds + blocks2, 256, D2::LDS_BYTES, s>>>(dw13, blocks13, dw2, blocks_ds, ds ? *ds : RouterDs{});
  BTX_LAUNCH_CHECK();
  return BTX_OK;
}
template <typename ET> int launch_dw_strips(const MArgs& dw13, const MArgs& dw2, const RouterDs* ds, bool stream13, bool stream2, bool prepare_only, hipStream_t s) {
  if (stream13)
    return stream2 ? launch_dw_strips<ET, true, true>(dw13, dw2, ds, prepare_only, s) : launch_dw_strips<ET, true, false>(dw13, dw2, ds, prepare_only, s);
  return stream2 ? launch_dw_strips<ET, false, true>(dw13, dw2, ds, prepare_only, s) : launch_dw_strips<ET, false, false>(dw13, dw2, ds, prepare_only, s);
}

// Weight gradients: strips of few rows per expert (mfma_dw_direct()), 256 x 256 tiles above.
// Streamed stores want whole lines: 64 experts of 4096 x 688, 188 rows, dW2 (rows of 4096 columns) 188 us plain, 163 streamed; 32 of
// 4096 x 1376, 4096 rows 1236 -> 1208.  dW1 and dW3 leave a 256 x 256 tile in halves of lines and keep plain stores; with
// the two panels side by side, which makes them whole, the transposing reads cost what the stores gain (8192 rows 4346 ->
// 4450 us, 1000 rows 357 -> 367).
bool rows_of_lines(const MArgs& g) { return g.N % (g.c_is_f32 ? 32 : 64) == 0; }
// strips: streamed from half lines on (300 tokens, 64 experts of 4096 x 688, dW2 shifted by 64 bytes: the backward pass 748
// us with plain stores, 729 streamed), not from any 16-byte piece (761, 862); tiles: streamed anyhow (1501 tokens: 1066, 1054)
bool stream_strips(const MArgs& g) {
  return rows_of_lines(g) && ((uintptr_t)g.C0 % 64 | (uintptr_t)g.C1 % 64 | (uintptr_t)(g.strideC_e * (g.c_is_f32 ? 4 : 2)) % 64) == 0;
}
template <int MODE> int launch_dw(const MArgs& g, bool stream, bool prepare_only, hipStream_t s) {
  if constexpr (MODE == DW2)
    if (g.row_bytes)
      return stream ? launch<256, 256, 64, 2, 4, 3, 2, MODE, 0, false, true, true>(g, prepare_only, s)
                    : launch<256, 256, 64, 2, 4, 3, 2, MODE, 0, false, false, true>(g, prepare_only, s);
  if constexpr (MODE == DW2)
    if (stream) return launch<256, 256, 64, 2, 4, 3, 2, MODE, 0, false, true>(g, prepare_only, s);
  return launch<256, 256, 64, 2, 4, 3, 2, MODE, 0, false, false>(g, prepare_only, s);
}
int prepare_dw() {
  const MArgs g{};
  for (bool stream : {false, true}) {
    if (int rc = launch_dw<DW13>(g, stream, true, nullptr)) return rc;
    if (int rc = launch_dw<DW2>(g, stream, true, nullptr)) return rc;
    MArgs rows{};
    uint32_t any = 0;
    rows.row_bytes = &any;
    if (int rc = launch_dw<DW2>(rows, stream, true, nullptr)) return rc;
    for (bool stream2 : {false, true}) {
      if (int rc = launch_dw_strips<float>(g, g, nullptr, stream, stream2, true, nullptr)) return rc;
      if (int rc = launch_dw_strips<bf16_t>(g, g, nullptr, stream, stream2, true, nullptr)) return rc;
    }
  }
  return BTX_OK;
}

}  // namespace

int mfma_prepare() {
  if (compute_units() <= 0) return BTX_ERR_HIP;        // looked up once per device, here rather than in a launch
  if (int rc = prepare_rows<UP>()) return rc;
  if (int rc = prepare_rows<DOWN>()) return rc;
  if (int rc = prepare_rows<BWD_ACT>()) return rc;
  if (int rc = prepare_rows<BWD_DX>()) return rc;
  return prepare_dw();
}
// one dg partial per column tile of BWD_ACT
int mfma_bwd_act_partials(const FfShapes& sh) {
  MArgs g{};
  g.R = sh.R; g.E = sh.E; g.N = sh.f; g.K = sh.d;
  return ceil_div(sh.f, row_tile<BWD_ACT>(g) == 256 ? 256 : 128);
}
int mfma_bwd_act_partials_most(int f) { return ceil_div(f, 128); }

size_t mfma_forward_split_bytes(const FfShapes& sh) {
  return std::max(split_bytes<UP>(sh.R, sh.E, sh.f, sh.d), split_bytes<DOWN>(sh.R, sh.E, sh.d, sh.f));
}
size_t mfma_backward_split_bytes(const FfShapes& sh) { return split_bytes<BWD_DX>(sh.R, sh.E, sh.d, sh.f); }

// Bytes from a k tile's first k row of dh1, dh3 or ga on, rows of f elements: strips of 32 k rows, 256 x 256 tiles of 64
bool mfma_dw_ok(int R, int f, bool direct) {
  return (int64_t)std::min(R, direct ? 32 : 64) * f * 2 + (direct ? 0 : kCopyBias) <= (int64_t)1 << 32;
}

bool mfma_gather_ok(int T, int d) { return (int64_t)T * d * 2 + kCopyBias < ((int64_t)1 << 32); }

int mfma_up_swiglu(const RowSource& xs, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh,
                   void* h1, void* h3, void* act, void* partial, hipStream_t s) {
  MArgs g{};
  g.A0 = (const bf16_t*)xs.base; g.a_perm = xs.perm; g.a_k = xs.k; g.B0 = (const bf16_t*)W1; g.B1 = (const bf16_t*)W3; g.C0 = h1; g.C1 = h3; g.C2 = act; g.partial = (f32x4*)partial;
  g.offsets = off; g.E = sh.E; g.N = sh.f; g.K = sh.d; g.lda = sh.d; g.ldb = sh.f; g.ldc = sh.f; g.ldp = mfma_act_pitch(sh.f);
  g.strideB_e = sh.s13; g.R = sh.R;
  return launch_rows<UP>(g, s);
}

int mfma_down(const void* act, const void* W2, const int32_t* off, const FfShapes& sh, void* y, void* partial,
              int* slices, hipStream_t s) {
  MArgs g{};
  g.A0 = (const bf16_t*)act; g.B0 = (const bf16_t*)W2; g.C0 = y; g.partial = (f32x4*)partial;
  g.offsets = off; g.E = sh.E; g.N = sh.d; g.K = sh.f; g.lda = mfma_act_pitch(sh.f); g.ldb = sh.d; g.ldc = sh.d;
  g.strideB_e = sh.s2; g.R = sh.R;
  return launch_rows<DOWN>(g, s, slices);
}

int mfma_bwd_act(const RowSource& dys, const void* W2, const void* h1, const void* h3, const float* gates,
                 const int32_t* perm, const int32_t* off, const FfShapes& sh, void* dh1, void* dh3, void* ga,
                 bool ga_transposed, uint32_t* row_bytes, float* dg_part, hipStream_t s) {
  MArgs g{};
  g.A0 = (const bf16_t*)dys.base; g.a_perm = dys.perm; g.a_k = dys.k;
  g.B0 = (const bf16_t*)W2; g.C0 = dh1; g.C1 = dh3;
  if (ga_transposed) g.T2 = (bf16_t*)ga;
  else g.C2 = ga;
  g.row_bytes = row_bytes;
  g.ldt = mfma_dw_pitch(sh.R, sh.E);
  g.H1 = (const bf16_t*)h1; g.H3 = (const bf16_t*)h3; g.gates = gates; g.perm = perm; g.dg_part = dg_part;
  g.n_part = mfma_bwd_act_partials(sh);
  g.offsets = off; g.E = sh.E; g.N = sh.f; g.K = sh.d; g.lda = sh.d; g.ldb = sh.d; g.ldc = sh.f; g.ldp = mfma_act_pitch(sh.f);
  g.strideB_e = sh.s2; g.R = sh.R;
  return launch_rows<BWD_ACT>(g, s);
}

int mfma_bwd_dx(const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* off,
                const FfShapes& sh, void* dxs, void* partial, hipStream_t s) {
  MArgs g{};
  g.A0 = (const bf16_t*)dh1; g.A1 = (const bf16_t*)dh3; g.B0 = (const bf16_t*)W1; g.B1 = (const bf16_t*)W3; g.C0 = dxs; g.partial = (f32x4*)partial;
  g.offsets = off; g.E = sh.E; g.N = sh.d; g.K = sh.f; g.lda = mfma_act_pitch(sh.f); g.ldb = sh.f; g.ldc = sh.d;
  g.strideB_e = sh.s13; g.R = sh.R;
  return launch_rows<BWD_DX>(g, s);
}

// Rows of act, dh1, dh3 and ga start on whole lines: of rows that do not, the 128 bytes of k that a copy takes lie in two lines, of which a
// compute unit has at most 32 KB on their way, and streamed stores leave parts of lines.  Training pass, rows as wide as the expert /
// padded: 16384 tokens, 32 experts of 4096 x 1376, top-8 12047 / 11870 us (BWD_DX 2430 / 2340); 64 of 1024 x 344 1554 / 1440; 16 of 2048 x 1376,
// top-4 3394 / 3328; 64 of 1024 x 136 1062 / 1025; 1501 tokens, 64 of 4096 x 688 1251 / 1227; 800, 64 of 4040 x 616 1011 / 986; 100, 16 of
// 1000 x 264 79.2 / 79.2.  Not where that nearly doubles the rows (8 of 256 x 72 295 / 298), nor where their offsets grow past 32 bits.
int mfma_act_pitch(int f) { return f > 128 && f <= 65536 ? (int)align_up((size_t)f, 64) : f; }
int mfma_dw_pitch(int R, int E) { return (int)align_up((size_t)R, 64) + 64 * E; }
bool mfma_rows_ok(int R, int E) { return ((int64_t)align_up((size_t)R, 64) + 64 * E) * 256 * 2 < ((int64_t)1 << 32); }

// Strips from rows as they lie in memory, or 256 x 256 tiles from transposed ones: those halve the operands' way into LDS, which
// counts the more, the more rows an expert has; transposing costs the less per product, the wider the experts are.  Backward
// pass, us, tiles / strips, experts of d x f, rows per expert:
//   4096 x 11008, 4 experts:  100 722 / 583, 250 870 / 777, 360 1102 / 1079, 500 1343 / 1372, 800 1797 / 1931
//   2048 x 5504, 8 experts:   100 413 / 322, 360 617 / 586, 420 655 / 628, 600 843 / 854, 1000 1151 / 1213
//   1024 x 2752, 8 experts:   250 206 / 184, 600 315 / 294, 1000 405 / 401, 1500 521 / 535
//   4096 x 1376, 16 experts:  250 575 / 519, 1000 1280 / 1234, 1500 1801 / 1776, 2200 2504 / 2541; 520 x 1400, 8: 1000 229 / 230
//   4096 x 688, 64 experts:   188 1000 / 881, 500 1807 / 1646; 8: 3200 1180 / 1112;  1032 x 264, 16: 3200 655 / 476
//   256 x 192, 64 experts:    188 178 / 94, 500 251 / 154, 5000 2284 / 1555;  8: 375 77 / 60, 1500 137 / 131, 2500 199 / 200, 5000 335 / 350
// Few strips, those of few experts of few columns, leave a long contraction to few workgroups, the more so when the 256 columns of a
// row tile are not all there; from d * E = 4096 on nothing is lost at any number of rows (8192 with fp32 gradients, whose k tiles take
// more reads from LDS: 512 x 64, 8 experts of 5290 rows 342 / 361, 1024 x 128, 8 of 2567 238 / 227):
//   512 x 64:  1 expert 1800 118 / 117, 3700 190 / 200, 20000 814 / 903;  4: 2566 162 / 160, 5043 273 / 282;  8: 5290 344 / 337, 21361 1311 /
//   1263;  512 x 352, 4: 2566 176 / 176;  1024 x 64, 4: 20165 1133 / 1100
//   64 x 64:  4 experts 742 69 / 68, 2569 140 / 153;  64: 9442 2119 / 1789;  128 x 352:  16: 700 129 / 119, 3061 283 / 292;  32: 3354 589 / 492
// The average decides, and a favoured expert's rows are more: half of all rows on one of 8, average as given: 512 x 520 1300 313 / 326,
// 256 x 192 375 119 / 113, 700 173 / 172, 1000 220 / 230, 504 x 1400 750 247 / 265.  Below 512 columns, where the chain is the larger part,
// the limits are tighter for that.
bool mfma_dw_direct(const FfShapes& sh, int dW_dtype) {
  const int64_t rows = sh.R / std::max(sh.E, 1);
  if (rows <= 360) return true;
  if ((int64_t)sh.d * sh.E < (dW_dtype == BTX_F32 ? 8192 : 4096) && rows > (sh.d < 512 ? 700 : 2500)) return false;
  return rows * sh.f <= (sh.d < 512 ? 700000 : 1300000);
}

// dW2 of 256 x 256 tiles from token rows of dY as they lie, turned around by transposing reads as dh1 and dh3 are, or from rows that the
// gather has transposed with x's?  Rows spare half of that gather, the same for experts of any width (0.63 us per million elements), and take a
// quarter more reads from LDS per product and the looking up of the rows: 0.12 us of a k tile and round of tiles, so what is lost grows with
// the width, counted with what a last column tile has too much, and where the tiles do not fill the chip with the k tiles alone.  Backward
// pass, us, transposed / rows: 16384 tokens, 32 experts of 4096 x 1376, top-8 8364 / 8077 (the gather 677 / 341, dW2 1217 / 1290); 64 of 4096 x
// 688 5599 / 5266; 16 of 4096 x 2752, top-4 7274 / 7182; 32 of 1024 x 688, top-8 1756 / 1626; 4 of 4096 x 4096, top-2 5010 / 4948, 6144 7363 / 7335,
// 8192 9622 / 9623, 11008 (a training pass) 19254 / 19357; 4001, 4 of 2048 x 5504 1026 / 1029; 8192, 1 of 4096 x 6144 1910 / 1917.  Few tiles and
// narrow rows: 16384 tokens, 1 expert of 1024 x 1376 734 / 745, 64 x 344 556 / 587; 4, top-2, of 64 x 344 378 / 393, 512 x 344 454 / 452; 1050 rows,
// 1 of 64 x 1400 83 / 87, 9 of 520 x 2752 336 / 337.  Of 262 random shapes that the rule takes three are 0.6 to 1.4 % slower, all together 3 % faster;
// 58 beside it would gain 0.7 % all together, the best 4 %.
bool mfma_dw2_rows(const FfShapes& sh) {
  return sh.d >= 256 && (int64_t)sh.d * sh.E >= 4096 && (int64_t)sh.f * (int64_t)align_up((size_t)sh.d, 256) <= (int64_t)4096 * sh.d;
}

namespace {
MArgs dw13_args(int dW_dtype, const RowSource& xs, const void* dh1, const void* dh3, const int32_t* off, const FfShapes& sh, void* dW1, void* dW3) {
  MArgs g{};
  g.A0 = (const bf16_t*)xs.base; g.B0 = (const bf16_t*)dh1; g.B1 = (const bf16_t*)dh3; g.C0 = dW1; g.C1 = dW3;
  g.offsets = off; g.E = sh.E; g.M = sh.d; g.N = sh.f; g.lda = xs.perm ? sh.d : mfma_dw_pitch(sh.R, sh.E); g.ldb = mfma_act_pitch(sh.f); g.ldc = sh.f;
  g.strideC_e = sh.s13; g.R = sh.R; g.c_is_f32 = dW_dtype == BTX_F32;
  return g;
}
MArgs dw2_args(int dW_dtype, const void* ga, const RowSource& dys, const int32_t* off, const FfShapes& sh, void* dW2) {
  MArgs h{};
  h.A0 = (const bf16_t*)ga; h.B0 = (const bf16_t*)dys.base; h.C0 = dW2;
  h.offsets = off; h.E = sh.E; h.M = sh.f; h.N = sh.d; h.lda = h.ldb = mfma_dw_pitch(sh.R, sh.E); h.ldc = sh.d;
  if (dys.perm) { h.lda = mfma_act_pitch(sh.f); h.ldb = sh.d; }          // strips; tiles: mfma_bwd_dw2()
  h.strideC_e = sh.s2; h.R = sh.R; h.c_is_f32 = dW_dtype == BTX_F32;
  return h;
}
}  // namespace

int mfma_bwd_dw13(int dW_dtype, const RowSource& xs, const void* dh1, const void* dh3, const int32_t* off, const FfShapes& sh, void* dW1,
                  void* dW3, hipStream_t s) {
  const MArgs g = dw13_args(dW_dtype, xs, dh1, dh3, off, sh, dW1, dW3);
  return launch_dw<DW13>(g, rows_of_lines(g), false, s);
}
int mfma_bwd_dw2(int dW_dtype, const void* ga, const RowSource& dys, const int32_t* off, const FfShapes& sh, uint32_t* row_bytes, void* dW2,
                 hipStream_t s) {
  MArgs g = dw2_args(dW_dtype, ga, dys, off, sh, dW2);
  g.lda = mfma_dw_pitch(sh.R, sh.E);
  g.row_bytes = row_bytes;
  return launch_dw<DW2>(g, rows_of_lines(g), false, s);
}
int mfma_bwd_dw_direct(int dW_dtype, const RowSource& xs, const RowSource& dys, const void* dh1, const void* dh3, const void* ga,
                       const int32_t* off, const FfShapes& sh, uint32_t* row_bytes, void* dW1, void* dW3, void* dW2,
                       const RouterDs* ds, hipStream_t s) {
  MArgs g = dw13_args(dW_dtype, xs, dh1, dh3, off, sh, dW1, dW3), h = dw2_args(dW_dtype, ga, dys, off, sh, dW2);
  g.row_bytes = h.row_bytes = row_bytes;
  if (g.c_is_f32) return launch_dw_strips<float>(g, h, ds, stream_strips(g), stream_strips(h), false, s);
  return launch_dw_strips<bf16_t>(g, h, ds, stream_strips(g), stream_strips(h), false, s);
}

}  // namespace btx
