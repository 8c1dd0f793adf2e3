// Linear layers: C[M,N] = A[M,K] * Wt[N,K]^T with fused epilogues.
//   bf16: MFMA (v_mfma_f32_16x16x32_bf16) kernels, operands DMA'd into swizzled LDS tiles,
//         fp32 accumulation.
//   fp32: MFMA kernels, on three bf16 parts of a value or (small products, and what the parts cannot hold)
//         v_mfma_f32_32x32x2_f32; a plain LDS-tiled FMA kernel for operands that are not made of whole aligned 16-byte chunks.
// Both operands are contiguous along K ("TN" form): activations are [tokens, K]
// and weights are stored [out, in].
#include <type_traits>
#include "common.h"

namespace fc {

// ---------------------------------------------------------------- bf16 MFMA kernel, direct-to-LDS
// Block tile BM x BN x 64, NW = WR x WC waves, each wave owns a (BM/WR) x (BN/WC) tile built
// from 16x16 MFMA accumulators.  MFMA operand layout (16x16x32, wave64), lane = i + 16*h:
//   A: row i of the 16-row tile, k = 8h .. 8h+7        (8 bf16 = one 16-byte LDS read)
//   B: column i of the 16-col tile, k = 8h .. 8h+7
//   D: column i, rows 4h + e in register e
// 16x16x32 and not 32x32x16: the matrix pipe runs at the power limit, and 16x16x32, which reads and writes half as many
// sums per product, holds a higher clock there (fc_bench_pipe_rates, random operands out of registers: 1926 TFLOP/s at 1.99 GHz against
// 1716 at 1.72), and its sums are those of two 32x32x16 bit for bit.
// The operand tiles go from global memory straight into LDS (buffer_load ... lds: lane l's 16 bytes land at
// base + 16 l), two or three stages of A's rows and, behind them, two of B's (DldsStages), with no register staging and no ds_write.
//
// LDS layout of a stage: its rows, 128 bytes each, unpadded.
// A 256-byte LDS line holds 2 rows; chunk kc (16 bytes) of row r sits at
//   line r/2, slot (r % 2) * 8 + (kc ^ ((r/2) % 8)),
// so that the 16 rows a ds_read_b128 touches at one kc fall into 16 distinct slots
// (no bank conflicts).  Because the DMA fixes the LDS position per lane, the swizzle
// is applied on the global side: each lane fetches the chunk that belongs in its slot.
//
// Tile order.  Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.
// Id -> tile index is chosen so that 32 workgroups running together on one XCD hold 32
// consecutive tile indices, and consecutive indices walk 8 tile rows before moving to
// the next tile column: an XCD works on an 8 x 4 patch of C and streams 8 + 4 operand
// panels through its L2 instead of 1 + 32.  (Products of few tile columns row by row, so that no rows are read by two XCDs: 2 to 9 % faster
// where operands come by turns from four products, 1 to 2 % slower inside a step.)
[[maybe_unused]] constexpr int kPatchRows = 8;
// (tile_index: the tile of a workgroup id, and how a last round of fewer than 256 is dealt out.)
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void gbl_void;

// s_waitcnt vmcnt(N) only (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14])
template <int N> __device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// acc += x * y, 16x16x32.  An instruction of its own in asm for one reason: its sum has to stay in its registers.  The compiler ties the
// sums of 32x32 instructions to their inputs but not those of four registers, moves them about between the two halves of a K
// tile and then spills (50 registers of the 256x256 tile).  What the compiler would see to otherwise: nothing but other
// such instructions on the same registers touches a sum before settled(), and no vector instruction writes an operand, a copied fragment or a
// zeroed sum, within two issue slots in front.  The source does not force either; both are read off the built code in a test.
__device__ __forceinline__ void mfma_into(f32x4& acc, const bf16x8& x, const bf16x8& y) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(__builtin_bit_cast(f32x4, x)), "v"(__builtin_bit_cast(f32x4, y)));
#endif
}
// The last of them are over (a result is there 11 cycles of issue behind its instruction): other instructions may use the sums.
template <int TM, int TN>
__device__ __forceinline__ void settled(f32x4 (&acc)[TM][TN]) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));
#endif
}

__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Split-K partial tiles: a wave's accumulators in the order (i, j, lane), 16
// bytes per lane, so that every wave-store covers 1 KB of consecutive addresses.  The
// fix-up kernel reads them back in the same order: no layout knowledge beyond this pair.
template <int TM, int TN>
__device__ __forceinline__ void store_partial(const f32x4 (&acc)[TM][TN], float* tile) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  f32x4* dst = (f32x4*)tile + (size_t)wave * (TM * TN * 64) + lane;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) dst[(i * TN + j) * 64] = acc[i][j];
}
// acc = the sum of `splits` of them, `stride` floats apart, in order.  Loads run a group ahead of the additions: left to itself the compiler
// keeps one to three on their way (300 x 2304 x 2048 in 256x192 tiles, four ranges of K: 48.7 us with one, 30.2 with three, 23.2 here).
template <int TM, int TN>
__device__ __forceinline__ void add_partials(f32x4 (&acc)[TM][TN], const float* tile, int wave, int splits, size_t stride) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int G = TM * TN % 8 == 0 ? 8 : 6, NG = TM * TN / G;
  static_assert(TM * TN % G == 0, "whole groups");
  const f32x4* src = (const f32x4*)(tile + (size_t)wave * (TM * TN * 256)) + (threadIdx.x & 63);
  f32x4 v[2][G];
  auto load = [&](int r, int g, f32x4 (&to)[G]) {
#pragma unroll
    for (int x = 0; x < G; ++x) to[x] = src[(size_t)r * (stride / 4) + (g * G + x) * 64];
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{-0.0f, -0.0f, -0.0f, -0.0f};      // (x + -0 is x)
  load(0, 0, v[0]);
  for (int r = 0; r < splits; ++r) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      // past the end the last group again (never used)
      load(g + 1 < NG ? r : min(r + 1, splits - 1), (g + 1) % NG, v[(g + 1) & 1]);
#pragma unroll
      for (int x = 0; x < G; ++x) acc[(g * G + x) / TN][(g * G + x) % TN] += v[g & 1][x];
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NG % 2 == 1) {
#pragma unroll
      for (int x = 0; x < G; ++x) v[0][x] = v[1][x];
    }
  }
#endif
}

// Bias and gate of a wave's WTN columns, one value a lane and register, and as the epilogue reads them: in LDS that the wave alone uses.
// Fetched when the tile is begun (loads in the epilogue are waited for in turn behind the stores issued before them: the counter is
// shared); LDS holds them only there, in a stage that is then idle, so that the operands have all of it until then.
// Columns past N, never stored, read as zero.
template <int WTN, typename Epi>
struct TileVectors {
  static constexpr int NV = ((Epi::kHasGate ? 2 : 1) * WTN + 63) / 64, BYTES = 2 * WTN * 4;
  float v[NV];
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type
  __device__ __forceinline__ void fetch(const Epi& epi, int lane, int n0, int N) {       // n0: the wave's first column
    const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)epi.P.bias, 0, epi.P.bias ? N * 4 : 0, 0x00020000);
    const auto rg = __builtin_amdgcn_make_buffer_rsrc((void*)epi.P.gate, 0, Epi::kHasGate && epi.P.gate ? N * 4 : 0, 0x00020000);
#pragma unroll
    for (int x = 0; x < NV; ++x) {
      const int c = x * 64 + lane;
      // (WTN is 32, 48, 64, 96 or 128: lanes of one load may belong to bias and to gate)
      if (x * 64 + 63 < WTN || !Epi::kHasGate)
        v[x] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb, (n0 + c) * 4, 0, 0));
      else if (x * 64 >= WTN)
        v[x] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, (n0 + c - WTN) * 4, 0, 0));
      else
        v[x] = c < WTN ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb, (n0 + c) * 4, 0, 0))
                       : __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, (n0 + c - WTN) * 4, 0, 0));
    }
  }
#endif
  __device__ __forceinline__ void to_lds(const Epi& epi, int lane, float* lds) const {   // bias, then gate (absent: ones)
    const bool ones = Epi::kHasGate && !epi.P.gate;
#pragma unroll
    for (int x = 0; x < NV; ++x) {
      const int c = x * 64 + lane;
      if (c < (Epi::kHasGate ? 2 : 1) * WTN) lds[c] = ones && c >= WTN ? 1.0f : v[x];
    }
  }
};

// Epilogue of a wave's WTM x WTN part of a tile, shared by the product kernels and the split-K fix-up: bias,
// activation / gate / q scale, conversion and stores.  (wm0, wn0): its place in the output, the same for all lanes; `cst`: SLICE bytes of
// LDS that the wave alone uses (output rows pass through them), `vectors` those that TileVectors wrote.
template <int WTM, int WTN, int SLICE, typename Epi>
__device__ __forceinline__ void wave_epilogue(const f32x4 (&acc)[WTM / 16][WTN / 16], unsigned char* cst, const float* vectors,
                                              const Epi& epi, int wm0, int wn0, int M, int N) {
  constexpr int TM = WTM / 16, TN = WTN / 16;
  // The lane number passes through an empty asm: everything derived from it here (LDS
  // staging offsets, output offsets) is then computed inside the epilogue.  Left to itself the
  // compiler computes these per-lane constants once, ahead of the persistent tile loop, finds no
  // registers for them across the K loop and reloads them from scratch in the epilogue, each
  // reload waiting for the stores issued before it.
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int li = lane & 15, lh = lane >> 4;
  if constexpr (Epi::kRowRuns) {
    // Accumulator lane (li, lh) holds row m = 16 i + li, columns 16 j + 4 lh + e.
    // The finished bf16 values go, PR rows at a time, through this wave's slice of the
    // idle operand stage, swizzled by 16-byte chunk, and leave as 16-byte stores: a
    // wave-store covers whole 2 WTN-byte row segments instead of 2 bytes per lane.
    constexpr int ROWB = WTN * 2;                     // bytes per staged row
    constexpr int CPRW = WTN / 8;                     // 16-byte chunks per row
    constexpr int RPLC = 256 / ROWB > 0 ? 256 / ROWB : 1;   // rows per 256-byte LDS line
    constexpr bool POW2 = (CPRW & (CPRW - 1)) == 0;
    constexpr int PR = 32 * ROWB <= SLICE ? 32 : 16;
    static_assert(PR * ROWB <= SLICE && WTM % PR == 0, "staging area");
    static_assert((PR * CPRW) % 64 == 0, "whole wave-stores");
    // chunk position inside a row: XOR with the line index (power-of-two rows), else a rotation
    auto swz = [](int row, int chunk) {
      return POW2 ? (chunk ^ ((row / RPLC) & (CPRW - 1))) : (chunk + row) % CPRW;
    };
#pragma unroll
    for (int i = 0; i < WTM / PR; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int h = 0; h < PR / 16; ++h) {
          const f32x4& a = acc[i * (PR / 16) + h][j];
          const int c0 = j * 16 + lh * 4, row = h * 16 + li;      // of the wave's columns, of the pass's rows
          float v[4] = {a[0], a[1], a[2], a[3]};
          epi.apply4(wn0 + c0, v, vectors + c0, vectors + WTN + c0);
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16_t)v[e];
          *(bf16x4*)(cst + row * ROWB + (swz(row, 2 * j + (lh >> 1)) << 4) + (lh & 1) * 8) = o;
        }
      constexpr int NIT = PR * CPRW / 64;
      const int m0 = wm0 + i * PR;
      if (m0 + PR <= M && wn0 + WTN <= N) {
        // whole rows (wave-uniform): all reads of the pass in flight together, no predicates,
        // and for the row-major outputs a wave-uniform row pointer plus a 32-bit lane offset
        constexpr int RB = NIT % 4 == 0 ? 4 : NIT % 3 == 0 ? 3 : NIT % 2 == 0 ? 2 : 1;   // reads in flight together
        // per-head outputs: with 64 % CPRW == 0 a lane keeps its column over all passes
        constexpr bool kFixedCol = !Epi::kLinearOut && 64 % CPRW == 0;
        bf16_t* colp = nullptr;
        if constexpr (kFixedCol) colp = epi.head_col_ptr(wn0 + (lane % CPRW) * 8);
#pragma unroll
        for (int it0 = 0; it0 < NIT; it0 += RB) {
          bf16x8 o[RB];
#pragma unroll
          for (int r = 0; r < RB; ++r) {
            const int idx = (it0 + r) * 64 + lane;
            const int row = idx / CPRW, chunk = idx % CPRW;
            o[r] = *(const bf16x8*)(cst + row * ROWB + (swz(row, chunk) << 4));
          }
#pragma unroll
          for (int r = 0; r < RB; ++r) {
            const int idx = (it0 + r) * 64 + lane;
            const int row = idx / CPRW, chunk = idx % CPRW;
            if constexpr (Epi::kLinearOut)
              __builtin_nontemporal_store(o[r], (bf16x8*)(epi.row_ptr(m0, wn0) + ((unsigned)row * (unsigned)epi.P.ldo + (unsigned)chunk * 8u)));
            else if constexpr (kFixedCol)
              __builtin_nontemporal_store(o[r], (bf16x8*)(colp + epi.head_row_off(m0 + row)));
            else
              __builtin_nontemporal_store(o[r], (bf16x8*)epi.run8(m0 + row, wn0 + chunk * 8));
          }
        }
      } else {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int idx = it * 64 + lane;
          const int row = idx / CPRW, chunk = idx % CPRW;
          const bf16x8 o = *(const bf16x8*)(cst + row * ROWB + (swz(row, chunk) << 4));
          const int m = m0 + row, n0 = wn0 + chunk * 8;
          if (m < M && n0 < N) __builtin_nontemporal_store(o, (bf16x8*)epi.run8(m, n0));
        }
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const auto col = epi.col(wn0 + j * 16 + li);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
        epi.store4(col, wm0 + i * 16 + lh * 4, v);
      }
    }
  }
}

// s_waitcnt vmcnt(N) lgkmcnt(0)
template <int N> __device__ __forceinline__ void wait_vm_lgkm0() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4));
}
// The same where the operations that may stay in flight are plain loads: nothing that touches memory moves across, neither in the
// optimiser (the empty asm; it does not hold loads through a __restrict__ pointer, which such a kernel therefore does not take) nor
// in the scheduler.
template <int N> __device__ __forceinline__ void counted_wait_lgkm0() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  wait_vm_lgkm0<N>();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
// ---------------------------------------------------------------- the product kernel
// Addresses are buffer offsets.  A lane's byte offset inside an operand panel is the
// same for every tile and every K tile: the tile enters through the base of a buffer resource
// rebuilt per tile in scalar registers, the K tile through the scalar offset of the load.  Rows
// past the end of an operand are out of the resource's range and load as zero.
//
// A K tile is 2 TN columns of products (two halves of K, 32 each), TM matrix instructions a column.  The fragment of
// a column is read AHEAD columns before it is multiplied; the row fragments of the second half are read
// during the first.  The barrier that publishes K tile g + 1 sits TAIL columns before the end of g, whose
// fragments are all in registers by then.  After it a wave requests K tile g + 2 (of A's rows, where they have three stages, g + 3) into the stages it
// has just stopped reading, reads the first fragments of g + 1, and only then multiplies g's
// last columns: neither the requests nor the LDS latency of the first fragments find the matrix
// pipe empty, and a DMA still has a whole K tile of matrix work to land.
// us, with 32x32x16 instructions and this form, same products by turns: 256x256 tiles 17776 x 12288 x 3072 1108, 1046, 9326 x 8192 x 2048
// 284, 263; 384x192 17776 x 3072 x 12288 1047, 981; 256x192 32768 x 1152 x 1152 98, 92; 128x128 9326 x 2048 x 2048 85, 80.
// LDS of k_gemm_dlds: a row of either operand is 128 bytes of a K tile; SA stages of A rows, two of B rows.  A's rows come from HBM and have two K
// tiles of time to arrive with three stages, the weights, which all workgroups read, from the caches.  us with two stages and three,
// operands by turns: 32768 x 1152 x 4608 in 256x192 tiles 319, 284, 32768 x 1152 x 1152 93, 82, 8192 x 1152 x 4608 104, 90; 32768 x 4608 x 1152
// in 256x256 327, 308.  384x192 tiles have no room for a third; 128x128 tiles, two to a CU, gain at some sizes (0.89) and lose at others (1.12).
template <int BM, int BN, int NW> struct DldsStages {
  static constexpr int A = BM * 128, B = BN * 128, SA = NW == 8 && 3 * A + 2 * B <= 160 * 1024 ? 3 : 2, BYTES = SA * A + 2 * B;
};
constexpr int kUnitKTiles = 2;                             // K tiles of the shortest unit of work of a tile with three stages (the dispatch and split_ranges)
template <int BM, int BN, int WR, int WC, typename Epi>
__global__ __launch_bounds__(WR * WC * 64) void k_gemm_dlds(const bf16_t* A, const bf16_t* Wt,
                                                           int M, int N, int K, int tiles_m, int tiles_n, Epi epi,
                                                           int splits, float* partial) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  constexpr int NW = WR * WC;
  constexpr int WTM = BM / WR, WTN = BN / WC;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int AHEAD = TN < 5 ? TN : 5, TAIL = AHEAD - 1, COLS = 2 * TN;
  static_assert(TN >= 4 && TM <= 2 * TN, "fragments of the second half are read during the first");
  constexpr int BK = 64, CPR = BK / 8, RPL = 16 / CPR, RW = 4 * RPL;      // 128-byte rows, two halves of 32
  constexpr int LA = BM / RW / NW, LB = BN / RW / NW;      // wave-loads per wave and K tile: rows of A, rows of Wt
  static_assert(BM % (RW * NW) == 0 && BN % (RW * NW) == 0, "loads must divide among waves");
  static_assert(LB <= LA, "B shares A's lane offsets");
  static_assert(TAIL * TM >= LB + LA && TAIL * TM >= TM + AHEAD, "requests and first fragments go between the last columns' products");
  static_assert((NW * 4) % CPR == 0 && (BM / RW * 4) % CPR == 0, "the swizzle must not depend on the load index");
  using L = DldsStages<BM, BN, NW>;
  constexpr int SA = L::SA, B_REGION = SA * L::A;
  static_assert(SA - 1 <= kUnitKTiles, "a unit's requests reach at most into the next one");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / WC, wc = wave % WC;
  const int li = lane & 15, lh = lane >> 4;
  // ---- tiles of this workgroup: virtual ids blockIdx.x, + gridDim.x, ... below `padded`
  // (the grid may be one workgroup per slot of the chip: persistent).  gridDim.x is a
  // multiple of 8, so every id of a workgroup lands on its XCD.
  // Split-K remainder (splits >= 2; the grid is then 256 workgroups): the tiles of the last,
  // partial round of 256 are each cut into `splits` ranges of K and dealt to the workgroups
  // of that round, which store their fp32 accumulators to `partial` (slot = tile-in-round *
  // splits + range) instead of running the epilogue; k_gemm_fixup adds the ranges in a
  // fixed order and finishes the tile.  A round that leaves most of the chip idle for the
  // time of a whole tile thus costs 1 / splits of it.
  const int total = tiles_m * tiles_n;
  const int nkt = K / BK;
  const int full = total / 256 * 256, rem = total - full;
  // virtual ids run over the whole rounds and, behind them, the units of the last one
  const int padded = splits >= 2 ? ((full + rem * splits + 7) & ~7) : (total + 255) / 256 * 256;
  auto tile_of = [&](int vb, int& bm0, int& bn0, int& kt0, int& kt1, int& slot) {
    int t = tile_index(vb, total);
    kt0 = 0; kt1 = nkt; slot = -1;
    if (splits >= 2 && vb >= full) {
      const int w = vb - full;
      if (w >= rem * splits) return false;
      const int r = w / rem;
      t = full + w % rem;
      kt0 = r * nkt / splits; kt1 = (r + 1) * nkt / splits;
      slot = (w % rem) * splits + r;
    }
    if (t >= total) return false;
    constexpr int GM = kPatchRows;
    const int per_group = GM * tiles_n;
    const int group = t / per_group;
    const int first_m = group * GM;
    const int gsz = min(tiles_m - first_m, GM);
    bm0 = (first_m + (t % per_group) % gsz) * BM;
    bn0 = ((t % per_group) / gsz) * BN;
    return true;
  };
  // advances vb to this workgroup's next unit of work: a tile, or a K range of a split tile
  auto next_tile = [&](int& vb, int& bm0, int& bn0, int& kt0, int& kt1, int& slot) {
    for (vb += gridDim.x; vb < padded; vb += gridDim.x)
      if (tile_of(vb, bm0, bn0, kt0, kt1, slot)) return true;
    return false;
  };

  // ---- this lane's byte offsets inside an operand panel, one per wave-load (the swizzled
  // 16-byte chunk of row (wave + NW j) RW + ... that lands in its LDS slot)
  unsigned voff[LA];
  {
    const int line_in = lane >> 4, sl = lane & 15;
    const int row0 = wave * RW + line_in * RPL + sl / CPR;
    const int kc = (sl % CPR) ^ ((wave * 4 + line_in) % CPR);
#pragma unroll
    for (int j = 0; j < LA; ++j) voff[j] = (unsigned)(row0 + NW * RW * j) * (unsigned)K * 2u + (unsigned)kc * 16u;
  }
  struct Panels { __amdgpu_buffer_rsrc_t a, b; int kbase; };
  auto panels = [&](int bm0, int bn0, int kt_first) {      // (the rows of a tile alone: below 4 GB, however large the operand)
    Panels p;
    p.a = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)bm0 * K), 0, (int)((unsigned)min(M - bm0, BM) * (unsigned)K * 2u), 0x00020000);
    p.b = __builtin_amdgcn_make_buffer_rsrc((void*)(Wt + (size_t)bn0 * K), 0, (int)((unsigned)min(N - bn0, BN) * (unsigned)K * 2u), 0x00020000);
    p.kbase = kt_first * BK * 2;
    return p;
  };
  auto dma_a = [&](const Panels& p, int kt, int stage, int j) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(p.a, (lds_void*)(smem + stage + (wave + NW * j) * 1024), 16, (int)voff[j], p.kbase + kt * (BK * 2), 0, 0);
  };
  auto dma_b = [&](const Panels& p, int kt, int stage, int j) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(p.b, (lds_void*)(smem + B_REGION + stage + (wave + NW * j) * 1024), 16, (int)voff[j], p.kbase + kt * (BK * 2), 0, 0);
  };
  // ---- fragment read offsets (bytes within a stage): the chunk of half 0, half 1's is 64 bytes across
  const int ra = wr * WTM + li, rb = wc * WTN + li;
  const int oa = (ra / RPL) * 256 + (ra % RPL) * 128 + ((lh ^ ((ra / RPL) % CPR)) << 4);
  const int ob = (rb / RPL) * 256 + (rb % RPL) * 128 + ((lh ^ ((rb / RPL) % CPR)) << 4);

  int vb = (int)blockIdx.x - (int)gridDim.x, bm0 = 0, bn0 = 0, kt0 = 0, kt1 = 0, slot = -1;
  if (!next_tile(vb, bm0, bn0, kt0, kt1, slot)) return;
  Panels cur = panels(bm0, bn0, kt0);
  int nk = kt1 - kt0;                              // K tiles of the current unit, at least SA - 1
  int ata = 0, atb = 0;                            // offsets of the stages that hold the K tile being multiplied
  auto next_a = [&](int stage) { return stage == (SA - 1) * L::A ? 0 : stage + L::A; };
#pragma unroll
  for (int j = 0; j < LB; ++j) dma_b(cur, 0, 0, j);
#pragma unroll
  for (int kt = 0; kt < SA - 1; ++kt)
#pragma unroll
    for (int j = 0; j < LA; ++j) dma_a(cur, kt, kt * L::A, j);
  counted_wait_lgkm0<(SA - 2) * LA>();
  __builtin_amdgcn_s_barrier();

  for (;;) {
    int nvb = vb, nbm0 = 0, nbn0 = 0, nkt0 = 0, nkt1 = 0, nslot = -1;
    const bool has_next = next_tile(nvb, nbm0, nbn0, nkt0, nkt1, nslot);
    Panels nxt = cur;
    if (has_next) nxt = panels(nbm0, nbn0, nkt0);
    TileVectors<WTN, Epi> vectors;
    if constexpr (Epi::kRowRuns) vectors.fetch(epi, lane, bn0 + wc * WTN, N);

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 fa[2][TM], fb[2][TN];
    auto load_a = [&](int stage, int half, int i) { fa[half][i] = *(const bf16x8*)(smem + stage + (oa ^ (half * 64)) + i * 2048); };
    auto load_b = [&](int stage, int n) { fb[n / TN][n % TN] = *(const bf16x8*)(smem + B_REGION + stage + (ob ^ (n / TN * 64)) + n % TN * 2048); };
    // fragment r of a K tile's first ones: the rows' half 0, AHEAD columns
    auto load_first = [&](int sa, int sb, int r) { if (r < TM) load_a(sa, 0, r); else load_b(sb, r - TM); };
    // A wave's requests r = 0 .. LB + LA - 1: K tile kb of B, then K tile ka of A, into stages just read.  K tiles count on into the next unit; past
    // the last unit K tile 0 of the current panels again (in range, never read) rather than branching around the loads.
    auto request = [&](int kb, int sb, int ka, int sa, int r) {
      if (r < LB) dma_b(kb < nk ? cur : nxt, kb < nk ? kb : (has_next ? kb - nk : 0), sb, r);
      else if (r < LB + LA) dma_a(ka < nk ? cur : nxt, ka < nk ? ka : (has_next ? ka - nk : 0), sa, r - LB);
    };
    auto multiply = [&](int n, int i) {
      // row-run epilogues want a lane to hold consecutive n: D rows come from the A
      // operand, so the weight fragment goes there (the operand layouts are alike)
      if constexpr (Epi::kRowRuns) mfma_into(acc[i][n % TN], fb[n / TN][n % TN], fa[n / TN][i]);
      else mfma_into(acc[i][n % TN], fa[n / TN][i], fb[n / TN][n % TN]);
    };

    // One K tile, in this order of instructions.  LAST: the unit's last one (no requests: the stage it frees is where the
    // epilogue stages its output rows).
    auto kstep = [&](auto last, int kt) {
      constexpr bool LAST = decltype(last)::value;
#pragma unroll
      for (int n = 0; n < COLS - TAIL; ++n) {
        if (n + AHEAD < COLS) load_b(atb, n + AHEAD);
#pragma unroll
        for (int i = 2 * n; i < 2 * n + 2; ++i)
          if (i < TM) load_a(ata, 1, i);
#pragma unroll
        for (int i = 0; i < TM; ++i) multiply(n, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      // K tile kt + 1 has landed (behind it came A's K tile kt + 2, if it has three stages); this wave is done reading kt
      counted_wait_lgkm0<(SA - 2) * LA>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < TAIL * TM; ++r) {
        multiply(COLS - TAIL + r / TM, r % TM);
        if constexpr (!LAST) {
          if (r < TM + AHEAD) load_first(next_a(ata), L::B - atb, r);
          request(kt + 2, atb, kt + SA, ata, r);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      ata = next_a(ata);
      atb = L::B - atb;
    };

    // B's K tile 1 and A's K tile SA - 1, into the stages that the last unit's rows went through
#pragma unroll
    for (int r = 0; r < LB + LA; ++r) {
      request(1, L::B - atb, SA - 1, SA == 3 ? next_a(next_a(ata)) : next_a(ata), r);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < TM + AHEAD; ++r) load_first(ata, atb, r);      // the only reads of a unit with no matrix work in front of them
    wait_lgkm0();                                  // (and nothing else is on its way, so that the loop's waits can count)
    __builtin_amdgcn_sched_barrier(0);
    for (int kt = 0; kt + 1 < nk; ++kt) kstep(std::false_type{}, kt);
    kstep(std::true_type{}, nk - 1);
    settled(acc);

    // Every wave is done reading the stages just multiplied: the epilogue stages its output rows in A's, its vectors in B's; the
    // next unit's first K tile is complete in others.
    if (slot < 0) {
      const int last_a = ata == 0 ? (SA - 1) * L::A : ata - L::A, last_b = B_REGION + L::B - atb;
      float* const mine = (float*)(smem + last_b + wave * TileVectors<WTN, Epi>::BYTES);
      if constexpr (Epi::kRowRuns) vectors.to_lds(epi, lane, mine);
      wave_epilogue<WTM, WTN, L::A / NW>(acc, smem + last_a + wave * (L::A / NW), mine, epi, bm0 + wr * WTM, bn0 + wc * WTN, M, N);
    } else {
      store_partial<TM, TN>(acc, partial + (size_t)slot * (BM * BN));
    }
    if (!has_next) break;
    // the staging slices are read out: the next unit's second K tile may overwrite that stage
    __builtin_amdgcn_s_barrier();
    vb = nvb; bm0 = nbm0; bn0 = nbn0; nk = nkt1 - nkt0; slot = nslot;
    cur = nxt;
  }
  wait_vm<0>();                                    // nothing is on its way to LDS when the workgroup ends
#endif
}

// ---------------------------------------------------------------- the product kernel, weights straight to registers
// For weights that were packed into fragment order when the model was loaded ([N / 16][K / 32][lane][8], k_pack_weights): a
// fragment is 1 KB in a row and goes from L2 to the registers of the one wave column that needs it; LDS holds A alone.  A
// workgroup is four waves side by side, each 128 rows by BN / 4 columns, so that no fragment is fetched twice, and small
// enough that two (BN 256: 206 registers, 34 KB of LDS), three (BN 192: 168) or four of them (BN 128: 126) share a CU: one's epilogue and first loads run
// under another's products, and tiles half the size fill the last round better.  Of k_gemm_dlds it keeps the tile order, the
// swizzled A stages and the epilogue.  Sums are those of k_gemm_dlds bit for bit where that does not split a tile along K.
//
// Products go column by column of 16 weights, all 128 rows of a column in a row: a column's registers are loaded for the next K
// tile right behind it and have nearly a whole K tile to arrive (row by row, with every column's registers in
// use to the end of a half, that was half a K tile: 0 to 18 % slower, most where a CU has one or two workgroups).  The price is that all
// row fragments of a half are needed from its first column on: they are replaced in place, one by one, under the last column before.
// Bound by the power limit with large products (17776 x 12288 x 3072: 1361 TFLOP/s), by rounds of tiles with small ones.
// us, 32x32x16 instructions row by row, and this form, operands by turns: 8192 x 1152 x 1152 (BN 128) 30.6, 25.5; 8192 x 3456 x 1152
// (BN 256) 73.8, 63.1; 32768 x 4608 x 1152 314, 304; 32768 x 1152 x 4608 304, 283; 17776 x 9216 x 3072 783, 731.
template <int BM, int BN, typename Epi>
__global__ __launch_bounds__(256, BN == 128 ? 4 : BN == 192 ? 3 : 2) void k_gemm_packed(const bf16_t* A, const void* Wp, int M, int N,
                                                        int K, int tiles_m, int tiles_n, Epi epi) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  constexpr int BK = 64, NW = 4, WTN = BN / NW, TM = BM / 16, TN = WTN / 16;
  constexpr int CPR = BK / 8, RPL = 16 / CPR, RW = 4 * RPL, LA = BM / RW / NW;
  static_assert(BM % (RW * NW) == 0 && BN % 64 == 0 && BN <= 256 && Epi::kRowRuns, "whole wave-loads");
  constexpr int STAGE_BYTES = BM * BK * 2;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lh = lane >> 4;
  float* const mine = (float*)(smem + 2 * STAGE_BYTES + wave * TileVectors<WTN, Epi>::BYTES);

  const int total = tiles_m * tiles_n, nk = K / BK, padded = (total + 255) / 256 * 256;
  auto next_tile = [&](int& vb, int& bm0, int& bn0) {      // k_gemm_dlds's order, no split tiles
    for (vb += gridDim.x; vb < padded; vb += gridDim.x) {
      const int t = tile_index(vb, total);
      if (t >= total) continue;
      constexpr int gm = kPatchRows;
      const int per_group = gm * tiles_n, group = t / per_group, first_m = group * gm, gsz = min(tiles_m - first_m, gm);
      bm0 = (first_m + (t % per_group) % gsz) * BM;
      bn0 = ((t % per_group) / gsz) * BN;
      return true;
    }
    return false;
  };
  unsigned voff[LA];                                       // this lane's byte offsets inside an A panel, as in k_gemm_dlds
  {
    const int line_in = lane >> 4, sl = lane & 15;
    const int row0 = wave * RW + line_in * RPL + sl / CPR, kc = (sl % CPR) ^ ((wave * 4 + line_in) % CPR);
#pragma unroll
    for (int j = 0; j < LA; ++j) voff[j] = (unsigned)(row0 + NW * RW * j) * (unsigned)K * 2u + (unsigned)kc * 16u;
  }
  struct Panels { __amdgpu_buffer_rsrc_t a; int b[TN]; };
  // Rows past the end of A load as zero; columns past N, which are never stored, repeat the last 16 columns: the offset that
  // chooses a fragment is a scalar one, which the buffer's range check does not cover.
  auto panels = [&](int bm0, int bn0) {
    Panels p;
    p.a = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)bm0 * K), 0, (int)((unsigned)(M - bm0) * (unsigned)K * 2u), 0x00020000);
#pragma unroll
    for (int j = 0; j < TN; ++j) p.b[j] = min((bn0 + wave * WTN) / 16 + j, N / 16 - 1) * (K / 32) * 1024;
    return p;
  };
  const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)Wp, 0, (int)((unsigned)N * (unsigned)K * 2u), 0x00020000);
  auto dma_a = [&](const Panels& p, int kt, int stage, int j) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(p.a, (lds_void*)(smem + stage + (wave + NW * j) * 1024), 16, (int)voff[j], kt * (BK * 2), 0, 0);
  };
  const int oa = (li / RPL) * 256 + (li % RPL) * 128 + ((lh ^ ((li / RPL) % CPR)) << 4);      // half 0's chunk, half 1's is 64 bytes across

  int vb = (int)blockIdx.x - (int)gridDim.x, bm0 = 0, bn0 = 0;
  if (!next_tile(vb, bm0, bn0)) return;
  Panels cur = panels(bm0, bn0);
  bf16x8 fa[TM], fb[2][TN];
  auto load_b = [&](const Panels& p, int kt, int half, int j) {
    fb[half][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, lane * 16, p.b[j] + (kt * 2 + half) * 1024, 0));
  };
  int at = 0;                                              // offset of the stage that holds the K tile being multiplied
#pragma unroll
  for (int j = 0; j < LA; ++j) dma_a(cur, 0, at, j);
#pragma unroll
  for (int n = 0; n < 2 * TN; ++n) load_b(cur, 0, n / TN, n % TN);
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  for (;;) {
    int nvb = vb, nbm0 = 0, nbn0 = 0;
    const bool has_next = next_tile(nvb, nbm0, nbn0);
    Panels nxt = cur;
    if (has_next) nxt = panels(nbm0, nbn0);
    // The tile's first product waits for all that is on its way, K tile 1 too: how many stores the epilogue put behind the fragments it
    // needs is not known when this is compiled.
    TileVectors<WTN, Epi> vectors;
    vectors.fetch(epi, lane, bn0 + wave * WTN, N);
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto load_a = [&](int stage, int half, int i) { fa[i] = *(const bf16x8*)(smem + stage + (oa ^ (half * 64)) + i * 2048); };
    // weights as the A operand: a lane ends up with consecutive columns
    auto multiply = [&](int half, int j, int i) { mfma_into(acc[i][j], fb[half][j], fa[i]); };
    // One K tile, in this order of instructions: 2 TN columns of products (two halves of K), TM instructions each.  A column's
    // weights are requested for the next K tile right behind it; the row fragments are replaced one by one
    // under the last column of a half.  LAST: the tile's last one (no requests of A: the stage it frees is where the epilogue stages its rows).
    auto kstep = [&](auto last, int kt) {
      constexpr bool LAST = decltype(last)::value;
      // past the end of this tile the next one's first K tiles, past the last tile this one's K tile 0 again (never used)
      const int kb = kt + 1 < nk ? kt + 1 : 0, ka = kt + 2 < nk ? kt + 2 : (has_next ? kt + 2 - nk : 0);
      const Panels& pb = kt + 1 < nk ? cur : nxt;
      const Panels& pa = kt + 2 < nk ? cur : nxt;
#pragma unroll
      for (int n = 0; n < 2 * TN; ++n) {
        const int half = n / TN, j = n % TN;
        if (n == 2 * TN - 1) {
          // K tile kt + 1 of A has landed: behind its DMA came 2 TN - 1 columns of weights requested since (and in front of them, but
          // for a tile's first K tile, those of this column, which it needs anyway); this wave is done reading kt
          counted_wait_lgkm0<2 * TN - 1>();
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          multiply(half, j, i);
          if (j == TN - 1 && !(LAST && half == 1)) {
            load_a(half == 0 ? at : STAGE_BYTES - at, half ^ 1, i);
            if (half == 1 && i < LA) dma_a(pa, ka, at, i);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);                 // the DMA stays ahead of the weights
        load_b(pb, kb, half, j);
        __builtin_amdgcn_sched_barrier(0);
      }
      at = STAGE_BYTES - at;
    };
#pragma unroll
    for (int j = 0; j < LA; ++j) dma_a(cur, 1, STAGE_BYTES - at, j);      // (at least two K tiles)
#pragma unroll
    for (int i = 0; i < TM; ++i) load_a(at, 0, i);
    __builtin_amdgcn_sched_barrier(0);
    for (int kt = 0; kt + 1 < nk; ++kt) kstep(std::false_type{}, kt);
    kstep(std::true_type{}, nk - 1);
    settled(acc);
    // the next tile's first K tile is complete in the other stage
    vectors.to_lds(epi, lane, mine);
    wave_epilogue<BM, WTN, STAGE_BYTES / NW>(acc, smem + (STAGE_BYTES - at) + wave * (STAGE_BYTES / NW), mine, epi, bm0, bn0 + wave * WTN, M, N);
    if (!has_next) break;
    __builtin_amdgcn_s_barrier();                          // the staging slices are read out
    vb = nvb; bm0 = nbm0; bn0 = nbn0;
    cur = nxt;
  }
#endif
}

// W [N, K] as [N / 16][K / 32][lane][8]: lane i + 16 h holds row i, columns 8 h .. 8 h + 7.  Once per model.
__global__ __launch_bounds__(256) void k_pack_weights(const bf16_t* __restrict__ W, bf16_t* __restrict__ out, int N, int K) {
  const long long x = (long long)blockIdx.x * 256 + threadIdx.x, blk = x >> 6;
  if (x >= (long long)N * K / 8) return;
  const int lane = (int)(x & 63), ks = (int)(blk % (K / 32)), nb = (int)(blk / (K / 32));
  *(bf16x8*)(out + x * 8) = *(const bf16x8*)(W + (size_t)(nb * 16 + (lane & 15)) * K + ks * 32 + (lane >> 4) * 8);
}
bool packs_weights(int N, int K) { return N % 32 == 0 && K % 64 == 0 && K >= 128 && (unsigned long long)N * K * 2 < (1ull << 31); }
hipError_t launch_pack_weights(const void* W, void* out, int N, int K, hipStream_t s) {
  if (!packs_weights(N, K)) return hipErrorInvalidValue;
  k_pack_weights<<<ceil_div((long long)N * K / 8, 256), 256, 0, s>>>((const bf16_t*)W, (bf16_t*)out, N, K);
  return hipGetLastError();
}

// ---------------------------------------------------------------- the product kernel, tiles of 128 x 288
// For widths that are whole multiples of 288 (models of 576 and 1152 columns) where such tiles fill the chip and those above do not: 8192 x 1152
// is 192 tiles of 256x192 but 256 of 128x288.  One tile to a workgroup, one workgroup to a CU.  A wave owns 64 rows by 144 columns, the
// shape that keeps LDS reads under the matrix instructions (13 fragments per 36 v_mfma_f32_16x16x32_bf16; 16 wide, as 144 is no
// multiple of 32), so the tile is four waves, one to a SIMD, and what would stop the wave stops the SIMD: fragments are read four
// columns of products ahead, and requests for operand tiles are spread over the matrix instructions (all thirteen of a wave in
// the tail of a step: 96 us where it is 76).  Sums go along K in order, and one v_mfma_f32_16x16x32_bf16 rounds like two
// v_mfma_f32_32x32x16_bf16 would: results are those of k_gemm_dlds bit for bit where that does not split a tile along K.  LDS layout, DMA and
// swizzle are those of k_gemm_dlds, as is the barrier ahead of a stage's last products, behind which the next stage's first fragments
// are read.  Three stages of LDS.
// Bound by the operand stream (53 KB per K tile in 0.9 us and CU) and, where K is small, by what is not the K loop (10 us: first tile,
// epilogue).  us, best form before and this one, operands by turns from four to six products: 8192 x 1152 x 4608 106, 76;
// 7300 x 1152 x 4608 95, 70; 15742 x 576 x 2304 57, 43; 900 x 9216 x 2304 51, 37.  (Eight waves in two groups, each on one half of every
// K tile, added at the end, took 80, 74, 44 and 38 and gave a row other sums than the other tiles do.)
struct Tile288 {
  static constexpr int BM = 128, BN = 288, kStages = 3, kStage = (BM + BN) * 128;
  static constexpr int kRow = 304;                         // bytes of a staged row of 144 results, 16 of them padding
  static constexpr int kBytes = kStages * kStage + 2 * BN * 4;        // and bias and gate of the tile's columns
};
template <typename Epi>
__global__ __launch_bounds__(256, 2) void k_gemm_288(const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wt, int M, int N, int K,
                                                     int tiles_m, int tiles_n, Epi epi) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  using L = Tile288;
  constexpr int BM = L::BM, BN = L::BN, S = L::kStages, TM = 4, TN = 9, RW = 32;        // RW: rows of a load by all waves
  static_assert(Epi::kRowRuns, "stores of 16-byte runs");
  static_assert(BM % RW == 0 && BN % RW == 0, "whole loads");
  static_assert(S * L::kStage >= 4 * 64 * L::kRow, "the results fit the stages");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  float* const sbias = (float*)(smem + S * L::kStage);
  float* const sgate = sbias + BN;

  const int total = tiles_m * tiles_n, t = tile_index(blockIdx.x, total);
  if (t >= total) return;                                  // k_gemm_dlds's tile order
  constexpr int gm = kPatchRows;
  const int per_group = gm * tiles_n, group = t / per_group, first_m = group * gm, gsz = min(tiles_m - first_m, gm);
  const int bm0 = (first_m + (t % per_group) % gsz) * BM, bn0 = ((t % per_group) / gsz) * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lh = lane >> 4;
  const int wm = wave & 1, wn = wave >> 1;
  for (int c = tid; c < BN; c += 256) {
    sbias[c] = epi.P.bias ? epi.P.bias[bn0 + c] : 0.0f;
    if constexpr (Epi::kHasGate) sgate[c] = epi.P.gate ? epi.P.gate[bn0 + c] : 1.0f;
  }

  // ---- operand tiles: 8 rows of 128 bytes a wave-load, swizzled as in k_gemm_dlds
  const int row0 = wave * 8 + (lane >> 4) * 2 + ((lane & 15) >> 3), kc = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
  const unsigned v0 = (unsigned)row0 * (unsigned)K * 2u + (unsigned)kc * 16u, rows = (unsigned)RW * (unsigned)K * 2u;
  const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)bm0 * K), 0, (int)((unsigned)(M - bm0) * (unsigned)K * 2u), 0x00020000);
  const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(Wt + (size_t)bn0 * K), 0, (int)((unsigned)BN * (unsigned)K * 2u), 0x00020000);
  auto request_a = [&](int st, int stage, int j) {         // rows past the end of A load as zero
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(smem + stage + wave * 1024 + j * RW * 128), 16, (int)(v0 + j * rows), st * 128, 0, 0);
  };
  auto request_b = [&](int st, int stage, int j) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(smem + stage + wave * 1024 + (BM + j * RW) * 128), 16, (int)(v0 + j * rows), st * 128, 0, 0);
  };
  // ---- fragments: two halves of a stage's K, one after the other
  const int fo = (li >> 1) * 256 + ((li & 1) * 8 + (lh ^ (li >> 1))) * 16;
  const int oa = fo + wm * 64 * 128, ob = fo + BM * 128 + wn * (144 * 128);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  bf16x8 fa[2][TM], fb[2][TN];
  auto load_a = [&](int stage, int half, int i) { fa[half][i] = *(const bf16x8*)(smem + stage + (oa ^ (half * 64)) + i * 2048); };
  auto load_b = [&](int stage, int half, int j) { fb[half][j] = *(const bf16x8*)(smem + stage + (ob ^ (half * 64)) + j * 2048); };
  auto multiply = [&](int half, int j) {                   // weights as the A operand: a lane ends up with consecutive columns
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[half][j], fa[half][i], acc[i][j], 0, 0, 0);
  };

  // Stages are numbered by K; stage st lies at offset st % S of LDS.  Past the end the last one is requested again (never used).
  const int nst = K / 64;
  // A stage's rows of A are requested in the tail of the step that frees its buffer, its weights along the step after.
  constexpr int kDsRead = 0x100, kMfma = 0x008, kVmem = 0x010, AHEAD = 4, LA = BM / RW, LB = BN / RW, LOADS = LA + LB;
  // All but the last `stages` stages requested; this wave's LDS reads too.
  auto landed = [&](auto stages) {
    wait_vm_lgkm0<decltype(stages)::value * LOADS>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int st = 0; st < S; ++st) {
    if (st == S - 1) landed(std::integral_constant<int, 0>{});
#pragma unroll
    for (int j = 0; j < LA; ++j) request_a(min(st, nst - 1), st * L::kStage, j);
    if (st < S - 1) {
#pragma unroll
      for (int j = 0; j < LB; ++j) request_b(min(st, nst - 1), st * L::kStage, j);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) load_a(0, 0, i);
#pragma unroll
  for (int j = 0; j < AHEAD; ++j) load_b(0, 0, j);
  __builtin_amdgcn_sched_barrier(0);
  int at = 0;                                              // offset of the stage being multiplied
  auto step = [&](int st) {
    const int after = at == (S - 1) * L::kStage ? 0 : at + L::kStage, before = at == 0 ? (S - 1) * L::kStage : at - L::kStage;
    // every fragment of the stage is read ahead of its last AHEAD columns of products
#pragma unroll
    for (int j = 0; j < 2 * TN - AHEAD; ++j) {
      const int n = j + AHEAD;
      load_b(at, n / TN, n % TN);
      if (j < TM) load_a(at, 1, j);
      if (j < LB) request_b(min(st + S - 1, nst - 1), before, j);
      multiply(j / TN, j % TN);
    }
#pragma unroll
    for (int j = 0; j < 2 * TN - AHEAD; ++j) {
      __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
      if (j < TM) __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
      if (j < LB) __builtin_amdgcn_sched_group_barrier(kVmem, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kMfma, TM - 3, 0);
    }
    landed(std::integral_constant<int, S - 2>{});          // stage st + 1 has, and every wave is done reading st
#pragma unroll
    for (int j = 0; j < LA; ++j) request_a(min(st + S, nst - 1), at, j);
#pragma unroll
    for (int i = 0; i < TM; ++i) load_a(after, 0, i);
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) load_b(after, 0, j);
#pragma unroll
    for (int j = TN - AHEAD; j < TN; ++j) multiply(1, j);
#pragma unroll
    for (int r = 0; r < AHEAD * TM; ++r) {
      __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
      if (r < LA) __builtin_amdgcn_sched_group_barrier(kVmem, 1, 0);
      else if (r < LA + TM + AHEAD) __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    at = after;
  };
  int st = 0;
  for (; st + 1 < nst; st += 2) {
    step(st);
    step(st + 1);
  }
  if (st < nst) step(st);

  // ---- epilogue: a wave's 64 rows of 144 columns through LDS that it alone uses, no longer read as stages; out in runs of 16 bytes
  wait_vm_lgkm0<0>();
  __syncthreads();
  unsigned char* const cst = smem + wave * (64 * L::kRow);
  const int nw = wn * 144, m0 = bm0 + wm * 64;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = 16 * j + 4 * lh;
      float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      epi.apply4(bn0 + nw + c, v, sbias + nw + c, sgate + nw + c);
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)v[e];
      *(bf16x4*)(cst + (i * 16 + li) * L::kRow + c * 2) = o;
    }
#pragma unroll
  for (int it = 0; it < 64 * 18 / 64; ++it) {
    const int idx = it * 64 + lane, row = idx / 18, chunk = idx - row * 18;
    const bf16x8 o = *(const bf16x8*)(cst + row * L::kRow + chunk * 16);
    if (m0 + row < M) __builtin_nontemporal_store(o, (bf16x8*)epi.run8(m0 + row, bn0 + nw + chunk * 8));
  }
#endif
}

// ---------------------------------------------------------------- split-K fix-up
// One wave's part of a tile of the split round to a workgroup (of one wave: nothing is shared, and eight times the workgroups reach
// CUs that a tile to a workgroup leaves idle): adds the part's `splits` partial accumulators in
// range order (bitwise repeatable) and runs the product kernel's epilogue on the sum.
template <int BM, int BN, int WR, int WC, typename Epi>
__global__ __launch_bounds__(64) void k_gemm_fixup(int M, int N, int tiles_m, int tiles_n, Epi epi, int splits, const float* __restrict__ partial) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  constexpr int NW = WR * WC, WTM = BM / WR, WTN = BN / WC, SLICE = 32 * WTN * 2;
  __shared__ __attribute__((aligned(256))) unsigned char smem[SLICE + TileVectors<WTN, Epi>::BYTES];
  const int total = tiles_m * tiles_n, in_round = (int)blockIdx.x / NW, wave = (int)blockIdx.x % NW;
  const int t = total / 256 * 256 + in_round;
  if (t >= total) return;
  constexpr int GM = kPatchRows;                     // the product kernel's tile order
  const int per_group = GM * tiles_n;
  const int group = t / per_group;
  const int first_m = group * GM;
  const int gsz = min(tiles_m - first_m, GM);
  const int wm0 = (first_m + (t % per_group) % gsz) * BM + wave / WC * WTM;
  const int wn0 = ((t % per_group) / gsz) * BN + wave % WC * WTN;
  if (wm0 >= M || wn0 >= N) return;
  float* const vectors = (float*)(smem + SLICE);
  TileVectors<WTN, Epi> v;
  if constexpr (Epi::kRowRuns) v.fetch(epi, threadIdx.x, wn0, N);
  f32x4 acc[WTM / 16][WTN / 16];
  add_partials<WTM / 16, WTN / 16>(acc, partial + (size_t)in_round * splits * (BM * BN), wave, splits, BM * BN);
  if constexpr (Epi::kRowRuns) v.to_lds(epi, threadIdx.x, vectors);
  wave_epilogue<WTM, WTN, SLICE>(acc, smem, vectors, epi, wm0, wn0, M, N);
#endif
}

// ---------------------------------------------------------------- MFMA kernel for products with few tiles
// A 128x128 grid of C leaves most CUs idle when there are only a few tiles, and each of
// them walks the whole K alone.  Here a workgroup owns one 32x32 tile and its NW waves split K:
// each brings 32 rows of 128 bytes of either operand (a K tile: 64 bf16 or 32 floats) into LDS of its own by
// DMA, eight rows of a whole line per load and one K tile ahead, and no wave waits for another before
// the end, where the partial tiles are added in a fixed order and four waves run the column-form
// epilogue on a quarter of the rows each.  LDS layout and fragment addresses are those of the tile kernels;
// fp32 takes four v_mfma_f32_32x32x2_f32 per pair of 16-byte chunks, instruction e contracting elements e of
// both.  K is a whole number of chunks; what lies past its end reads as zero.
// A CU's loads bound it.  Fragments straight from global memory, 32 bytes of 32 rows a load, got through 12 bytes
// a clock and CU whatever the number of waves.  bf16, us before and now: 120 x 1152 x 4096 18.0 and 8.6,
// 240 x 1152 x 4096 28.8 and 12.3, 154 x 1536 x 2048 10.8 and 5.3, 40960 x 16 x 1152 33.6 and 20.7,
// 120 x 1152 x 64 3.8 and 3.2; fp32: 120 x 1152 x 4096 43 and 22, 512 x 192 x 64 4.0 and 3.9.
template <typename T, int NW, typename Epi>
__global__ __launch_bounds__(NW * 64) void k_gemm_skinny(const T* __restrict__ A, const T* __restrict__ Wt, int M,
                                                             int N, int K, Epi epi) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  constexpr int ES = sizeof(T), BK = 128 / ES;           // elements of K per K tile
  constexpr int OPERAND = 32 * 128, STAGE = 2 * OPERAND;
  typedef typename std::conditional<sizeof(T) == 2, bf16x8, f32x4>::type vec;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const int kts = (K + BK - 1) / BK, k0 = wave * kts / NW, k1 = (wave + 1) * kts / NW;
  // rows past the end of an operand are out of the resource's range and load as zero
  const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)m0 * K), 0, (int)((unsigned)min(M - m0, 32) * (unsigned)K * ES), 0x00020000);
  const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(Wt + (size_t)n0 * K), 0, (int)((unsigned)min(N - n0, 32) * (unsigned)K * ES), 0x00020000);
  const int sl = lane & 15, row0 = (lane >> 4) * 2 + sl / 8;      // of the 8 rows of a load
  auto issue = [&](int kt, int stage) {
    unsigned char* dst = smem + (wave * 2 + stage) * STAGE;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = 8 * j + row0, kc = (sl % 8) ^ ((row >> 1) % 8);
      // past the end of K: out of range as well
      const unsigned off = kt * BK + kc * (16 / ES) < K ? (unsigned)row * (unsigned)K * ES + (unsigned)kc * 16u : 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(dst + j * 1024), 16, (int)off, kt * 128, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(dst + OPERAND + j * 1024), 16, (int)off, kt * 128, 0, 0);
    }
  };
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  const int row_off = (li >> 1) * 256 + (li & 1) * 128, x = (li >> 1) % 8;
  if (k0 < k1) issue(k0, 0);
  for (int kt = k0; kt < k1; ++kt) {
    const int stage = (kt - k0) & 1;
    if (kt + 1 < k1) {
      issue(kt + 1, stage ^ 1);                          // its reads of the round before last are in registers: multiplied
      wait_vm<8>();                                      // all but the eight loads just issued have landed
    } else {
      wait_vm<0>();
    }
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char* st = smem + (wave * 2 + stage) * STAGE + row_off;
    vec fa[4], fb[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int at = ((2 * ks + lh) ^ x) << 4;
      fa[ks] = *(const vec*)(st + at);
      fb[ks] = *(const vec*)(st + OPERAND + at);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if constexpr (sizeof(T) == 2) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks], fb[ks], acc, 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[ks][e], fb[ks][e], acc, 0, 0, 0);
      }
    }
    wait_lgkm0();                                        // the stage is read out before a DMA may overwrite it
    __builtin_amdgcn_sched_barrier(0);
  }
  // partial tiles, each in its wave's own LDS: [16][64]
  float* part = (float*)smem;
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave * (2 * STAGE / 4) + r * 64 + lane] = acc[r];
  __syncthreads();
  if (wave >= 4) return;
  // D: lane (li, lh) holds column li, rows 8 g + 4 lh + e in register 4 g + e; wave g takes those of g
  const auto col = epi.col(n0 + li);
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int w = 0; w < NW; ++w)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += part[w * (2 * STAGE / 4) + (4 * wave + e) * 64 + lane];
  epi.store4(col, m0 + wave * 8 + lh * 4, v);
#endif
}

template <typename T, int NW, int MODE>
static hipError_t run_skinny_waves(const T* A, const T* Wt, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using Epi = Epilogue<T, MODE>;
  Epi epi = Epi::make(ep, M, N);
  constexpr size_t smem = (size_t)NW * 2 * 2 * 32 * 128;
  auto kern = k_gemm_skinny<T, NW, Epi>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  kern<<<dim3(ceil_div(N, 32), ceil_div(M, 32)), NW * 64, smem, s>>>(A, Wt, M, N, K, epi);
  return hipGetLastError();
}

// Eight waves fill a CU's LDS: for as many tiles as there are CUs.  Above that four, two workgroups to a CU.
constexpr int kSkinnyMaxK = 1 << 22;                     // 32 rows within a buffer resource's 31-bit range
template <typename T, int MODE>
static hipError_t run_skinny(const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  if ((long long)ceil_div(N, 32) * ceil_div(M, 32) <= 256)
    return run_skinny_waves<T, 8, MODE>((const T*)A, (const T*)Wt, M, N, K, ep, s);
  return run_skinny_waves<T, 4, MODE>((const T*)A, (const T*)Wt, M, N, K, ep, s);
}

// ---------------------------------------------------------------- fp32 on the fp32 matrix cores
// v_mfma_f32_32x32x2_f32: exact fp32 products and sums at 256 FLOP per clock and CU.  For products that are at most one
// 64x64 tile to a CU, and without split weights some of one 64x128 tile (the dispatch): a slice of K is over sooner here than in the
// kernel below, which is built for throughput (216 tiles of 500 x 1728 x 576: 16 us against 19).  Operand
// lane (i, h) supplies row i, k = h, so four instructions consume one 16-byte chunk per lane (4
// floats of K; instruction e contracts elements e of both halves' chunks): tiles, LDS layout,
// DMA and fragment addressing are those of the bf16 kernels with 32 floats of K in a 128-byte
// row.  Plain double buffering, no pinned schedule, one 32x32 accumulator per wave, and the column-form epilogue
// (a wave-store covers 32 consecutive floats of a row).
// K need only be a whole number of chunks: past its end a lane's offset is moved out of the buffer
// resource's range, which loads zero, as do rows past the end of an operand.
template <int BM, int BN, int WR, int WC, typename Epi>
__global__ __launch_bounds__(WR * WC * 64) void k_gemm_f32(const float* __restrict__ A, const float* __restrict__ Wt, int M,
                                                          int N, int K, int tiles_m, int tiles_n, Epi epi) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  constexpr int NW = WR * WC, BK = 32;
  constexpr int WTM = BM / WR, WTN = BN / WC, TM = WTM / 32, TN = WTN / 32;
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;      // wave-loads (8 rows, 1 KB) per wave and K tile
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && NW % 2 == 0 && BM % 16 == 0, "loads must divide among waves");
  constexpr int STAGE_BYTES = (BM + BN) * 128, B_REGION = BM * 128;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE_BYTES];

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = wave / WC, wc = wave % WC;
  const int li = lane & 31, lh = lane >> 5;
  // workgroup -> tile as in k_gemm_dlds
  const int t = tile_index(blockIdx.x, tiles_m * tiles_n);
  if (t >= tiles_m * tiles_n) return;
  constexpr int gm = kPatchRows;
  const int per_group = gm * tiles_n, group = t / per_group, first_m = group * gm, gsz = min(tiles_m - first_m, gm);
  const int bm0 = (first_m + (t % per_group) % gsz) * BM, bn0 = ((t % per_group) / gsz) * BN;

  const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)bm0 * K), 0, (int)((unsigned)min(M - bm0, BM) * (unsigned)K * 4u), 0x00020000);
  const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(Wt + (size_t)bn0 * K), 0, (int)((unsigned)min(N - bn0, BN) * (unsigned)K * 4u), 0x00020000);
  const int line_in = lane >> 4, sl = lane & 15;
  const int row0 = wave * 8 + line_in * 2 + sl / 8, kc = (sl % 8) ^ ((wave * 4 + line_in) % 8);
  const int chunks = K / 4;
  auto issue = [&](int kt, int stage) {
    const bool in = kt * 8 + kc < chunks;
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const unsigned off = (unsigned)(row0 + NW * 8 * j) * (unsigned)K * 4u + (unsigned)kc * 16u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(smem + stage * STAGE_BYTES + (wave + NW * j) * 1024), 16,
                                               (int)(in ? off : 0x80000000u), kt * (BK * 4), 0, 0);
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const unsigned off = (unsigned)(row0 + NW * 8 * j) * (unsigned)K * 4u + (unsigned)kc * 16u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(smem + stage * STAGE_BYTES + B_REGION + (wave + NW * j) * 1024), 16,
                                               (int)(in ? off : 0x80000000u), kt * (BK * 4), 0, 0);
    }
  };
  const int rowa = wr * WTM + li, rowb = wc * WTN + li;
  const int a_off = (rowa / 2) * 256 + (rowa % 2) * 128, a_x = (rowa / 2) % 8;
  const int b_off = B_REGION + (rowb / 2) * 256 + (rowb % 2) * 128, b_x = (rowb / 2) % 8;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  const int nkt = (K + BK - 1) / BK;
  issue(0, 0);
  for (int kt = 0; kt < nkt; ++kt) {
    // This K tile has landed and this wave's reads of the other stage are in registers, whatever the scheduler has made
    // of the multiplications that use them; after the barrier that holds for every wave, and the DMA may overwrite it.
    __builtin_amdgcn_sched_barrier(0);
    wait_vm_lgkm0<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (kt + 1 < nkt) issue(kt + 1, (kt + 1) & 1);
    const unsigned char* st = smem + (kt & 1) * STAGE_BYTES;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      f32x4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *(const f32x4*)(st + a_off + i * 4096 + (((2 * ks + lh) ^ a_x) << 4));
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = *(const f32x4*)(st + b_off + j * 4096 + (((2 * ks + lh) ^ b_x) << 4));
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const auto col = epi.col(bn0 + wc * WTN + j * 32 + li);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        epi.store4(col, bm0 + wr * WTM + i * 32 + g * 8 + lh * 4, v);
      }
  }
#endif
}

template <int BM, int BN, int WR, int WC, int MODE>
static hipError_t run_f32(const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using Epi = Epilogue<float, MODE>;
  Epi epi = Epi::make(ep, M, N);
  const int tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
  const long long grid = ((long long)tiles_m * tiles_n + 255) / 256 * 256;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  k_gemm_f32<BM, BN, WR, WC, Epi><<<(unsigned)grid, WR * WC * 64, 0, s>>>((const float*)A, (const float*)Wt, M, N, K, tiles_m, tiles_n, epi);
  return hipGetLastError();
}

// ---------------------------------------------------------------- fp32 on the bf16 matrix cores
// An fp32 value of at least 2^-110 is the sum of three bf16 values of 8 bits each (high, middle, low: exact), so an fp32 product
// is nine bf16 products that the matrix cores form exactly and add in fp32.  Six of them are taken: what is
// left out (middle x low twice, low x low) is at most 2^-23 of a product and of either sign, below what the fp32
// additions round away.  Six bf16 instructions do what eight v_mfma_f32_32x32x2_f32 of twice the length do:
// 2.7 times the rate of the fp32 matrix pipe, and with fewer roundings (six per 16 products instead of eight) the
// smaller error: 0.84 to 0.88 of that kernel's against float64, over 24 shapes with K from 256 to 4608.
//
// A value is split once, on its way from global memory (registers, one slice of 16 of K ahead) to LDS, where a row
// holds its three parts of a slice one after the other, 96 bytes: rows 24 banks apart, so that the 8 rows that a
// ds_read_b128 takes at a time do not meet.  SPLIT_W: the weights have been split already (k_split_weights, once per
// model) and come by DMA, two slices ahead, three stages.  Fragments are those of the bf16 kernels: lane (i, h) holds
// row i, k = 8h .. 8h+7.  Of a slice's instructions the splitting (7.5 per value) is spread over the matrix
// instructions; written as a block behind them it cost 10 %.
// LDS bounds the small tiles (64x128: 580 cycles of reads and writes against 384 of matrix instructions per slice),
// the power limit the large ones (1.2 PFLOP/s of bf16 products, as in the bf16 kernels).
// us, fp32 matrix pipe, weights split on the way, and before (forms of the dispatch, one box): 4096 x 3456 x 1152 292, 216, 177;
// 4096 x 4608 x 1152 370, 271, 226; 4096 x 1152 x 4608 383, 386, 312; 4096 x 1152 x 1152 103, 100, 84.
// K need only be a whole number of 16-byte chunks: past its end a lane's offset is moved out of the buffer
// resource's range, which loads zero, as do rows past the end of an operand.
//
// Below 2^-110 a value's low bits lie under bf16's smallest step (2^-133, so at most 2^-134 of it is lost), and above bf16's range
// or next to infinities and NaN the parts make inf - inf and inf * 0.  Where that could show, a wave forms its products
// again on the fp32 matrix pipe, operands straight from global memory, sums in the order of k_gemm_f32: if a sum is not finite, and
// if the tile's operands hold a nonzero value below 2^-110 (noted as they are split) and a sum is below 2^-100 of their
// largest; to a larger sum all that is lost is 2^-34 per product.  (GELU leaves values between 0 and 2^-110 of inputs around -9.6, decay
// leaves them in weights that training no longer moves: common enough to be in every tile of a large model.)
// 4096 x 3456 x 1152: 230 us in parts, 498 where every wave adds the second pass, 282 for k_gemm_f32 alone.
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
// a value's bits without the sign, and those shifted one up, less one: a zero comes out above every other value
__device__ __forceinline__ unsigned magnitude(float x) { return __builtin_bit_cast(unsigned, x) & 0x7fffffffu; }
__device__ __forceinline__ unsigned magnitude_or_top(float x) { return (__builtin_bit_cast(unsigned, x) << 1) - 1u; }
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  bf16x2 p;
  p[0] = (bf16_t)x; p[1] = (bf16_t)y;
  unsigned w = __builtin_bit_cast(unsigned, p);
  asm("" : "+v"(w));                                     // else the first half is converted once more where it is used alone
  return w;
}
__device__ __forceinline__ float bf16_lo(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_hi(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// f(A) .. f(B - 1) as compile-time constants
template <int A, int B, typename F>
__device__ __forceinline__ void unrolled(F f) {
  if constexpr (A < B) {
    f(std::integral_constant<int, A>{});
    unrolled<A + 1, B>(f);
  }
}

template <int BM, int BN, int WR, int WC, int PER_SIMD, bool SPLIT_W, typename Epi>
__global__ __launch_bounds__(WR * WC * 64, PER_SIMD) void k_gemm_f32_parts(const float* A, const float* Wt, const void* parts,
                                                                     int M, int N, int K, int tiles_m, int tiles_n, Epi epi) {
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type: the host pass sees an empty body
  constexpr int NW = WR * WC, NT = NW * 64;
  constexpr int WTM = BM / WR, WTN = BN / WC, TM = WTM / 32, TN = WTN / 32;
  constexpr int LA = BM * 4 / NT, LB = SPLIT_W ? 0 : BN * 4 / NT;      // 16-byte chunks per thread and slice to be split
  constexpr int WL = SPLIT_W ? BN * 96 / 1024 : 0, LD = (WL + NW - 1) / NW;   // wave-loads of split weights per slice, and per wave
  static_assert(BM * 4 % NT == 0 && (SPLIT_W || BN * 4 % NT == 0) && BN % 32 == 0, "loads must divide among threads");
  constexpr int ROWS = SPLIT_W ? BM : BM + BN;           // split on the way
  constexpr int STAGE = ROWS * 96, W_STAGE = BN * 96;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WC, wc = wave % WC;
  const int li = lane & 31, lh = lane >> 5;
  // workgroup -> tile as in k_gemm_dlds
  const int t = tile_index(blockIdx.x, tiles_m * tiles_n);
  if (t >= tiles_m * tiles_n) return;
  constexpr int gm = kPatchRows;
  const int per_group = gm * tiles_n, group = t / per_group, first_m = group * gm, gsz = min(tiles_m - first_m, gm);
  const int bm0 = (first_m + (t % per_group) % gsz) * BM, bn0 = ((t % per_group) / gsz) * BN;
  const int slices = (K + 15) / 16;

  const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)bm0 * K), 0, (int)((unsigned)min(M - bm0, BM) * (unsigned)K * 4u), 0x00020000);
  const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)(Wt + (size_t)bn0 * K), 0, (int)((unsigned)min(N - bn0, BN) * (unsigned)K * 4u), 0x00020000);
  // split weights: [N / 32][slices][32 rows][3 parts][16] bf16, rows past N zero, then of each 32 rows the least and the largest magnitude
  const int w_blocks = min((N + 31) / 32 - bn0 / 32, BN / 32);
  const auto rb = SPLIT_W ? __builtin_amdgcn_make_buffer_rsrc((void*)((const unsigned char*)parts + (size_t)(bn0 / 32) * slices * 3072), 0, (int)((unsigned)w_blocks * (unsigned)slices * 3072u), 0x00020000) : rw;
  constexpr unsigned kLeast = ((127u - 110u) << 24) - 1u;              // magnitude_or_top(2^-110)
  unsigned least = ~0u, most = 0;                        // magnitude_or_top and magnitude of the operands' values, this thread's share
  if constexpr (SPLIT_W) {
    const unsigned* ranges = (const unsigned*)((const unsigned char*)parts + (size_t)((N + 31) / 32) * slices * 3072) + bn0 / 32 * 2;
    for (int x = 0; x < w_blocks; ++x) { least = min(least, ranges[2 * x]); most = max(most, ranges[2 * x + 1]); }
  }
  // chunk tid + NT j of a slice: row (tid >> 2) + NT / 4 j, floats 4c .. 4c+3
  const int row0 = tid >> 2, c = tid & 3;
  f32x4 raw[2][LA + LB];                                 // of the next slice and of the one behind it
  auto fetch = [&](f32x4 (&raw)[LA + LB], int j, int ks) {
    const unsigned off = (unsigned)(row0 + NT / 4 * (j < LA ? j : j - LA)) * (unsigned)K * 4u + (unsigned)c * 16u;
    raw[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(j < LA ? ra : rb, (int)(ks * 16 + c * 4 < K ? off : 0x80000000u), ks * 64, 0));
  };
  // split weights go to LDS as they lie: 1 KB a wave-load, three to a block of 32 rows; wave-load wave + NW j.  A wave for which
  // there is no such one loads its first once more: all have the same number on their way, and no branch parts them.
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  int w_load[LD > 0 ? LD : 1], w_off[LD > 0 ? LD : 1];
#pragma unroll
  for (int j = 0; j < LD; ++j) {
    w_load[j] = wave_u + NW * j < WL ? wave_u + NW * j : wave_u;
    w_off[j] = w_load[j] / 3 * slices * 3072 + w_load[j] % 3 * 1024 + lane * 16;
  }
  auto request = [&](int at, int stage) {
    const int ks = min(at, slices - 1);                  // the scalar offset is not range-checked: past the end the last slice again
#pragma unroll
    for (int j = 0; j < LD; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(smem + 2 * STAGE + stage * W_STAGE + w_load[j] * 1024), 16, w_off[j], ks * 3072, 0, 0);
  };
  auto put = [&](int j, int stage, u32x2 h, u32x2 m, u32x2 l) {
    const int row = j < LA ? row0 + NT / 4 * j : BM + row0 + NT / 4 * (j - LA);
    unsigned char* dst = smem + stage * STAGE + row * 96 + c * 8;
    *(u32x2*)dst = h;
    *(u32x2*)(dst + 32) = m;
    *(u32x2*)(dst + 64) = l;
  };
  // Step X of the splitting of slice ks: chunk X / 6, a pair of its values after the other in steps of 7, 5 and 5 vector
  // instructions; behind the last the chunk is fetched for slice ks + 2.
  float a0 = 0.0f, a1 = 0.0f;                            // what is left of the pair
  unsigned h0 = 0, m0 = 0, l0 = 0, h1 = 0, m1 = 0;
  auto split_step = [&](auto step, auto par, int ks) {
    constexpr int P = decltype(par)::value;                // ks & 1
    constexpr int X = decltype(step)::value, j = X / 6, half = X % 6 / 3;
    if constexpr (X % 3 == 0) {
      a0 = raw[P][j][2 * half]; a1 = raw[P][j][2 * half + 1];
      least = min(least, min(magnitude_or_top(a0), magnitude_or_top(a1)));
      most = max(most, max(magnitude(a0), magnitude(a1)));
      (half ? h1 : h0) = pack_bf16(a0, a1);
    } else if constexpr (X % 3 == 1) {
      const unsigned h = half ? h1 : h0;
      a0 -= bf16_lo(h); a1 -= bf16_hi(h);
      (half ? m1 : m0) = pack_bf16(a0, a1);
    } else {
      const unsigned m = half ? m1 : m0, l = pack_bf16(a0 - bf16_lo(m), a1 - bf16_hi(m));
      if constexpr (half == 0) {
        l0 = l;
      } else {
        put(j, P, u32x2{h0, h1}, u32x2{m0, m1}, u32x2{l0, l});
        fetch(raw[P], j, ks + 2);
      }
    }
  };
  constexpr int STEPS = 6 * (LA + LB), NM = 6 * TM * TN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  const int a_off = (wr * WTM + li) * 96 + lh * 16, b_off = ((SPLIT_W ? 0 : BM) + wc * WTN + li) * 96 + lh * 16;
  using P0 = std::integral_constant<int, 0>; using P1 = std::integral_constant<int, 1>;
  request(0, 0);
  request(1, 1);
#pragma unroll
  for (int j = 0; j < LA + LB; ++j) fetch(raw[0], j, 0);
#pragma unroll
  for (int j = 0; j < LA + LB; ++j) fetch(raw[1], j, 1);
  // Everything has landed, the weights of slice 1 too: behind those come fewer loads than the count at the end of a slice
  // leaves on their way (one round of fetches and one of weights, against two and one in every later slice).
  wait_vm<0>();
  unrolled<0, STEPS>([&](auto x) { split_step(x, P0{}, 0); });
  __builtin_amdgcn_sched_barrier(0);
  int w_stage = 0;                                       // of three
  wait_vm_lgkm0<2 * (LA + LB) + LD>();                   // the values just split are in LDS
  __builtin_amdgcn_s_barrier();
  // One slice.  Past the last one zeros are fetched and split, and weights requested that nothing reads: no branch parts
  // the vector instructions from the matrix ones, and the number of loads in flight is the same throughout.
  auto slice = [&](auto par, int ks) {
    constexpr int P = decltype(par)::value;
    __builtin_amdgcn_sched_barrier(0);
    request(ks + 2, w_stage == 0 ? 2 : w_stage - 1);     // the stage read a slice ago
    const unsigned char* sa = smem + P * STAGE;
    const unsigned char* sb = SPLIT_W ? smem + 2 * STAGE + w_stage * W_STAGE : sa;
    w_stage = w_stage == 2 ? 0 : w_stage + 1;
    bf16x8 fa[3][TM], fb[3][TN];
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};   // smallest products first
    constexpr int RA[3] = {2, 0, 1}, RB[3] = {0, 2, 1};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[RA[p]][i] = *(const bf16x8*)(sa + RA[p] * 32 + a_off + i * 3072);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[RB[p]][j] = *(const bf16x8*)(sb + RB[p] * 32 + b_off + j * 3072);
    }
    // The next slice's splitting, a few steps behind each matrix instruction, into the stage last read a slice ago.
    unrolled<0, NM>([&](auto at) {
      constexpr int R = decltype(at)::value, x = R / (TM * TN), i = R / TN % TM, j = R % TN;
      __builtin_amdgcn_sched_barrier(0);
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[x]][i], fb[PB[x]][j], acc[i][j], 0, 0, 0);
      unrolled<R * STEPS / NM, (R + 1) * STEPS / NM>([&](auto y) { split_step(y, std::integral_constant<int, P ^ 1>{}, ks + 1); });
    });
    counted_wait_lgkm0<2 * (LA + LB) + LD>();            // the next slice's weights have landed, those behind them may be on their way
    __builtin_amdgcn_s_barrier();
  };
  int ks = 0;
  for (; ks + 1 < slices; ks += 2) {                     // whole pairs: a way round the second slice would have the first one of the next wait for more
    slice(P0{}, ks);
    slice(P1{}, ks + 1);
  }
  if (ks < slices) slice(P0{}, ks);
  wait_vm<0>();                                          // nothing is on its way to LDS when the workgroup ends
  // The stages of split values are read out and nothing is written to them any more.
  unsigned* const of_waves = (unsigned*)smem;
  if (lane == 0) of_waves[wave] = 0;
  if (__any(least < kLeast) && lane == 0) of_waves[wave] = 1;
  __syncthreads();
  unsigned small = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) small |= of_waves[w];
  float finite = 0.0f;                                   // NaN behind a sum that is not
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) finite = __builtin_fmaf(acc[i][j][r], 0.0f, finite);
  bool again = finite != 0.0f;
  if (small) {                                           // the same in all waves
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) most = max(most, (unsigned)__shfl_xor((int)most, m, 64));
    if (lane == 0) of_waves[NW + wave] = most;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) most = max(most, of_waves[NW + w]);
    const float bar = __builtin_fmaxf(__builtin_bit_cast(float, min(most, 0x7f800000u)) * 0x1p-100f, 0x1p-110f);
    float low = bar;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool in = bm0 + wr * WTM + i * 32 + r / 4 * 8 + lh * 4 + r % 4 < M && bn0 + wc * WTN + j * 32 + li < N;
          low = in ? __builtin_fminf(low, __builtin_fabsf(acc[i][j][r])) : low;
        }
    again |= low < bar;
  }
  if (__any(again)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // lane (i, h) holds floats 4h .. 4h + 3 of eight of a row; instruction e contracts elements e of both halves (as k_gemm_f32)
    const unsigned at_a = (unsigned)(wr * WTM + li) * (unsigned)K * 4u + lh * 16, at_w = (unsigned)(wc * WTN + li) * (unsigned)K * 4u + lh * 16;
    f32x4 fa[2][TM], fw[2][TN];
    auto load = [&](int p, int k) {                      // past the end zeros
      const bool in = k + 4 * lh < K;
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[p][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(in ? at_a + (unsigned)(i * 32) * (unsigned)K * 4u : 0x80000000u), k * 4, 0));
#pragma unroll
      for (int j = 0; j < TN; ++j) fw[p][j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(in ? at_w + (unsigned)(j * 32) * (unsigned)K * 4u : 0x80000000u), k * 4, 0));
    };
    auto multiply = [&](int p) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[p][i][e], fw[p][j][e], acc[i][j], 0, 0, 0);
    };
    constexpr bool AHEAD = TM * TN < 8;                  // registers for a second set of fragments
    if constexpr (AHEAD) load(0, 0);
#pragma unroll 1
    for (int k = 0; k < K; k += 16) {
      if constexpr (AHEAD) load(1, k + 8); else load(0, k);
      multiply(0);
      load(0, AHEAD ? k + 16 : k + 8);
      multiply(AHEAD ? 1 : 0);
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const auto col = epi.col(bn0 + wc * WTN + j * 32 + li);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        epi.store4(col, bm0 + wr * WTM + i * 32 + g * 8 + lh * 4, v);
      }
  }
#endif
}

// Split weights of a product, as k_gemm_f32_parts reads them: [N / 32][slices of 16][32 rows][3 parts][16] bf16, zero
// past N and K.  Once per model.
__global__ __launch_bounds__(256) void k_split_weights(const float* __restrict__ Wt, unsigned char* __restrict__ out, int N, int K, int slices) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;       // a row's slice
  const int row = (int)(i / slices), ks = (int)(i % slices);
  if (row >= (N + 31) / 32 * 32) return;
  unsigned h[8], m[8], l[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int k = ks * 16 + 2 * x;
    const float a = row < N && k < K ? Wt[(size_t)row * K + k] : 0.0f, b = row < N && k + 1 < K ? Wt[(size_t)row * K + k + 1] : 0.0f;
    h[x] = pack_bf16(a, b);
    m[x] = pack_bf16(a - bf16_lo(h[x]), b - bf16_hi(h[x]));
    l[x] = pack_bf16((a - bf16_lo(h[x])) - bf16_lo(m[x]), (b - bf16_hi(h[x])) - bf16_hi(m[x]));
  }
  unsigned* dst = (unsigned*)(out + ((size_t)(row / 32) * slices + ks) * 3072 + (row % 32) * 96);
#pragma unroll
  for (int x = 0; x < 8; ++x) { dst[x] = h[x]; dst[8 + x] = m[x]; dst[16 + x] = l[x]; }
}

// Least (magnitude_or_top) and largest magnitude of each 32 rows, behind the parts.
__global__ __launch_bounds__(256) void k_split_ranges(const float* __restrict__ Wt, unsigned* __restrict__ out, int N, int K) {
  const int row0 = blockIdx.x * 32, rows = min(N - row0, 32);
  unsigned least = ~0u, most = 0;
  for (long long i = threadIdx.x; i < (long long)rows * K; i += 256) {
    const float w = Wt[(size_t)row0 * K + i];
    least = min(least, magnitude_or_top(w));
    most = max(most, magnitude(w));
  }
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    least = min(least, (unsigned)__shfl_xor((int)least, m, 64));
    most = max(most, (unsigned)__shfl_xor((int)most, m, 64));
  }
  __shared__ unsigned waves[4][2];
  if ((threadIdx.x & 63) == 0) { waves[threadIdx.x >> 6][0] = least; waves[threadIdx.x >> 6][1] = most; }
  __syncthreads();
  if (threadIdx.x != 0) return;
  out[2 * blockIdx.x] = min(min(waves[0][0], waves[1][0]), min(waves[2][0], waves[3][0]));
  out[2 * blockIdx.x + 1] = max(max(waves[0][1], waves[1][1]), max(waves[2][1], waves[3][1]));
}

size_t split_weights_bytes(int N, int K) { return (size_t)((N + 31) / 32) * (((K + 15) / 16) * (size_t)3072 + 8); }
hipError_t launch_split_weights(const float* Wt, void* out, int N, int K, hipStream_t s) {
  const int slices = (K + 15) / 16;
  const long long blocks = ((long long)(N + 31) / 32 * 32 * slices + 255) / 256;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  k_split_weights<<<(unsigned)blocks, 256, 0, s>>>(Wt, (unsigned char*)out, N, K, slices);
  k_split_ranges<<<(N + 31) / 32, 256, 0, s>>>(Wt, (unsigned*)((unsigned char*)out + (size_t)((N + 31) / 32) * slices * 3072), N, K);
  return hipGetLastError();
}

template <int BM, int BN, int WR, int WC, int PER_SIMD, bool SPLIT_W, int MODE>
static hipError_t run_f32_parts(const void* A, const void* Wt, const void* parts, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using Epi = Epilogue<float, MODE>;
  Epi epi = Epi::make(ep, M, N);
  const int tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
  const long long grid = ((long long)tiles_m * tiles_n + 255) / 256 * 256;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  constexpr size_t smem = (size_t)(SPLIT_W ? 2 * BM + 3 * BN : 2 * (BM + BN)) * 96;
  auto kern = k_gemm_f32_parts<BM, BN, WR, WC, PER_SIMD, SPLIT_W, Epi>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  kern<<<(unsigned)grid, WR * WC * 64, smem, s>>>((const float*)A, (const float*)Wt, parts, M, N, K, tiles_m, tiles_n, epi);
  return hipGetLastError();
}

// ---------------------------------------------------------------- plain kernel (any T, any shape)
// 64x64 block tile, BK = 16, 256 threads each owning a 4(row) x 4(col) micro-tile.
template <typename T, typename Epi>
__global__ __launch_bounds__(256) void k_gemm_plain(const T* __restrict__ A, const T* __restrict__ Wt, int M, int N,
                                                    int K, Epi epi) {
  __shared__ float As[16][64 + 4];
  __shared__ float Bs[16][64 + 4];
  const int tid = threadIdx.x;
  const int tr = tid / 16, tc = tid % 16;
  const int bm0 = blockIdx.y * 64, bn0 = blockIdx.x * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int i = tid; i < 64 * 16; i += 256) {
      int row = i / 16, kk = i % 16;
      int gm = bm0 + row, gn = bn0 + row, gk = k0 + kk;
      As[kk][row] = (gm < M && gk < K) ? to_f32(A[(size_t)gm * K + gk]) : 0.0f;
      Bs[kk][row] = (gn < N && gk < K) ? to_f32(Wt[(size_t)gn * K + gk]) : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][tr * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tc * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v[4] = {acc[0][j], acc[1][j], acc[2][j], acc[3][j]};
    epi.store4(epi.col(bn0 + tc * 4 + j), bm0 + tr * 4, v);
  }
}

// ---------------------------------------------------------------- dispatch
// Ranges of K that the tiles of a last round are split into, 1: none (run_dlds says when).
template <int BM, int BN>
static int split_ranges(long long total, long long slots, int K, const void* scratch, size_t scratch_bytes) {
  const long long rem = total % 256, full = total - rem;
  if (total / 256 > 8 || rem == 0 || rem > slots / 2 || (slots != 256 && full != 0) || !scratch || ((uintptr_t)scratch & 15) != 0) return 1;
  long long sp = slots / rem;
  sp = sp > 4 ? 4 : sp;
  sp = sp > K / (64 * kUnitKTiles) ? K / (64 * kUnitKTiles) : sp;
  if (sp < 2 || (long long)K * (sp - 1) / sp < 1536 || (size_t)(rem * sp) * BM * BN * sizeof(float) > scratch_bytes) return 1;
  return (int)sp;
}

template <int BM, int BN, int WR, int WC, int MODE>
static hipError_t run_dlds(const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep, void* scratch,
                           size_t scratch_bytes, hipStream_t s) {
  using Epi = Epilogue<bf16_t, MODE>;
  Epi epi = Epi::make(ep, M, N);
  constexpr size_t smem = DldsStages<BM, BN, WR * WC>::BYTES;
  auto kern = k_gemm_dlds<BM, BN, WR, WC, Epi>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
  const long long total = (long long)tiles_m * tiles_n;
  // persistent: as many workgroups as the chip holds at once (by LDS: one of the large
  // configurations per CU, two of the 128x128 one), each walking its share of the tiles
  const long long padded = (total + 255) / 256 * 256;
  const long long slots = 256LL * (smem > 80 * 1024 ? 1 : 2);
  const unsigned grid = (unsigned)(padded < slots ? padded : slots);
  // Split-K for a last round that would leave most of the chip idle: at most half the slots
  // taken, few enough rounds that one of them matters (measured: 3.3 rounds become 11 %
  // faster, 13.1 rounds not at all), a K long enough that the saved part of a tile outweighs
  // the fix-up launch, and a caller that lends scratch memory for the partial tiles.
  unsigned launch = grid;
  const long long rem = total % 256, full = total - rem;
  // (A product of fewer tiles than half the slots is all remainder: its tiles are split the
  // same way; with two workgroups per CU there are 512 slots for the units.)
  // (With two workgroups per CU every product of up to 512 tiles runs in one round anyway: only
  // the all-remainder case is split there.)
  const int splits = split_ranges<BM, BN>(total, slots, K, scratch, scratch_bytes);
  if (splits >= 2) {
    const long long units = (full + rem * splits + 7) / 8 * 8;
    launch = (unsigned)(units < slots ? units : slots);
    if (launch < grid) launch = grid;
  }
  kern<<<launch, WR * WC * 64, smem, s>>>((const bf16_t*)A, (const bf16_t*)Wt, M, N, K, tiles_m, tiles_n, epi, splits, (float*)scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits < 2) return e;
  k_gemm_fixup<BM, BN, WR, WC, Epi><<<(unsigned)rem * WR * WC, 64, 0, s>>>(M, N, tiles_m, tiles_n, epi, splits, (const float*)scratch);
  return hipGetLastError();
}

template <int BM, int BN, int PER_CU, int MODE>
static hipError_t run_packed(const void* A, const void* Wp, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using Epi = Epilogue<bf16_t, MODE>;
  Epi epi = Epi::make(ep, M, N);
  constexpr size_t smem = (size_t)2 * BM * 128 + BN * 8;   // two stages of A, bias and gate of a tile
  auto kern = k_gemm_packed<BM, BN, Epi>;
  const int tiles_m = ceil_div(M, BM), tiles_n = ceil_div(N, BN);
  const long long padded = ((long long)tiles_m * tiles_n + 255) / 256 * 256;
  const unsigned grid = (unsigned)(padded < 256LL * PER_CU ? padded : 256LL * PER_CU);   // persistent, as in run_dlds
  kern<<<grid, 256, smem, s>>>((const bf16_t*)A, Wp, M, N, K, tiles_m, tiles_n, epi);
  return hipGetLastError();
}

template <int MODE>
static hipError_t run_288(const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using Epi = Epilogue<bf16_t, MODE>;
  using L = Tile288;
  Epi epi = Epi::make(ep, M, N);
  auto kern = k_gemm_288<Epi>;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, L::kBytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int tiles_m = ceil_div(M, L::BM), tiles_n = N / L::BN;
  kern<<<round_up((size_t)tiles_m * tiles_n, 256), 256, L::kBytes, s>>>((const bf16_t*)A, (const bf16_t*)Wt, M, N, K, tiles_m, tiles_n, epi);
  return hipGetLastError();
}

template <typename T, int MODE>
static hipError_t run_plain(const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using Epi = Epilogue<T, MODE>;
  Epi epi = Epi::make(ep, M, N);
  dim3 grid(ceil_div(N, 64), ceil_div(M, 64));
  k_gemm_plain<T, Epi><<<grid, 256, 0, s>>>((const T*)A, (const T*)Wt, M, N, K, epi);
  return hipGetLastError();
}

// fp32 products.  The plain kernel keeps what is not made of whole aligned 16-byte chunks.
template <int MODE>
static hipError_t dispatch_f32(const void* A, const void* Wt, const void* w_parts, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  if (K % 4 != 0 || (((uintptr_t)A | (uintptr_t)Wt) & 15) != 0 || K >= kSkinnyMaxK) return run_plain<float, MODE>(A, Wt, M, N, K, ep, s);
  // Few tiles: one 32x32 tile per workgroup, K split over its waves (500 x 512 x 512: 8.6 us
  // against 13.6 with 64x64 tiles; at 192 of those, 500 x 1536 x 512, 18 against 14).
  const long long t64 = (long long)ceil_div(M, 64) * ceil_div(N, 64);
  if ((t64 <= 128 || N < 32) && ceil_div(M, 32) <= 65535) return run_skinny<float, MODE>(A, Wt, M, N, K, ep, s);
  if (t64 <= 256) return run_f32<64, 64, 2, 2, MODE>(A, Wt, M, N, K, ep, s);
  // The CU that gets the most tiles bounds the launch: rounds of 256 tiles times what a tile takes per slice of K, in
  // tenths of a microsecond, measured where several tiles share a CU and (second figure) where one has it to itself.
  auto estimate = [&](int bm, int bn, double shared, double alone) {
    const long long rounds = ((long long)ceil_div(M, bm) * ceil_div(N, bn) + 255) / 256;
    return rounds == 1 ? alone : rounds * shared;
  };
  if constexpr (MODE == EPI_HEADS || MODE == EPI_GATE || MODE == EPI_GELU) {           // a model's products over token rows
    if (w_parts && K < (1 << 18)) {                      // (K: 32-bit offsets into the split weights)
      const double e64 = estimate(64, 64, 2.3, 4.2), e128 = estimate(64, 128, 3.7, 5.0), e192 = estimate(128, 192, 9.9, 12.0),
                   e256 = estimate(256, 256, 22.0, 23.0);
      if (e256 < e192 && e256 < e128 && e256 < e64) return run_f32_parts<256, 256, 4, 2, 2, true, MODE>(A, Wt, w_parts, M, N, K, ep, s);
      if (e192 < e128 && e192 < e64) return run_f32_parts<128, 192, 2, 2, 2, true, MODE>(A, Wt, w_parts, M, N, K, ep, s);
      if (e64 < e128) return run_f32_parts<64, 64, 2, 2, 4, true, MODE>(A, Wt, w_parts, M, N, K, ep, s);
      return run_f32_parts<64, 128, 2, 2, 4, true, MODE>(A, Wt, w_parts, M, N, K, ep, s);
    }
  }
  // Both operands split on the way.  Where 64x128 tiles of the fp32 pipe make one round and there are more than 330 of 64x64, those are
  // over first (1274 x 1536 x 512: 24.1 us against 25.9, 2000 x 1024 x 4096 164 and 169; below that 712 x 1536 x 512 23.3 and 21.7,
  // 1167 x 1024 x 1024 43.4 and 40.5).
  if (t64 > 330 && (long long)ceil_div(M, 64) * ceil_div(N, 128) <= 256) return run_f32<64, 128, 2, 4, MODE>(A, Wt, M, N, K, ep, s);
  if (estimate(128, 128, 7.0, 9.0) < estimate(64, 64, 2.4, 4.7)) return run_f32_parts<128, 128, 2, 2, 2, false, MODE>(A, Wt, nullptr, M, N, K, ep, s);
  return run_f32_parts<64, 64, 2, 2, 4, false, MODE>(A, Wt, nullptr, M, N, K, ep, s);
}

// K that the tiles take: the rows of one lie within 32-bit offsets, up to kTileMaxK those of all tiles (384 of them), up to kNarrowMaxK those of 128x128
// ones.  320 x 320 x 4 194 368: 67 ms, in the plain kernel 565.
constexpr int kTileMaxK = 1 << 22, kNarrowMaxK = 1 << 24;
// The tile of a product of k_gemm_dlds.
static Bf16Form bf16_tile(bool unpatch, int M, int N, int K) {
  if (K < 64 * kUnitKTiles || K >= kTileMaxK) return F128;           // (128x128 tiles have two stages)
  // Tile choice.  256x256 (8 waves, one workgroup per CU) has the best operand reuse but
  // needs several rounds of tiles per CU and wastes the ragged part of N; 256x192 takes
  // over where N is a multiple of 192 that 256 would pad by more than 5 % (N = 1152:
  // 11 % padding and 2.5 rounds of tiles become none and 3); 128x128 (4 waves, two
  // workgroups per CU, so one's epilogue overlaps the other's main loop) wins for
  // narrow or short-K products.  Thresholds from timings of the workload shapes.
  const long long tiles256 = (long long)ceil_div(M, 256) * ceil_div(N, 256);
  const double waste = (double)ceil_div(N, 256) * 256.0 / N - 1.0;
  auto fill = [](long long t) { return (double)t / (double)((t + 255) / 256 * 256); };
  // 384x192 (96x96 per wave) is no faster per tile than 256x256, but where its tile count fills
  // whole rounds of 256 and that of 256x256 does not, it saves most of a round (the full-3D
  // out-projection and fc2: 752 tiles = 2.94 rounds against 840 = 3.28; 2-5 % over the split
  // last round)
  if (N % 192 == 0 && waste > 0.05 && (long long)ceil_div(M, 256) * (N / 192) >= 192) return F192;
  if (!unpatch && N % 192 == 0 && K >= 2048 && tiles256 >= 600 && waste <= 0.05 &&
           fill((long long)ceil_div(M, 384) * (N / 192)) >= 0.95 && fill(tiles256) < 0.85) return F384;
  if (tiles256 >= 600 && (waste <= 0.05 || K >= 2048)) return F256;
  // Mid-size products (a few thousand rows) that the thresholds above leave to 128x128: the large
  // tiles still win where their tile count fills its rounds of 256 workgroups (measured at
  // M = 4096 and 8192: QKV of the 1152-wide model 8-14 % faster with 256x256, its fc1 at
  // M = 8192 7 % faster with 256x192; where the last round would be mostly empty, 128x128 stays)
  if (tiles256 >= 200 && waste <= 0.05 && fill(tiles256) >= 0.85) return F256;
  if (N % 192 == 0 && (long long)ceil_div(M, 256) * (N / 192) >= 200 && fill((long long)ceil_div(M, 256) * (N / 192)) >= 0.95) return F192;
  return F128;
}

// The form of a model's product without packed weights: the tile just chosen, or one whose estimated time is below that tile's.  The
// estimates, in us: tiles of the fullest CU times a time per K tile and one per tile, fitted over 325 products (M 256 to 38 000, N and K 576 to
// 12 288, the same product again and again) with 32x32x16 instructions; for the tiles of 288 columns also the tiles per CU of the whole
// chip (the power limit), over 400 products.  They rank forms that differ by whole rounds: 978 products of ten widths from 576 to 3072 and 25
// numbers of rows take 1.04 of their best staged form's time in the mean, 1.026 in the sum (1.57 where a product of 128x128 tiles would be best in
// 256x192: 13113 x 768 x 3072 99 us, 61).
//   128x288, 384x192: where the estimate is 6 % (384x192: 9 %) lower, a nearly empty last round counted as what it takes.  Their tiles
//   fill rounds that the others leave half empty (all rounds counted as full: up to 1.29 times as long, 6545 x 576 x 2304 28 us, and 36).  128x288
//   from K = 2048 on: below it is mostly first tile and epilogue, which the estimate was not held against.
static Bf16Form staged_form(int M, int N, int K, const void* scratch, size_t scratch_bytes) {
  const Bf16Form tile = bf16_tile(false, M, N, K);
  const double kt = K / 64.0;
  auto tiles = [&](int bm, int bn) { return (long long)ceil_div(M, bm) * ceil_div(N, bn); };
  auto per_cu = [&](int bm, int bn) { return (double)((tiles(bm, bn) + 255) / 256); };
  auto rounds = [&](int bm, int bn, int sp, double start, double k, double fixed) {
    if (sp < 2) return start + per_cu(bm, bn) * (k * kt + fixed);
    const double full = (double)(tiles(bm, bn) / 256);
    return start + full * (k * kt + fixed) + (k * kt / sp + fixed) + 14.0;
  };
  auto lone = [&](double k, double fixed) { return per_cu(128, 128) == 1.0 ? k * kt + fixed : 0.0; };
  const double e384 = rounds(384, 192, split_ranges<384, 192>(tiles(384, 192), 256, K, scratch, scratch_bytes), -0.74, 1.386, 11.56);
  const int splits256 = split_ranges<256, 256>(tiles(256, 256), 256, K, scratch, scratch_bytes);
  Bf16Form form = tile;
  double now = 0.0;
  switch (tile) {
    case F256: now = rounds(256, 256, splits256, -1.75, 1.266, 8.84); break;
    case F192: now = rounds(256, 192, split_ranges<256, 192>(tiles(256, 192), 256, K, scratch, scratch_bytes), 0.04, 1.051, 6.49); break;
    case F384: now = e384; break;
    default:
      if (split_ranges<128, 128>(tiles(128, 128), 512, K, scratch, scratch_bytes) >= 2) return F128;
      now = rounds(128, 128, 1, 1.84, 0.443, 1.40) + lone(0.21, -0.72);
      break;
  }
  if ((unsigned long long)M * K * 2 >= (1ull << 32) || (unsigned long long)N * K * 2 >= (1ull << 32)) return form;     // 128x288: 32-bit offsets
  // What a nearly empty last round takes less than the others: 128x128 tiles, two to a CU, and 256x256 tiles where it is less than a
  // quarter full (for the former: and the second that CUs share).
  auto empty = [&](int bm, int bn) { return per_cu(bm, bn) - tiles(bm, bn) / 256.0; };
  if (form == F128 && empty(128, 128) > 0.75 && (long long)per_cu(128, 128) % 2 == 0) now -= 0.5 * empty(128, 128) * (0.443 * kt + 1.40);
  else if (form == F256 && empty(256, 256) > 0.75 && splits256 < 2) now -= 0.15 * empty(256, 256) * (1.266 * kt + 8.84);
  double least = 0.94 * now;
  if (N % 288 == 0 && K >= 2048) {
    const double e = 2.53 + per_cu(128, 288) * (0.629 * kt + 5.71) + tiles(128, 288) / 256.0 * 0.234 * kt;
    if (e < least) { form = W288; least = e; }
  }
  if (N % 192 == 0 && e384 < 0.97 * least) form = F384;
  return form;
}

// What the forms take, in us: start + c (k kt + fixed) + tiles / 256 chip kt, kt K tiles, c tiles on the fullest CU (chip: what all CUs share, the
// power limit and the memory); a CU's only tile takes lone + lone_k kt more (fewer waves hide its latencies), a last round in ranges of K
// only its part and the fix-up.  Fitted over 978 products of ten widths from 576 to 3072 and 25 numbers of rows from 300 to 40 960, each in every form,
// operands by turns from four products; those where the form is within 15 % of the best count five times (rms of these 3 to 6 %).
struct FormTime { int bm, bn; double start, k, fixed, chip, lone, lone_k, fixup; };
static constexpr FormTime kF128{128, 128, 0.756, 0.318, 1.629, 0.157, 2.003, 0.219, 5.000}, kF192{256, 192, 0.000, 0.732, 5.514, 0.434, 0.847, 0.018, 10.757},
    kF256{256, 256, 0.000, 0.889, 6.654, 0.571, 0.279, 0.022, 10.808}, kF384{384, 192, 0.000, 1.051, 7.722, 0.610, 0.109, 0.044, 12.090},
    kP128{128, 128, 1.825, 0.322, 1.058, 0.111, 1.387, 0.104, 0.000}, kP192{128, 192, 1.506, 0.408, 2.042, 0.189, 2.027, 0.008, 0.000},
    kP256{128, 256, 1.302, 0.405, 2.376, 0.342, 1.481, 0.027, 0.000}, kW288{128, 288, 1.483, 0.515, 6.489, 0.365, 0.644, -0.038, 0.000};
static double form_time(const FormTime& f, int M, int N, int K, int splits = 1) {
  const long long tiles = (long long)ceil_div(M, f.bm) * ceil_div(N, f.bn);
  const double kt = K / 64.0, chip = f.start + tiles / 256.0 * f.chip * kt;
  if (splits >= 2) {
    const double full = (double)(tiles / 256);
    return chip + full * (f.k * kt + f.fixed) + f.k * kt / splits + f.fixed + f.fixup;
  }
  const double c = (double)((tiles + 255) / 256);
  return chip + c * (f.k * kt + f.fixed) + (c == 1.0 ? f.lone + f.lone_k * kt : 0.0);
}
// Packed tiles of 128x128 or 128x192 (P128): 192 columns where their estimate is the lower one, three of them for four rounds of the
// others.  us, 128x128 and 128x192: 4096 x 1152 x 1152 17.0, 14.6; 4096 x 4608 x 1152 44.3, 40.6; 8192 x 3456 x 1152 71.6, 63.4.
static bool narrow_is_192(int M, int N, int K) { return form_time(kP192, M, N, K) < form_time(kP128, M, N, K); }

// The form of a model's product; dispatch_mode launches the one named here.  With packed weights: the tile that bf16_tile gives, or packed
// ones.  Wide ones (128x256) where they are 2 % lower than 256x192 tiles, 3.2 % than larger ones or 2.5 % than a lone 256x256 tile to a CU
// (the weights are held twice for them; the three lines are drawn by one call, a full-3D step 2048 wide, that took 1.013 of its time with wide
// tiles wherever their estimate was the lower one, though three of its four products are 3 to 5 % faster in them alone; why is not known), narrow ones
// 6 % (all packed estimates are somewhat short where a product has many rounds), both wherever the tile would be 128x128; narrow ones only where wide ones
// take 3 % more (a 128x128 tile writes per-head outputs in pieces of 64 bytes, which the estimates, all epilogues alike, leave out: 4096 x 1728 x 576
// 13.3 us wide, 16.6 narrow; 128x192 tiles write pieces of 96 bytes and are kept back by the same line, also where they are faster: 8192 x 3456 x
// 1152 62 us, 66 in the form taken).  128x288 (K from 2048) where it is 6 % lower than the choice so far, 384x192 likewise;
// that is taken over narrow tiles at any lower estimate (in the mean that is level or better), and takes nothing from wide ones (66 products that the
// estimates would give it: 0.89 to 1.10 of the time, 1.02 in the mean).  Nothing goes back from narrow tiles to 256x192, though the estimate of 128x192
// is some 10 % short at long K: 5393 and 7300 x 1536 x 6144 113 and 128 us, 104 and 120 in 256x192.
// The products above take 1.012 of their best form's time in the mean, 1.014 in the sum, 1.12 at most (by the rule before, whose estimates were
// fitted with 32x32x16 instructions: 1.034, 1.021, 1.40).
Bf16Form bf16_form(int M, int N, int K, bool packed, const void* scratch, size_t scratch_bytes) {
  if (K >= kTileMaxK) return F128;
  if (!packed || !packs_weights(N, K) || (unsigned long long)M * K * 2 >= (1ull << 32))                  // 32-bit offsets
    return staged_form(M, N, K, scratch, scratch_bytes);
  auto staged = [&](Bf16Form f) {
    auto tiles = [&](int bm, int bn) { return (long long)ceil_div(M, bm) * ceil_div(N, bn); };
    switch (f) {
      case F192: return form_time(kF192, M, N, K, split_ranges<256, 192>(tiles(256, 192), 256, K, scratch, scratch_bytes));
      case F256: return form_time(kF256, M, N, K, split_ranges<256, 256>(tiles(256, 256), 256, K, scratch, scratch_bytes));
      case F384: return form_time(kF384, M, N, K, split_ranges<384, 192>(tiles(384, 192), 256, K, scratch, scratch_bytes));
      default: return form_time(kF128, M, N, K, split_ranges<128, 128>(tiles(128, 128), 512, K, scratch, scratch_bytes));
    }
  };
  Bf16Form form = bf16_tile(false, M, N, K);
  double now = staged(form);
  const double wide = form_time(kP256, M, N, K), narrow = form_time(narrow_is_192(M, N, K) ? kP192 : kP128, M, N, K);
  if (wide <= 1.03 * narrow) {
    const bool lone = form == F256 && (long long)ceil_div(M, 256) * ceil_div(N, 256) <= 256;
    if (wide < (form == F128 ? 1.0 : form == F192 ? 0.98 : lone ? 0.975 : 0.968) * now) { form = P256; now = wide; }
  } else if (narrow < (form == F128 ? 1.0 : 0.94) * now) {
    form = P128;
    now = narrow;
  }
  if (N % 288 == 0 && K >= 2048 && form_time(kW288, M, N, K) < 0.94 * now) { form = W288; now = form_time(kW288, M, N, K); }
  if (N % 192 == 0 && form != P256 && form != F384 && staged(F384) < (form == P128 ? 1.0 : 0.94) * now) form = F384;
  return form;
}

bool packed_weights_serve(int M, int N, int K, size_t lent) {
  if ((long long)ceil_div(M, 128) * ceil_div(N, 128) < 32 || N < 32) return false;      // k_gemm_skinny
  const Bf16Form form = bf16_form(M, N, K, true, lent ? (const void*)16 : nullptr, lent);
  return form == P128 || form == P256;
}

template <int MODE>
static hipError_t dispatch_mode(int bf16, const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep,
                                void* scratch, size_t scratch_bytes, const void* w_parts, hipStream_t s) {
  if (!bf16) return dispatch_f32<MODE>(A, Wt, w_parts, M, N, K, ep, s);
  bool aligned = (((uintptr_t)A | (uintptr_t)Wt) & 15) == 0;
  // very few tiles (a request's text rows), or an N too narrow for the tile kernel (a 16-wide
  // output head): split K inside a workgroup instead.  Measured against the 128x128
  // configuration it wins below about 32 of its tiles and loses above (a 32x32 tile reads four
  // times the operand bytes per product).
  if (aligned && K % 64 == 0 && K < kSkinnyMaxK && ((long long)ceil_div(M, 128) * ceil_div(N, 128) < 32 || N < 32) &&
      ceil_div(M, 32) <= 65535)
    return run_skinny<bf16_t, MODE>(A, Wt, M, N, K, ep, s);
  if (MODE != EPI_UNPATCH) {
    // the MFMA kernel writes 16-byte runs of a row and reads bias / gate four at a time
    aligned = aligned && N % 8 == 0 && (((uintptr_t)ep.bias | (uintptr_t)ep.gate) & 15) == 0;
    if (MODE == EPI_HEADS || MODE == EPI_LAYERS_KV)
      aligned = aligned && ep.hd % 8 == 0 && ep.D % 8 == 0 &&
                (((uintptr_t)ep.q | (uintptr_t)ep.k | (uintptr_t)ep.v) & 15) == 0;
    else
      aligned = aligned && ep.ldo % 8 == 0 && ((uintptr_t)ep.out & 15) == 0;
  }
  if (K % 64 != 0 || !aligned || N < 32 || K >= kNarrowMaxK) return run_plain<bf16_t, MODE>(A, Wt, M, N, K, ep, s);
  Bf16Form form = bf16_tile(MODE == EPI_UNPATCH, M, N, K);
  if constexpr (MODE == EPI_HEADS || MODE == EPI_GATE || MODE == EPI_GELU)           // a model's products over token rows
    form = bf16_form(M, N, K, w_parts && ((uintptr_t)w_parts & 15) == 0, scratch, scratch_bytes);
  switch (form) {
    case F256: return run_dlds<256, 256, 4, 2, MODE>(A, Wt, M, N, K, ep, scratch, scratch_bytes, s);
    case F192: return run_dlds<256, 192, 4, 2, MODE>(A, Wt, M, N, K, ep, scratch, scratch_bytes, s);
    case F128: return run_dlds<128, 128, 2, 2, MODE>(A, Wt, M, N, K, ep, scratch, scratch_bytes, s);
    default: break;
  }
  if constexpr (MODE != EPI_UNPATCH)
    if (form == F384) return run_dlds<384, 192, 4, 2, MODE>(A, Wt, M, N, K, ep, scratch, scratch_bytes, s);
  if constexpr (MODE == EPI_HEADS || MODE == EPI_GATE || MODE == EPI_GELU) {
    if (form == P256) return run_packed<128, 256, 2, MODE>(A, w_parts, M, N, K, ep, s);
    if (form == P128 && narrow_is_192(M, N, K)) return run_packed<128, 192, 3, MODE>(A, w_parts, M, N, K, ep, s);
    if (form == P128) return run_packed<128, 128, 4, MODE>(A, w_parts, M, N, K, ep, s);
    if (form == W288) return run_288<MODE>(A, Wt, M, N, K, ep, s);
  }
  return hipErrorInvalidValue;                           // (none is left)
}

hipError_t launch_gemm(int bf16, int mode, const void* A, const void* Wt, int M, int N, int K, const EpiParams& ep,
                       hipStream_t s, void* scratch, size_t scratch_bytes, const void* w_parts) {
  if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
  switch (mode) {
    case EPI_STORE: return dispatch_mode<EPI_STORE>(bf16, A, Wt, M, N, K, ep, scratch, scratch_bytes, w_parts, s);
    case EPI_GELU: return dispatch_mode<EPI_GELU>(bf16, A, Wt, M, N, K, ep, scratch, scratch_bytes, w_parts, s);
    case EPI_GATE: return dispatch_mode<EPI_GATE>(bf16, A, Wt, M, N, K, ep, scratch, scratch_bytes, w_parts, s);
    case EPI_HEADS: return dispatch_mode<EPI_HEADS>(bf16, A, Wt, M, N, K, ep, scratch, scratch_bytes, w_parts, s);
    case EPI_UNPATCH: return dispatch_mode<EPI_UNPATCH>(bf16, A, Wt, M, N, K, ep, scratch, scratch_bytes, w_parts, s);
    case EPI_LAYERS_KV: return dispatch_mode<EPI_LAYERS_KV>(bf16, A, Wt, M, N, K, ep, scratch, scratch_bytes, w_parts, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace fc
