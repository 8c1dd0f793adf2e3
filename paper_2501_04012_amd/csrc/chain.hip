// Small fp32 models: everything of a block between two attentions in one launch.
//
// A block of a narrow model on a few hundred tokens is 16 launches of 3.6 to 4.8 us each in
// which next to nothing is computed: launch, first access to memory and drain bound it.  Apart
// from the keys and values of self-attention, every operator works on token rows alone, so
// a workgroup can take 16 rows of the residual stream through all of them in LDS: attention of its
// queries over the keys the previous launch wrote, output projection, residual, cross-attention,
// MLP, and the LayerNorm and QKV projection of the next attention (or the output head).  A
// factorized block is two launches, a full-3D block one; the patch embedding opens the first and
// the head closes the last.
//
// 16 rows: the smallest matrix-core tile (v_mfma_f32_16x16x4_f32, exact fp32), hence the most
// workgroups.  Weights are the A operand and rows the B operand, so that a lane ends up with four
// consecutive outputs of one row.  An operand lane (i, h) holds one 16-byte chunk of K and
// instruction e contracts element e of the four chunks (any order of K will do as long as both
// operands agree).  Weights come straight from global memory, laid out once per model in the order of the fragments
// (launch_pack_chain): a load of 64 lanes is 1 KB in a row, where rows of the plain layout gave it 64 bytes of each of 16
// (64 wide, six blocks full 3-D 123 -> 112 us; 128 wide, factorized 379 -> 351; 64 wide resume below 7.85 -> 7.61 ms).
//
// A workgroup is alone with its 16 rows, two waves to a SIMD, so what it takes is the latency of its loads (the weights of a
// deep model do not stay in an XCD's 4 MB of L2: some 2000 cycles a stage where a stage fetches its own) and the
// instructions of one wave after the other, 4 to 8 cycles each; the multiplications are a quarter.  Hence:
// - A product's first two batches of weights, its bias and gate, a LayerNorm's vectors and a head's first keys are on their way two
//   or three stages ahead (one stage, and only the first batch, with heads above 32, whose key tiles take the registers).
//   Barriers wait for LDS only.  A wait for a load counts the loads behind it, so these have to be known when this is compiled:
//   no branch of a single wave around them (what a wave does not need lies past the end of a buffer and reads as zero;
//   where no wave needs a second batch all skip it, as such a load still takes its 16 cycles of the CU's address unit),
//   and drain() where a rare path ends.
// - One miss for all of the kernel's arguments (touch_arguments), and little arithmetic on them: sizes in tiles and bytes come from the host.
// - No 64-bit lane addresses (a buffer, one 32-bit lane offset, immediate offsets), no predicates where a scalar branch will
//   do, the wave number a scalar (a masked-out matrix instruction would be issued all the same), one kernel per kind of launch.
//
// 64 wide, 4 heads, 28 blocks, 4 requests with guidance (512 rows), ten steps: 17.2 ms with a launch per operator, 7.53 with loads one
// stage ahead, 5.53 now; a spatial and a temporal launch 9 and 17 us before, 6 and 13 now.  Steps of one to three blocks, 160 sizes of 16
// to 128 columns: 0.92 of the time in the mean (64 and 128 wide factorized 0.80 to 0.86, full 3-D 0.9 to 1.0), none slower.
#include <type_traits>
#include "common.h"

namespace fc {

namespace {
constexpr int kChainWaves = 8;
constexpr int kChainRows = 16;
constexpr int kThreads = kChainWaves * 64;
constexpr int kThreadsPerRow = kThreads / kChainRows;     // 32 of four columns each: widths of up to 128

// floats of an LDS row; the 4 spread rows over the banks
__host__ __device__ __forceinline__ int lds_row(int v) { return v + 4; }

template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// v of this lane's 16-lane row and of its neighbour (row ^ 1), or of row and row ^ 2, in the same order for both
__device__ __forceinline__ void rows_xor1(float v, float& a, float& b) {
  const unsigned x = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const unsigned r0 = r[0], r1 = r[1];                    // a bit cast of a vector's element would read the first one
  a = __builtin_bit_cast(float, r0); b = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ void rows_xor2(float v, float& a, float& b) {
  const unsigned x = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  a = __builtin_bit_cast(float, r0); b = __builtin_bit_cast(float, r1);
}
// sum over the 32 lanes of an activation row
__device__ __forceinline__ float row_sum(float v) {
  v += dpp<0xB1>(v);                                      // lane ^ 1
  v += dpp<0x4E>(v);                                      // lane ^ 2
  v += dpp<0x141>(v);                                     // the other quad of 8 lanes
  v += dpp<0x140>(v);                                     // the other half of 16
  float a, b;
  rows_xor1(v, a, b);
  return a + b;
}
// over the four lanes that share lane & 15
__device__ __forceinline__ float quad_max(float v) {
  float a, b;
  rows_xor1(v, a, b);
  v = fmaxf(a, b);
  rows_xor2(v, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float quad_sum(float v) {
  float a, b;
  rows_xor1(v, a, b);
  v = a + b;
  rows_xor2(v, a, b);
  return a + b;
}

// barrier that orders LDS alone: loads from global memory stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources are a device-side type
// What lies past `bytes` loads as zero, without a request to memory: loads that a wave may not need are issued all the same, so that
// the number of loads behind one of them is known where it is waited for (under a branch the wait would be for all of them).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, unsigned byte) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte, 0, 0));
}
constexpr unsigned kAll = 0x7ffffff0, kNowhere = 0x7ffffff0;
// All loads have landed.  At the end of a path that few calls take: behind it a wait counts on the loads of either path, so what
// this one leaves on its way would be waited for, and all older loads with it, by those that did not take it.
__device__ __forceinline__ void drain() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Reads a word of every line of the kernel's arguments, all at once: left to their uses, a line at a time, each of them is a miss of
// the scalar cache that a stage begins with.
template <size_t BYTES> __device__ __forceinline__ void touch_arguments() {
  const auto* p = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
  int any = 0;
#pragma unroll
  for (size_t b = 0; b < BYTES; b += 64) any |= p[b / 4];
  asm volatile("" ::"s"(any));
}

// c + a b.  The sum never shares registers with c.  Left to itself the compiler moves the sum of a chain by two registers now and then, an
// output that overlaps the input it is added to without being the same registers.  What is known: a build with such products gave wrong
// sums (128 columns, third batch of a product, which is also the first whose weights take registers used before), and with this
// line, which changes schedule and waits besides, the sums are right.  That the overlap was the reason is inferred: waits for weights
// are the compiler's in either build.  tests/test_mfma_registers.py holds the rule.
__device__ __forceinline__ f32x4 mac(float a, float b, f32x4 c) {
  f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  asm volatile("" : "+v"(d) : "v"(c));
  return d;
}

using Yes = std::true_type; using No = std::false_type;

// 16 keys and values of a head, as attend() uses them; past the end the last key again
template <int HDT> struct KeyTile { f32x4 k[HDT]; float v[4][HDT]; };
template <int HDT>
__device__ __forceinline__ void fetch_keys(KeyTile<HDT>& t, const float* K, const float* V, bool on, int k0, int nk, int hd, unsigned stride) {
  const int lane = threadIdx.x & 63, i = lane & 15, h = lane >> 4;
  const bool half = hd & 8;
  const auto rk = buffer(K, on ? kAll : 0), rv = buffer(V, on ? kAll : 0);
  const unsigned ko = __umul24(min(k0 + i, nk - 1), stride);
#pragma unroll
  for (int j = 0; j < HDT; ++j) t.k[j] = load4(rk, 4 * (ko + (j + 1 < HDT || !half || h < 2 ? 16 * j + 4 * h : 0)));
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned vo = __umul24(min(k0 + 4 * h + e, nk - 1), stride);
#pragma unroll
    for (int j = 0; j < HDT; ++j)
      t.v[e][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rv, (int)(4 * (vo + (j + 1 < HDT || !half || i < 8 ? 16 * j + i : 0))), 0, 0));
  }
}

// One head of one sequence, or of several that lie one after the other, for 16 queries (a lane's
// query is lane & 15; qs: its head slice, scaled by log2(e) / sqrt(hd) already): scores as keys x
// queries, so that the probabilities are the B operand of V^T P as they stand.  Key j is at
// K + j * stride; keys lo .. hi - 1 count for this lane.  cur: the first 16 keys, on their way.  out(d, v): four consecutive
// outputs of the lane's query.  Returns whether a value is not finite: a key that does not count then leaves its mark
// all the same.
template <int HDT, typename Out>
__device__ __forceinline__ bool attend(const float* qs, int nk, int lo, int hi, int hd, const float* K, const float* V, unsigned stride,
                                       KeyTile<HDT>& cur, Out out) {
  const int lane = threadIdx.x & 63, i = lane & 15, h = lane >> 4;
  const bool half = hd & 8;                               // uniform: the last 16 columns are 8
  constexpr bool AHEAD = HDT <= 4;                        // the next tile's loads run under this one, registers permitting
  KeyTile<HDT> nxt;
  f32x4 q[HDT], acc[HDT];
#pragma unroll
  for (int j = 0; j < HDT; ++j) {
    q[j] = *(const f32x4*)(qs + (j + 1 < HDT || !half || h < 2 ? 16 * j + 4 * h : 0));
    acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  if (half && h >= 2) q[HDT - 1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // kNone: below every score, and finite: a lane may meet a tile without a key of its own first
  constexpr float kNone = -__FLT_MAX__;
  float m = kNone, l = 0.0f, probe = 0.0f;                // probe: 0, or NaN once a value is not finite
  auto tile = [&](int k0, auto more) {
    constexpr bool MORE = decltype(more)::value;
    if (AHEAD) { if (MORE && k0 + 16 < nk) fetch_keys<HDT>(nxt, K, V, true, k0 + 16, nk, hd, stride); }
    else if (k0 > 0) fetch_keys<HDT>(cur, K, V, true, k0, nk, hd, stride);
    __builtin_amdgcn_sched_barrier(0);
    if (half && h >= 2) cur.k[HDT - 1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < HDT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = mac(cur.k[j][e], q[j][e], s);
    const int key = k0 + 4 * h;
    bool in[4];
    float mc = kNone;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      in[e] = (unsigned)(key + e - lo) < (unsigned)(hi - lo);
      mc = fmaxf(mc, in[e] ? s[e] : kNone);
    }
    const float mn = fmaxf(m, quad_max(mc)), corr = __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    l *= corr;
    if (k0 > 0) {
#pragma unroll
      for (int j = 0; j < HDT; ++j) acc[j] *= corr;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float p = in[e] ? __builtin_amdgcn_exp2f(s[e] - m) : 0.0f;
      l += p;
#pragma unroll
      for (int j = 0; j < HDT; ++j) {
        // zero past the last key: its weight is 0, and 0 * inf is not
        float v = cur.v[e][j];
        if (k0 + 16 > nk) v = key + e < nk ? v : 0.0f;
        if (j + 1 == HDT && half) v = i < 8 ? v : 0.0f;
        acc[j] = mac(v, p, acc[j]);
        probe = __builtin_fmaf(v, 0.0f, probe);
      }
    }
    if (AHEAD && MORE) cur = nxt;
  };
  if (HDT <= 2 && nk <= 16) {                             // on its own, for the same reason as drain()
    tile(0, No{});
  } else {
    for (int k0 = 0; k0 < nk; k0 += 16) tile(k0, Yes{});
    drain();
  }
  const float inv = 1.0f / quad_sum(l);
#pragma unroll
  for (int j = 0; j < HDT; ++j)
    if (j + 1 < HDT || !half || h < 2) out(16 * j + 4 * h, acc[j] * inv);
  return probe != 0.0f;
}
#endif

// What a product starts with: the first two batches of a wave's weights, bias and gate of its first two tiles.
constexpr int U = 4;                                      // chunks of 16 of K per batch of loads
struct Ahead { f32x4 w[2][U], bias[2], gate[2]; };
// What a LayerNorm needs besides the rows
struct Modulation { f32x4 shift, scale; };

// The launches of a step.  CHAIN_EMBED: patch embedding.  CHAIN_SELF: self-attention.  CHAIN_CROSS,
// CHAIN_MLP: those branches.  All of them end with a LayerNorm and the next QKV projection or the head.
enum { CHAIN_EMBED = 1, CHAIN_SELF = 2, CHAIN_CROSS = 4, CHAIN_MLP = 8 };

template <int HDT, int KIND>
__global__ __launch_bounds__(kThreads) void k_chain(ChainArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr bool TEMPORAL = KIND & CHAIN_CROSS;            // rows in (b, s, t) order
  constexpr bool FULL = (KIND & CHAIN_MLP) && !(KIND & CHAIN_CROSS);            // full 3-D: one sequence per batch row
  extern __shared__ __attribute__((aligned(16))) float smem[];
  touch_arguments<sizeof(ChainArgs)>();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, h = lane >> 4;
  const int D = a.D, hd = a.hd, ld = lds_row(D), ldm = lds_row(a.mlp);
  float* const xt = smem;                                 // residual rows
  float* const u = xt + kChainRows * ld;                  // LayerNorm and attention output
  float* const o = u + kChainRows * ld;                   // queries
  float* const hid = o + kChainRows * ld;
  f32x4* const red = (f32x4*)(hid + (KIND & CHAIN_MLP ? kChainRows * ldm : 0));
  int* const again = (int*)(red + 6 * 64);                // the last KB of red: parts take 6 at most
  if (threadIdx.x == 0) *again = 0;

  // Row index -> row of the activations: natural order, or (b, s, t), in which temporal sequences are runs.
  // q, k and v of temporal attention are stored in that order.
  auto natural = [&](int idx) -> int {
    if (!TEMPORAL) return idx;
    const int b = a.by_N.div(idx), r = idx - b * a.N, s = a.by_T.div(r), t = r - s * a.T;
    return b * a.N + t * a.S + s;
  };
  const int idx0 = blockIdx.x * kChainRows;
  const int last = min(idx0 + kChainRows, a.rows) - 1;
  // elementwise stages: row er, columns ec .. ec + 3; matrix stages: row i.  Rows past the end are
  // copies of the last one, never stored.
  const int er = threadIdx.x / kThreadsPerRow, ec = threadIdx.x % kThreadsPerRow * 4;
  const bool e_in = ec < D;
  const int e_idx = min(idx0 + er, last), e_row = natural(e_idx);
  const int my = min(idx0 + i, last);
  const int my_row = natural(my);
  int my_alt = 0, e_alt = 0, e_b = 0, e_pos = 0;          // the text rows' own modulation set
  if ((FULL && a.alt_rows) || (KIND & CHAIN_EMBED)) {
    e_b = a.by_Ns.div(e_row);
    e_pos = e_row - e_b * a.Ns;
    e_alt = e_pos < a.alt_rows ? 6 * D : 0;
    my_alt = my_row - (int)a.by_Ns.div(my_row) * a.Ns < a.alt_rows ? 6 * D : 0;
  }

  // ---- loads ahead of their use
  auto issued = [] { __builtin_amdgcn_sched_barrier(0); };   // behind them: the scheduler would move the loads to their use
  // Products: tiles of 16 outputs, one per wave at a time; K in batches of U chunks.  K % 16 == 0; N % 16 == 0 but in the
  // head, whose rows past the end repeat the last.  With few tiles and a long K, several waves share a tile's K; their
  // parts are added in order through `red`.
  struct Share { int part, c0, c1, t; };
  auto share = [&](const ChainStep& p, bool split) {
    Share s{0, 0, p.chunks, wave};
    if (split && p.split) {
      s.part = (wave * p.split_mul) >> 8;                 // wave / tiles
      s.t = wave - s.part * p.tiles;
      s.c0 = (s.part * p.chunks) >> p.split;
      s.c1 = s.part >> p.split ? s.c0 : ((s.part + 1) * p.chunks) >> p.split;
    }
    return s;
  };
  auto fetch = [&](const ChainStep& p, int t, int c, f32x4 (&r)[U]) {
    const auto w = buffer(p.packed, p.w_bytes);
    const unsigned at = 1024u * (t * p.chunks + c) + 16u * lane;
#pragma unroll
    for (int x = 0; x < U; ++x) r[x] = load4(w, at + 1024 * x);
  };
  auto fetch_columns = [&](const ChainStep& p, int t, bool gated, f32x4& bias, f32x4& gate) {
    const unsigned at = 64u * t + 16u * h;
    bias = load4(buffer(p.bias, p.bias_bytes), at);
    if (gated) gate = load4(buffer(p.gate, p.vec_bytes), at + 4 * my_alt);
  };
  auto start_first = [&](const ChainStep& p, bool split, Ahead& f) {
    const Share s = share(p, split);
    fetch(p, s.t, s.c0, f.w[0]);
  };
  auto start_rest = [&](const ChainStep& p, bool split, bool gated, Ahead& f) {
    const Share s = share(p, split);
    fetch_columns(p, s.t, gated, f.bias[0], f.gate[0]);
    if (p.tiles > kChainWaves || p.chunks > U) {          // some wave has a second batch
      const bool same = s.c0 + U < s.c1;
      fetch(p, same ? s.t : s.t + kChainWaves, same ? s.c0 + U : s.c0, f.w[1]);
      if (p.tiles > kChainWaves) fetch_columns(p, s.t + kChainWaves, gated, f.bias[1], f.gate[1]);
    }
  };
  auto start = [&](const ChainStep& p, bool split, bool gated, Ahead& f) {
    start_first(p, split, f);
    start_rest(p, split, gated, f);
  };
  auto start_norm = [&](const ChainStep& p, int alt, Modulation& m) {
    const unsigned at = 4u * (alt + ec);                  // (columns past D are not used)
    m.shift = load4(buffer(p.shift, p.vec_bytes), at);
    m.scale = load4(buffer(p.scale, p.vec_bytes), at);
  };
  // A unit of attention is a head of one of the sequences (len rows each) these rows are in or, where those are shorter than
  // a key tile and lie one after the other, a head of all of them.
  struct Sequences { int first, n, mine; bool together; };
  auto sequences = [&](int len, const FastDiv& by_len, bool cross) {
    Sequences q;
    q.first = by_len.div(idx0);
    q.n = (int)by_len.div(last) - q.first + 1;
    q.mine = q.n > 1 ? (int)by_len.div(my) - q.first : 0;
    q.together = !cross && q.n > 1 && len < kChainRows;
    return q;
  };
  struct Unit { int sq, head, nk; size_t base; };
  auto unit = [&](int un, const Sequences& q, int len, int nk, bool cross, bool together) {
    Unit w;
    w.sq = un < a.heads ? 0 : (int)a.by_heads.div(un);
    w.head = un - w.sq * a.heads;
    const int seq = q.first + w.sq;
    w.nk = together ? q.n * len : nk;
    if (!cross) {
      w.base = (size_t)(seq * len) * D + w.head * hd;
    } else {
      const int kb = a.kv_shared_tail && seq >= a.kv_split ? a.kv_split : seq;
      w.base = ((size_t)kb * a.heads + w.head) * nk * hd;
    }
    return w;
  };
  auto start_keys = [&](const float* k, const float* v, int len, const FastDiv& by_len, int nk, bool cross, KeyTile<HDT>& t) {
    const Sequences q = sequences(len, by_len, cross);
    const Unit w = unit(wave, q, len, nk, cross, q.together);
    const bool on = wave < a.heads * (q.together ? 1 : q.n);
    fetch_keys<HDT>(t, k + (on ? w.base : 0), v + (on ? w.base : 0), on, 0, w.nk, hd, cross ? hd : D);
  };

  // ---- stages
  auto layer_norm = [&](const Modulation* m) {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (e_in) v = *(const f32x4*)(xt + er * ld + ec);
    const float mean = row_sum((v[0] + v[1]) + (v[2] + v[3])) * a.inv_d;
    f32x4 d = v - mean;
    if (!e_in) d = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float var = row_sum((d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3])) * a.inv_d;
    d = d * __builtin_amdgcn_rsqf(var + a.ln_eps);
    if (m) d = d * (1.0f + m->scale) + m->shift;
    if (e_in) *(f32x4*)(u + er * ld + ec) = d;
    return v;
  };
  auto product = [&](const ChainStep& p, auto split_k, auto gated_by, Ahead& f, const float* in, auto store) {
    constexpr bool SPLIT = decltype(split_k)::value, GATED = decltype(gated_by)::value;
    const Share s = share(p, SPLIT);
    const int nt = p.tiles;
    const bool split = SPLIT && p.split;
    const float* ap = in + 4 * h;
    int t = s.t, c = s.c0, ft = s.t, fc = s.c0;           // being multiplied; to be fetched next
    auto advance = [&](int& t, int& c) {
      c += U;
      if (c >= s.c1) { c = s.c0; t += kChainWaves; }
    };
    advance(ft, fc);
    advance(ft, fc);
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    // one batch; its registers take the one after the next; true while there is another
    auto batch = [&](f32x4 (&w)[U]) {
      f32x4 r[U];
#pragma unroll
      for (int x = 0; x < U; ++x) r[x] = *(const f32x4*)(ap + 16 * (c + x));
#pragma unroll
      for (int x = 0; x < U; ++x)
        if (x == 0 || c + x < s.c1)                       // past the end of K: other rows and weights
#pragma unroll
          for (int e = 0; e < 4; ++e) v = mac(w[x][e], r[x][e], v);
      if (ft < nt) {
        fetch(p, ft, fc, w);
        advance(ft, fc);
      }
      c += U;
      if (c < s.c1) return true;
      if (split) return false;
      store(t * 16 + 4 * h, v + f.bias[0], f.gate[0]);
      t += kChainWaves;
      if (t >= nt) return false;
      v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      c = s.c0;
      f.bias[0] = f.bias[1];
      if (GATED) f.gate[0] = f.gate[1];
      if (t + kChainWaves < nt) fetch_columns(p, t + kChainWaves, GATED, f.bias[1], f.gate[1]);
      return true;
    };
    if (t < nt && c < s.c1) {
      // the first two outside the loop: inside, a wait would have to hold for a fetch just made as well
      if (batch(f.w[0]) && batch(f.w[1])) {
        while (batch(f.w[0]) && batch(f.w[1])) {}
        drain();
      }
    }
    if (split) {
      const int parts = 1 << p.split;
      if (s.part > 0 && s.part < parts) red[((s.part - 1) * nt + s.t) * 64 + lane] = v;
      lds_barrier();
      if (s.part == 0) {
        for (int q = 1; q < parts; ++q) v += red[((q - 1) * nt + s.t) * 64 + lane];
        store(s.t * 16 + 4 * h, v + f.bias[0], f.gate[0]);
      }
    }
  };
  auto add = [&](int n, f32x4 v, f32x4) { *(f32x4*)(xt + i * ld + n) += v; };              // the residual; only this lane touches it
  auto add_gated = [&](int n, f32x4 v, f32x4 gate) { *(f32x4*)(xt + i * ld + n) += gate * v; };

  // Attention of the queries in o into u, and a barrier.  first: keys and values of this wave's first unit.  Units of several
  // sequences are repeated by sequence should a value of one not be finite, which zero weights do not keep from the others.
  auto attention = [&](const float* k, const float* v, int len, const FastDiv& by_len, int nk, bool cross, KeyTile<HDT>& first) {
    const Sequences q = sequences(len, by_len, cross);
    const unsigned stride = cross ? hd : D;
    bool together = q.together;
    auto one = [&](int un, KeyTile<HDT>& t) {
      const Unit w = unit(un, q, len, nk, cross, together);
      const bool mine = together || q.mine == w.sq;       // a lane of another sequence computes and drops
      const int lo = together ? q.mine * len : 0;
      return attend<HDT>(o + i * ld + w.head * hd, w.nk, lo, lo + nk, hd, k + w.base, v + w.base, stride, t,
                         [&](int d, f32x4 r) { if (mine) *(f32x4*)(u + i * ld + w.head * hd + d) = r; });
    };
    int un = wave, units = a.heads * (together ? 1 : q.n);
    bool bad = false;
    if (un < units) bad = one(un, first);
    un += kChainWaves;
    for (;;) {
      if (un < units) {
        for (; un < units; un += kChainWaves) {
          const Unit w = unit(un, q, len, nk, cross, together);
          KeyTile<HDT> t;
          fetch_keys<HDT>(t, k + w.base, v + w.base, true, 0, w.nk, hd, stride);
          bad |= one(un, t);
        }
        drain();
      }
      if (together && bad) *again = 1;
      lds_barrier();
      if (!together || !__builtin_amdgcn_readfirstlane(*again)) break;
      together = false;
      un = wave;
      units = a.heads * q.n;
    }
  };

  // ---- the rows, and what the first stages need
  constexpr bool EARLY = HDT <= 2;                        // registers permitting; else right before the stage
  const ChainStep& proj = a.step[CHAIN_PROJ];
  const ChainStep& next = a.step[CHAIN_NEXT];
  const bool head = !a.q_out;
  Ahead f_proj, f_xq, f_xproj, f_fc1, f_fc2, f_next;
  Modulation m_fc1, m_next;
  KeyTile<HDT> keys, xkeys;
  auto start_next = [&] {
    start(next, false, false, f_next);
    start_norm(next, head ? 0 : e_alt, m_next);
  };
  if constexpr (!(KIND & CHAIN_EMBED)) {
    const f32x4 x4 = load4(buffer(a.x, kAll), e_in ? 4u * (unsigned)(e_row * D + ec) : kNowhere);
    const f32x4 q4 = load4(buffer(a.q, kAll), e_in ? 4u * (unsigned)(e_idx * D + ec) : kNowhere);
    if constexpr (EARLY) {
      start_keys(a.k, a.v, a.seq_len, a.by_len, a.seq_len, false, keys);
      start(proj, false, true, f_proj);
      if constexpr (KIND & CHAIN_CROSS) start(a.step[CHAIN_XQ], false, false, f_xq);
      else if constexpr (KIND & CHAIN_MLP) { start(a.step[CHAIN_FC1], false, false, f_fc1); start_norm(a.step[CHAIN_FC1], e_alt, m_fc1); }
      else start_next();
    }
    issued();
    if (e_in) {
      *(f32x4*)(xt + er * ld + ec) = x4;
      *(f32x4*)(o + er * ld + ec) = q4;
    }
  } else {
    start_next();
    issued();
    if (e_in) {
      f32x4 x4;
      if (e_pos < a.text_rows) {
        const int tb = a.kv_shared_tail && e_b >= a.kv_split ? a.kv_split : e_b;
        x4 = *(const f32x4*)(a.y + ((size_t)tb * a.text_rows + e_pos) * D + ec);
      } else {
        const int run = a.p * a.C, n = e_pos - a.text_rows, t = a.by_S.div(n), s = n - t * a.S;
        const int ph = a.by_gw.div(s), pw = s - ph * a.by_gw.d;
        const float* src = a.latent + ((((size_t)(e_b < a.R ? e_b : e_b - a.R) * a.T + t) * a.H + (size_t)ph * a.p) * a.W + (size_t)pw * a.p) * a.C;
        const f32x4 pos = *(const f32x4*)(a.pos_sp + (size_t)s * D + ec) + *(const f32x4*)(a.pos_t + (size_t)t * D + ec);
        x4 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int dh = 0; dh < a.p; ++dh)
#pragma unroll 8
          for (int f = 0; f < run; ++f)
            x4 += src[(size_t)dh * a.W * a.C + f] * *(const f32x4*)(a.p_w + (size_t)(dh * run + f) * D + ec);
        x4 = (x4 + *(const f32x4*)(a.p_b + ec)) + pos;
      }
      *(f32x4*)(xt + er * ld + ec) = x4;
    }
  }

  if constexpr (KIND & CHAIN_SELF) {
    if constexpr (!EARLY) {
      start_keys(a.k, a.v, a.seq_len, a.by_len, a.seq_len, false, keys);
      start_first(proj, false, f_proj);
      issued();
    }
    lds_barrier();
    attention(a.k, a.v, a.seq_len, a.by_len, a.seq_len, false, keys);
    if constexpr (!EARLY) start_rest(proj, false, true, f_proj);
    if constexpr (EARLY && (KIND & CHAIN_CROSS)) {
      start_keys(a.xk, a.xv, a.Ns, a.by_Ns, a.L, true, xkeys);
      start(a.step[CHAIN_XPROJ], false, false, f_xproj);
    } else if constexpr (EARLY && (KIND & CHAIN_MLP)) {
      start(a.step[CHAIN_FC2], true, true, f_fc2);
    }
    issued();
    product(proj, No{}, Yes{}, f_proj, u + i * ld, add_gated);
  }
  if constexpr (KIND & CHAIN_CROSS) {
    const ChainStep& p = a.step[CHAIN_XQ];
    if constexpr (EARLY) {
      start(a.step[CHAIN_FC1], false, false, f_fc1);
      start_norm(a.step[CHAIN_FC1], e_alt, m_fc1);
    } else {
      start(p, false, false, f_xq);
    }
    issued();
    lds_barrier();
    layer_norm(nullptr);
    lds_barrier();
    product(p, No{}, No{}, f_xq, u + i * ld, [&](int n, f32x4 v, f32x4) { *(f32x4*)(o + i * ld + n) = v * a.qscale; });
    if constexpr (EARLY) {
      start(a.step[CHAIN_FC2], true, true, f_fc2);
    } else {
      start_keys(a.xk, a.xv, a.Ns, a.by_Ns, a.L, true, xkeys);
      start_first(a.step[CHAIN_XPROJ], false, f_xproj);
    }
    issued();
    lds_barrier();
    attention(a.xk, a.xv, a.Ns, a.by_Ns, a.L, true, xkeys);
    if constexpr (!EARLY) start_rest(a.step[CHAIN_XPROJ], false, false, f_xproj);
    issued();
    product(a.step[CHAIN_XPROJ], No{}, No{}, f_xproj, u + i * ld, add);
  }
  if constexpr (KIND & CHAIN_MLP) {
    const ChainStep& p = a.step[CHAIN_FC1];
    if constexpr (EARLY) {
      start_next();
    } else {
      start(p, false, false, f_fc1);
      start_norm(p, e_alt, m_fc1);
    }
    issued();
    lds_barrier();
    layer_norm(&m_fc1);
    lds_barrier();
    product(p, No{}, No{}, f_fc1, u + i * ld, [&](int n, f32x4 v, f32x4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_tanh_f(v[e]);
      *(f32x4*)(hid + i * ldm + n) = v;
    });
    if constexpr (!EARLY) start(a.step[CHAIN_FC2], true, true, f_fc2);
    issued();
    lds_barrier();
    product(a.step[CHAIN_FC2], Yes{}, Yes{}, f_fc2, hid + i * ldm, add_gated);
  }
  // ---- the next self-attention's queries, keys and values, or the output head
  if constexpr (!EARLY && !(KIND & CHAIN_EMBED)) start_next();
  issued();
  lds_barrier();
  const f32x4 x4 = layer_norm(&m_next);
  if (!head) {
    if (e_in && idx0 + er <= last) *(f32x4*)(a.x_out + (unsigned)(e_row * D + ec)) = x4;
    lds_barrier();
    int out_row = my_row;                                 // in the next attention's order
    if constexpr (KIND == CHAIN_SELF) {
      const int b = a.by_N.div(my_row), r = my_row - b * a.N, t = a.by_S.div(r), s = r - t * a.S;
      out_row = b * a.N + s * a.T + t;
    }
    const bool mine = idx0 + i <= last;
    product(next, No{}, No{}, f_next, u + i * ld, [&](int n, f32x4 v, f32x4) {
      const int which = n >= 2 * D ? 2 : n >= D ? 1 : 0, c = n - which * D;     // D % 16 == 0: uniform but for c
      float* dst = which == 0 ? a.q_out : which == 1 ? a.k_out : a.v_out;
      if (which == 0) v *= a.qscale;
      if (mine) *(f32x4*)(dst + (unsigned)(out_row * D + c)) = v;
    });
  } else {
    const ChainStep& p = next;
    lds_barrier();
    const int b = a.by_Ns.div(my_row), n0 = my_row - b * a.Ns - a.text_rows;
    const bool mine = idx0 + i <= last && n0 >= 0;        // text rows have no head
    const int f0 = a.by_S.div(mine ? n0 : 0), s = (mine ? n0 : 0) - f0 * a.S, ph = a.by_gw.div(s), pw = s - ph * a.by_gw.d;
    const size_t at = ((((size_t)b * a.T + f0) * a.H + (size_t)ph * a.p) * a.W + (size_t)pw * a.p) * a.C;
    for (int t = wave; t * 16 < p.N; t += kChainWaves) {
      const int row = t * 16 + i;
      const float* wp = p.w + (size_t)(row < p.N ? row : p.N - 1) * D + 4 * h;
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
      for (int c = 0; c < D; c += 16) {
        const f32x4 w = *(const f32x4*)(wp + c), r = *(const f32x4*)(u + i * ld + 4 * h + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) v = mac(w[e], r[e], v);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = t * 16 + 4 * h + e;
        if (mine && n < p.N) {
          const int dh = a.by_run.div(n), c = n - dh * a.by_run.d;
          const size_t o = at + (size_t)dh * a.W * a.C + c;
          const float est = v[e] + p.bias[n];
          if (a.latent_out) {                             // no other row reads or writes these elements
            const float x0 = (a.latent_out[o] - a.c1 * est) / a.c0;
            a.latent_out[o] = a.c2 * x0 + a.c3 * est;
          }
          if (a.eps) a.eps[o] = est;
        }
      }
    }
  }
#endif
}

__global__ __launch_bounds__(256) void k_pack_chain(const float* __restrict__ w, float* __restrict__ packed, int N, int K) {
  const int x = blockIdx.x * 256 + threadIdx.x, lane = x & 63, c = (x >> 6) % (K >> 4), t = (x >> 6) / (K >> 4);
  if (t * 16 >= N) return;
  *(f32x4*)(packed + (size_t)x * 4) = *(const f32x4*)(w + (size_t)(t * 16 + (lane & 15)) * K + c * 16 + (lane >> 4) * 4);
}

template <int HDT, int KIND>
hipError_t run_chain(const ChainArgs& a, hipStream_t s) {
  static_assert(kThreads == 512, "eight waves");
  const size_t smem = (size_t)kChainRows * (3 * lds_row(a.D) + (KIND & CHAIN_MLP ? lds_row(a.mlp) : 0)) * 4 + (kChainWaves - 1) * 1024;
  k_chain<HDT, KIND><<<ceil_div(a.rows, kChainRows), kThreads, smem, s>>>(a);
  return hipGetLastError();
}
template <int HDT>
hipError_t run_kind(const ChainArgs& a, hipStream_t s) {
  if (a.step[CHAIN_XQ].w) return run_chain<HDT, CHAIN_SELF | CHAIN_CROSS | CHAIN_MLP>(a, s);
  if (a.step[CHAIN_FC1].w) {                              // full 3-D: not at a width of 128 (chain_fits)
    if constexpr (HDT < 8) return run_chain<HDT, CHAIN_SELF | CHAIN_MLP>(a, s);
    else return hipErrorInvalidValue;
  }
  return run_chain<HDT, CHAIN_SELF>(a, s);
}
}  // namespace

// Where the chain is the faster form.  keys: of the longest self-attention; text: of the cross-attention, 0 in the
// full-3D form, where text and video are one sequence.  A workgroup walks all keys of its rows alone, a wave per
// head and eight heads at a time, and what it saves in launches shrinks with the width.  Steps of four blocks, us, chain
// against one launch per operator:
//   rows: 64 wide 134 against 274 at 16 and 408 against 630 at 3080; 128 wide 308 against 318 at 64, 16384 lose.
//   full 3-D: 128 wide loses at 1 to 16 heads (4: 167 against 156 at 72 keys; 16: 214 against 160 at 152).  Up to eight
//     heads the narrower ones win (112 wide, 7 heads: 0.90 to 0.99 of the time); above that 80 wide wins up to 390 keys
//     (0.99; 512: 1.06), 96 up to 170 (164: 0.99; 264: 1.06), 112 hardly (24: 0.96; 72: 1.02).
//   cross-attention: up to four heads win at any text tried (128 wide, 4: 0.91 at 4096); five to eight lose at
//     128 wide from about 600 text keys (512: 1.03 and 0.95, 1024: 1.06 and 0.98 at 64 and 256 rows; 4096: 1.12) and
//     at 64 wide above 2700 (0.96; 4096: 1.09); more than eight win while self-attention and text have fewer than 16 keys
//     per column that is missing to 128 (80 wide: 664 keys 0.93; 96: 320 0.94, 664 1.07; 112: 244 1.00, 272 1.04; 128,
//     16 heads: 80 1.03, 4096 rows but none else win).
// Above 640 keys a lone head of 16 or 32 columns still wins (1032 keys: 160 against 286 us), but not every form has been
// timed there.
bool chain_fits(const ChainArgs& a, int keys, int text) {
  const int missing = 128 - a.D;
  if (missing < 0 || a.D % 16 != 0 || a.mlp > 512 || a.mlp % 16 != 0 || (long long)a.rows * a.D > 1 << 20 || keys > 640 ||
      keys * a.D > 40960)
    return false;
  if (text == 0) return missing > 0 && (a.heads <= 8 || 6 * keys <= missing * missing);
  if (a.heads > 8) return keys + (long long)text < 16 * missing;
  return text <= (a.heads <= 4 ? 1 << 20 : missing > 0 ? 2560 : 512);    // 2^20: key offsets are 24-bit products
}

hipError_t launch_pack_chain(const float* w, float* packed, int N, int K, hipStream_t s) {
  if (N % 16 != 0 || K % 16 != 0 || (long long)N * K > 1 << 28) return hipErrorInvalidValue;
  k_pack_chain<<<ceil_div((long long)N * K / 4, 256), 256, 0, s>>>(w, packed, N, K);
  return hipGetLastError();
}

hipError_t launch_chain(const ChainArgs& args, hipStream_t s) {
  if (args.rows <= 0) return hipSuccess;
  ChainArgs a = args;
  a.inv_d = 1.0f / (float)a.D;
  a.by_N = FastDiv(a.N); a.by_Ns = FastDiv(a.Ns); a.by_T = FastDiv(a.T); a.by_S = FastDiv(a.S);
  a.by_heads = FastDiv(a.heads); a.by_len = FastDiv(a.seq_len > 0 ? a.seq_len : 1);
  for (ChainStep& p : a.step) {
    if (!p.w) continue;
    p.tiles = ceil_div(p.N, 16); p.chunks = p.K / 16;
    p.split = 2 * p.tiles <= kChainWaves && p.chunks >= 8 ? 4 * p.tiles <= kChainWaves ? 2 : 1 : 0;
    p.split_mul = 256 / p.tiles + 1;                      // wave * mul >> 8 = wave / tiles: 8 waves, up to 4 tiles
    p.w_bytes = p.packed ? (unsigned)p.N * p.K * 4 : 0;   // (nothing is loaded for the head, which reads w)
    p.bias_bytes = p.N * 4;
    p.vec_bytes = (a.alt_rows ? 7 : 1) * a.D * 4;         // gate, shift, scale; a text row's are 6 D on
  }
  a.by_run = FastDiv(a.p * a.C); a.by_gw = FastDiv(a.W / a.p);
  if (a.latent) return run_chain<1, CHAIN_EMBED>(a, s);
  switch ((a.hd + 15) / 16) {
    case 1: return run_kind<1>(a, s);
    case 2: return run_kind<2>(a, s);
    case 4: return run_kind<4>(a, s);
    case 6: return run_kind<6>(a, s);
    case 8: return run_kind<8>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace fc
