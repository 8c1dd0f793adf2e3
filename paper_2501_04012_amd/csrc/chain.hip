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
// A workgroup is alone with its 16 rows, two waves to a SIMD, so what it takes is the instructions of
// one wave after the other, 4 to 8 cycles each, and little of that is multiplication.  Hence: no
// 64-bit lane addresses (a uniform base, one 32-bit lane offset, immediate offsets), no predicates
// where a scalar branch will do, the wave number a scalar (a masked-out matrix instruction would be
// issued all the same), one kernel per kind of launch, and the first weights of a product on their way
// before the stage in front of it begins (barriers wait for LDS only).
//
// 64 wide, 4 heads, 28 blocks, 4 requests with guidance (512 rows), ten steps: 17.2 -> 7.6 ms, of which a
// spatial and a temporal launch take about 9 and 17 us.
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

// One head of one sequence, or of several that lie one after the other, for 16 queries (a lane's
// query is lane & 15; qs: its head slice, scaled by log2(e) / sqrt(hd) already): scores as keys x
// queries, so that the probabilities are the B operand of V^T P as they stand.  Key j is at
// K + j * stride; keys lo .. hi - 1 count for this lane.  out(d, v): four consecutive outputs of the
// lane's query.  Returns whether a value is not finite: a key that does not count then leaves its mark
// all the same.
template <int HDT, typename Out>
__device__ __forceinline__ bool attend(const float* qs, int nk, int lo, int hi, int hd, const float* __restrict__ K,
                                       const float* __restrict__ V, unsigned stride, Out out) {
  const int lane = threadIdx.x & 63, i = lane & 15, h = lane >> 4;
  struct Tile { f32x4 k[HDT]; float v[4][HDT]; };
  const bool half = hd & 8;                               // uniform: the last 16 columns are 8
  auto fetch = [&](int k0, Tile& t) {                     // past the end: the last key again
    const unsigned ko = __umul24(min(k0 + i, nk - 1), stride);
#pragma unroll
    for (int j = 0; j < HDT; ++j) t.k[j] = *(const f32x4*)(K + (ko + (j + 1 < HDT || !half || h < 2 ? 16 * j + 4 * h : 0)));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned vo = __umul24(min(k0 + 4 * h + e, nk - 1), stride);
#pragma unroll
      for (int j = 0; j < HDT; ++j) t.v[e][j] = V[vo + (j + 1 < HDT || !half || i < 8 ? 16 * j + i : 0)];
    }
  };
  constexpr bool AHEAD = HDT <= 4;                        // the next tile's loads run under this one, registers permitting
  Tile cur, nxt;
  fetch(0, cur);
  __builtin_amdgcn_sched_barrier(0);
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
  for (int k0 = 0; k0 < nk; k0 += 16) {
    if (AHEAD) { if (k0 + 16 < nk) fetch(k0 + 16, nxt); }
    else if (k0 > 0) fetch(k0, cur);
    __builtin_amdgcn_sched_barrier(0);
    if (half && h >= 2) cur.k[HDT - 1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < HDT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.k[j][e], q[j][e], s, 0, 0, 0);
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
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, p, acc[j], 0, 0, 0);
        probe = __builtin_fmaf(v, 0.0f, probe);
      }
    }
    if (AHEAD) cur = nxt;
  }
  const float inv = 1.0f / quad_sum(l);
#pragma unroll
  for (int j = 0; j < HDT; ++j)
    if (j + 1 < HDT || !half || h < 2) out(16 * j + 4 * h, acc[j] * inv);
  return probe != 0.0f;
}

// First weights of a product: what product() starts with.
constexpr int U = 4;                                      // chunks of 16 of K per batch of loads
struct Ahead { f32x4 w[U]; };

// The launches of a step.  CHAIN_EMBED: patch embedding.  CHAIN_SELF: self-attention.  CHAIN_CROSS,
// CHAIN_MLP: those branches.  All of them end with a LayerNorm and the next QKV projection or the head.
enum { CHAIN_EMBED = 1, CHAIN_SELF = 2, CHAIN_CROSS = 4, CHAIN_MLP = 8 };

template <int HDT, int KIND>
__global__ __launch_bounds__(kThreads) void k_chain(ChainArgs a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, h = lane >> 4;
  const int D = a.D, hd = a.hd, ld = lds_row(D), ldm = lds_row(a.mlp);
  float* const xt = smem;                                 // residual rows
  float* const u = xt + kChainRows * ld;                  // LayerNorm and attention output
  float* const o = u + kChainRows * ld;                   // queries
  float* const hid = o + kChainRows * ld;
  f32x4* const red = (f32x4*)(hid + (KIND & CHAIN_MLP ? kChainRows * ldm : 0));

  // Row index -> row of the activations: natural order, or (b, s, t), in which temporal sequences are runs.
  // q, k and v of temporal attention are stored in that order.
  auto natural = [&](int idx) -> int {
    if (!a.temporal) return idx;
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
  const int my_row = a.temporal ? natural(my) : my;
  int my_alt = 0, e_alt = 0, e_b = 0, e_pos = 0;          // the text rows' own modulation set
  if (a.alt_rows || (KIND & CHAIN_EMBED)) {
    e_b = a.by_Ns.div(e_row);
    e_pos = e_row - e_b * a.Ns;
    e_alt = e_pos < a.alt_rows ? 6 * D : 0;
    my_alt = my_row - (int)a.by_Ns.div(my_row) * a.Ns < a.alt_rows ? 6 * D : 0;
  }

  // ---- the rows
  if (e_in) {
    f32x4 x4;
    if constexpr (!(KIND & CHAIN_EMBED)) {
      x4 = *(const f32x4*)(a.x + (unsigned)(e_row * D + ec));
      *(f32x4*)(o + er * ld + ec) = *(const f32x4*)(a.q + (unsigned)(e_idx * D + ec));
    } else if (e_pos < a.text_rows) {
      const int tb = a.kv_shared_tail && e_b >= a.kv_split ? a.kv_split : e_b;
      x4 = *(const f32x4*)(a.y + ((size_t)tb * a.text_rows + e_pos) * D + ec);
    } else {
      const int run = a.p * a.C, n = e_pos - a.text_rows, t = a.by_S.div(n), s = n - t * a.S;
      const int ph = a.by_gw.div(s), pw = s - ph * a.by_gw.d;
      const float* src = a.latent + ((((size_t)(e_b < a.R ? e_b : e_b - a.R) * a.T + t) * a.H + (size_t)ph * a.p) * a.W + (size_t)pw * a.p) * a.C;
      const f32x4 pos = *(const f32x4*)(a.pos_sp + (size_t)s * D + ec) + *(const f32x4*)(a.pos_t + (size_t)t * D + ec);
      x4 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      for (int dh = 0; dh < a.p; ++dh)
#pragma unroll 4
        for (int f = 0; f < run; ++f)
          x4 += src[(size_t)dh * a.W * a.C + f] * *(const f32x4*)(a.p_w + (size_t)(dh * run + f) * D + ec);
      x4 = (x4 + *(const f32x4*)(a.p_b + ec)) + pos;
    }
    *(f32x4*)(xt + er * ld + ec) = x4;
  }

  // ---- stages
  auto layer_norm = [&](const float* shift, const float* scale, int alt) {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f}, sh = v, sc = v;
    if (e_in) {
      if (shift) { sh = *(const f32x4*)(shift + (unsigned)(alt + ec)); sc = *(const f32x4*)(scale + (unsigned)(alt + ec)); }
      v = *(const f32x4*)(xt + er * ld + ec);
    }
    const float mean = row_sum((v[0] + v[1]) + (v[2] + v[3])) * a.inv_d;
    f32x4 d = v - mean;
    if (!e_in) d = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float var = row_sum((d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3])) * a.inv_d;
    d = d * __builtin_amdgcn_rsqf(var + a.ln_eps);
    if (shift) d = d * (1.0f + sc) + sh;
    if (e_in) *(f32x4*)(u + er * ld + ec) = d;
    return v;
  };
  // Tiles of 16 outputs, one per wave at a time; K in batches of U chunks whose loads run one batch ahead and
  // on into the wave's next tile.  K % 16 == 0; N % 16 == 0 but in the head, whose rows past the end
  // repeat the last.  With few tiles and a long K, several waves share a tile's K; their parts are added in
  // order through `red`.
  struct Share { int nt, ch, part, parts, c0, c1, t; };
  auto share = [&](int N, int K, bool split) {
    Share s;
    s.nt = (N + 15) >> 4; s.ch = K >> 4; s.part = 0; s.parts = 1; s.c0 = 0; s.c1 = s.ch; s.t = wave;
    if (split && s.nt * 2 <= kChainWaves && s.ch >= 8) {
      s.parts = s.nt * 4 <= kChainWaves ? 4 : 2;
      for (; s.t >= s.nt; s.t -= s.nt) ++s.part;
      s.c0 = s.part * s.ch / s.parts;
      s.c1 = s.part < s.parts ? (s.part + 1) * s.ch / s.parts : s.c0;
    }
    return s;
  };
  auto fetch = [&](const ChainStep& p, int t, int c, int c1, f32x4 (&r)[U]) {
    const float* base = p.packed + (size_t)(t * (p.K >> 4) + c) * 256;     // uniform
#pragma unroll
    for (int x = 0; x < U; ++x)
      if (c + x < c1) r[x] = *(const f32x4*)(base + 256 * x + 4 * lane);
  };
  auto ahead = [&](const ChainStep& p, bool split) {
    Ahead f;
    const Share s = share(p.N, p.K, split);
    if (s.t < s.nt) fetch(p, s.t, s.c0, s.c1, f.w);
    __builtin_amdgcn_sched_barrier(0);
    return f;
  };
  auto product = [&](const ChainStep& p, bool split, Ahead& f, const float* in, auto gate_at, auto store) {
    const Share s = share(p.N, p.K, split);
    const float* ap = in + 4 * h;
    for (int t = s.t; t < s.nt; t += kChainWaves) {
      const int n = t * 16 + 4 * h;
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f}, bias = v;
      if (n < p.N) bias = *(const f32x4*)(p.bias + (unsigned)n);      // the buffer is a multiple of 256 bytes
      const f32x4 gate = gate_at(n);
      for (int c = s.c0; c < s.c1; c += U) {
        f32x4 nx[U];
        if (c + U < s.c1) fetch(p, t, c + U, s.c1, nx);
        else if (s.parts == 1 && t + kChainWaves < s.nt) fetch(p, t + kChainWaves, s.c0, s.c1, nx);
        __builtin_amdgcn_sched_barrier(0);                // the scheduler would move the loads to their use
#pragma unroll
        for (int x = 0; x < U; ++x)
          if (c + x < s.c1) {
            const f32x4 r = *(const f32x4*)(ap + 16 * (c + x));
#pragma unroll
            for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(f.w[x][e], r[e], v, 0, 0, 0);
          }
#pragma unroll
        for (int x = 0; x < U; ++x) f.w[x] = nx[x];
      }
      if (s.parts > 1) {
        if (s.part > 0 && s.part < s.parts) red[((s.part - 1) * s.nt + t) * 64 + lane] = v;
        lds_barrier();                                    // once, and by every wave: t < nt
        if (s.part > 0) break;
        for (int q = 1; q < s.parts; ++q) v += red[((q - 1) * s.nt + t) * 64 + lane];
      }
      store(n, v + bias, gate);
    }
  };
  auto no_gate = [](int) { return f32x4{1.0f, 1.0f, 1.0f, 1.0f}; };
  auto add = [&](int n, f32x4 v, f32x4 gate) { *(f32x4*)(xt + i * ld + n) += gate * v; };   // the residual; only this lane touches it

  // Attention of the queries in o into u.  A unit is a head of one of the sequences (len rows each) these rows
  // are in or, where those are shorter than a key tile and lie one after the other, a head of all of them:
  // repeated by sequence should a value of one not be finite, which zero weights do not keep from the others.
  auto attention = [&](const float* k, const float* v, int len, const FastDiv& by_len, int nk, bool cross) {
    const int seq0 = by_len.div(idx0), nseq = (int)by_len.div(last) - seq0 + 1;
    const int my_seq = nseq > 1 ? (int)by_len.div(my) - seq0 : 0;
    bool together = !cross && nseq > 1 && len < kChainRows;
    for (;;) {
      bool bad = false;
      const int units = a.heads * (together ? 1 : nseq);
      for (int un = wave; un < units; un += kChainWaves) {
        const int sq = un < a.heads ? 0 : (int)a.by_heads.div(un), head = un - sq * a.heads, seq = seq0 + sq;
        size_t base;
        if (!cross) {
          base = (size_t)(seq * len) * D + head * hd;
        } else {
          const int kb = a.kv_shared_tail && seq >= a.kv_split ? a.kv_split : seq;
          base = ((size_t)kb * a.heads + head) * nk * hd;
        }
        const bool mine = together || my_seq == sq;       // a lane of another sequence computes and drops
        const int lo = together ? my_seq * len : 0;
        bad |= attend<HDT>(o + i * ld + head * hd, together ? nseq * len : nk, lo, lo + nk, hd, k + base, v + base, cross ? hd : D,
                           [&](int d, f32x4 r) { if (mine) *(f32x4*)(u + i * ld + head * hd + d) = r; });
      }
      if (!together) break;
      together = false;
      if (!__syncthreads_or(bad)) break;
    }
  };

  if constexpr (KIND & CHAIN_SELF) {
    const ChainStep& p = a.step[CHAIN_PROJ];
    Ahead f = ahead(p, false);
    lds_barrier();
    attention(a.k, a.v, a.seq_len, a.by_len, a.seq_len, false);
    lds_barrier();
    product(p, false, f, u + i * ld, [&](int n) { return *(const f32x4*)(p.gate + (unsigned)(my_alt + n)); }, add);
  }
  if constexpr (KIND & CHAIN_CROSS) {
    const ChainStep& pq = a.step[CHAIN_XQ];
    Ahead f = ahead(pq, false);
    lds_barrier();
    layer_norm(nullptr, nullptr, 0);
    lds_barrier();
    product(pq, false, f, u + i * ld, no_gate, [&](int n, f32x4 v, f32x4) { *(f32x4*)(o + i * ld + n) = v * a.qscale; });
    const ChainStep& p = a.step[CHAIN_XPROJ];
    f = ahead(p, false);
    lds_barrier();
    attention(a.xk, a.xv, a.Ns, a.by_Ns, a.L, true);
    lds_barrier();
    product(p, false, f, u + i * ld, no_gate, add);
  }
  if constexpr (KIND & CHAIN_MLP) {
    const ChainStep& p1 = a.step[CHAIN_FC1];
    Ahead f = ahead(p1, false);
    lds_barrier();
    layer_norm(p1.shift, p1.scale, e_alt);
    lds_barrier();
    product(p1, false, f, u + i * ld, no_gate, [&](int n, f32x4 v, f32x4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_tanh_f(v[e]);
      *(f32x4*)(hid + i * ldm + n) = v;
    });
    const ChainStep& p2 = a.step[CHAIN_FC2];
    f = ahead(p2, true);
    lds_barrier();
    product(p2, true, f, hid + i * ldm, [&](int n) { return *(const f32x4*)(p2.gate + (unsigned)(my_alt + n)); }, add);
  }
  // ---- the next self-attention's queries, keys and values, or the output head
  const ChainStep& p = a.step[CHAIN_NEXT];
  if (!a.eps) {
    Ahead f = ahead(p, false);
    lds_barrier();
    const f32x4 x4 = layer_norm(p.shift, p.scale, e_alt);
    if (e_in && idx0 + er <= last) *(f32x4*)(a.x_out + (unsigned)(e_row * D + ec)) = x4;
    lds_barrier();
    int out_row = my_row;                                 // in the next attention's order
    if (a.next_temporal) {
      const int b = a.by_N.div(my_row), r = my_row - b * a.N, t = a.by_S.div(r), s = r - t * a.S;
      out_row = b * a.N + s * a.T + t;
    }
    const bool mine = idx0 + i <= last;
    product(p, false, f, u + i * ld, no_gate, [&](int n, f32x4 v, f32x4) {
      const int which = n >= 2 * D ? 2 : n >= D ? 1 : 0, c = n - which * D;     // D % 16 == 0: uniform but for c
      float* dst = which == 0 ? a.q_out : which == 1 ? a.k_out : a.v_out;
      if (which == 0) v *= a.qscale;
      if (mine) *(f32x4*)(dst + (unsigned)(out_row * D + c)) = v;
    });
  } else {
    lds_barrier();
    layer_norm(p.shift, p.scale, 0);
    lds_barrier();
    const int b = a.by_Ns.div(my_row), n0 = my_row - b * a.Ns - a.text_rows;
    const bool mine = idx0 + i <= last && n0 >= 0;        // text rows have no head
    const int f0 = a.by_S.div(mine ? n0 : 0), s = (mine ? n0 : 0) - f0 * a.S, ph = a.by_gw.div(s), pw = s - ph * a.by_gw.d;
    float* dst = a.eps + ((((size_t)b * a.T + f0) * a.H + (size_t)ph * a.p) * a.W + (size_t)pw * a.p) * a.C;
    for (int t = wave; t * 16 < p.N; t += kChainWaves) {
      const int row = t * 16 + i;
      const float* wp = p.w + (size_t)(row < p.N ? row : p.N - 1) * D + 4 * h;
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
      for (int c = 0; c < D; c += 16) {
        const f32x4 w = *(const f32x4*)(wp + c), r = *(const f32x4*)(u + i * ld + 4 * h + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], r[e], v, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = t * 16 + 4 * h + e;
        if (mine && n < p.N) {
          const int dh = a.by_run.div(n), c = n - dh * a.by_run.d;
          dst[(size_t)dh * a.W * a.C + c] = v[e] + p.bias[n];
        }
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_pack_chain(const float* __restrict__ w, float* __restrict__ packed, int N, int K) {
  const int x = blockIdx.x * 256 + threadIdx.x, lane = x & 63, c = (x >> 6) % (K >> 4), t = (x >> 6) / (K >> 4);
  if (t * 16 >= N) return;
  *(f32x4*)(packed + (size_t)x * 4) = *(const f32x4*)(w + (size_t)(t * 16 + (lane & 15)) * K + c * 16 + (lane >> 4) * 4);
}

template <int HDT, int KIND>
hipError_t run_chain(const ChainArgs& a, hipStream_t s) {
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
