// Restoring a cached latent, the input of the resume loop: stitching an object and a
// background cache with their 1-bit masks (Sec. 4.2.2), expanding a compressed entry
// (Sec. 4.1: first frame + alpha * base differentials, extra frames, repeated key frames),
// and the two reductions of the compressing side that define what is expanded (Eq. 2's
// least-squares coefficient, the frame cosine similarities the key frames are chosen by).
// All of it moves each byte once: the kernels are bound by HBM.
#include <type_traits>
#include "common.h"

namespace fc {

// ---------------------------------------------------------------- stitching
// take_obj(pixel) = m_obj OR NOT m_bg; out = take_obj ? x_obj : x_bg for every channel of
// the pixel.  Masks: pixel i is bit i % 8 of byte i / 8.  VEC: channels % 4 == 0 and all
// pointers 16-byte aligned, one thread per 4 channels; otherwise one thread per element.
template <bool VEC>
__global__ void k_stitch(const float* x_obj, const float* x_bg,      // either may be `out` itself: no __restrict__
                         const uint8_t* __restrict__ m_obj, const uint8_t* __restrict__ m_bg, float* out,
                         long long pixels, int channels) {
  const int per_pixel = VEC ? channels / 4 : channels;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= pixels * per_pixel) return;
  const long long px = i / per_pixel;
  bool take = (m_obj[px >> 3] >> (px & 7)) & 1;
  if (m_bg) take = take || !((m_bg[px >> 3] >> (px & 7)) & 1);
  if (VEC) {
    ((f32x4*)out)[i] = take ? ((const f32x4*)x_obj)[i] : ((const f32x4*)x_bg)[i];
  } else {
    out[i] = take ? x_obj[i] : x_bg[i];
  }
}

hipError_t launch_stitch(const float* x_obj, const float* x_bg, const uint8_t* m_obj, const uint8_t* m_bg, float* out,
                         long long pixels, int channels, hipStream_t s) {
  if (pixels == 0) return hipSuccess;
  const bool vec = channels % 4 == 0 && (((uintptr_t)x_obj | (uintptr_t)x_bg | (uintptr_t)out) & 15) == 0;
  const long long n = pixels * (vec ? channels / 4 : channels);
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (vec) k_stitch<true><<<blocks, 256, 0, s>>>(x_obj, x_bg, m_obj, m_bg, out, pixels, channels);
  else k_stitch<false><<<blocks, 256, 0, s>>>(x_obj, x_bg, m_obj, m_bg, out, pixels, channels);
  return hipGetLastError();
}

// ---------------------------------------------------------------- expanding a compressed entry
// Frame t of the output comes from source code src[t]: 0 = the stored first frame,
// j >= 1 = first + alpha * diff_base[j-1], -(e+1) = extra frame e.  blockIdx.y = t.
struct DecompressSrc { int code[kMaxCacheFrames]; };

// V: f32x4 where frames are whole aligned 16-byte pieces, else float.
template <typename V>
__global__ void k_decompress(const float* __restrict__ first, const float* __restrict__ diff_base, float alpha,
                             const float* __restrict__ extra, DecompressSrc src, long long F, float* __restrict__ out) {
  constexpr int W = sizeof(V) / 4;
  const int t = blockIdx.y;
  const int code = src.code[t];
  const V* add = (const V*)(code > 0 ? diff_base + (size_t)(code - 1) * F : nullptr);
  const V* base = (const V*)(code < 0 ? extra + (size_t)(-code - 1) * F : first);
  V* o = (V*)(out + (size_t)t * F);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < F / W; i += (long long)gridDim.x * blockDim.x)
    o[i] = add ? base[i] + alpha * add[i] : base[i];
}

hipError_t launch_decompress(const float* first, const float* diff_base, float alpha, const float* extra,
                             const int* src_host, int T, long long F, float* out, hipStream_t s) {
  if (T == 0 || F == 0) return hipSuccess;
  DecompressSrc src;
  for (int t = 0; t < T; ++t) src.code[t] = src_host[t];
  const bool vec = F % 4 == 0 && (((uintptr_t)first | (uintptr_t)diff_base | (uintptr_t)extra | (uintptr_t)out) & 15) == 0;
  const long long pieces = ((vec ? F / 4 : F) + 255) / 256;
  const dim3 grid((unsigned)(pieces < 1024 ? pieces : 1024), T);
  // us a launch, a value and a 16-byte piece a thread: 64 frames of 10 240 2.8 and 2.5, of 86 400 9.9 and 7.1
  if (vec) k_decompress<f32x4><<<grid, 256, 0, s>>>(first, diff_base, alpha, extra, src, F, out);
  else k_decompress<float><<<grid, 256, 0, s>>>(first, diff_base, alpha, extra, src, F, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- reductions of the compressing side
// Deterministic two-pass sums in double: kRedBlocks partial results, then one block adds
// them in a fixed order.  No atomics.
constexpr int kRedBlocks = 256;

__device__ __forceinline__ double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  return t;
}

// partial[b] = { sum (keys_s - first_s) * diff_base, sum diff_base^2 } over block b's share
__global__ __launch_bounds__(256) void k_alpha_partial(const float* __restrict__ first_s, const float* __restrict__ keys_s,
                                                       const float* __restrict__ diff_base, long long F, long long total,
                                                       double* __restrict__ partial) {
  __shared__ double sh[4];
  double num = 0.0, den = 0.0;
  long long i = (long long)blockIdx.x * 256 + threadIdx.x, f = i % F;
  const long long hop = (long long)kRedBlocks * 256 % F;
  for (; i < total; i += (long long)kRedBlocks * 256) {
    const double db = diff_base[i];
    num += ((double)keys_s[i] - (double)first_s[f]) * db;
    den += db * db;
    f += hop;                                             // i % F
    if (f >= F) f -= F;
  }
  num = block_sum(num, sh);
  den = block_sum(den, sh);
  if (threadIdx.x == 0) { partial[2 * blockIdx.x] = num; partial[2 * blockIdx.x + 1] = den; }
}

// A lane per kRedBlocks / 64 partial results, then the wave's sum: one thread that read all 256 in turn took
// 5.6 us.
__global__ __launch_bounds__(64) void k_alpha_final(const double* __restrict__ partial, float* __restrict__ alpha_out) {
  double num = 0.0, den = 0.0;
#pragma unroll
  for (int b = 0; b < kRedBlocks / 64; ++b) {
    const int at = 2 * (threadIdx.x * (kRedBlocks / 64) + b);
    num += partial[at];
    den += partial[at + 1];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { num += __shfl_xor(num, o, 64); den += __shfl_xor(den, o, 64); }
  // Diff_base identically zero: every alpha fits equally well and the restored frames do not
  // depend on it; the minimum-norm choice is 0
  if (threadIdx.x == 0) alpha_out[0] = den > 0.0 ? (float)(num / den) : 0.0f;
}

hipError_t launch_alpha(const float* first_s, const float* keys_s, const float* diff_base, int n_base, long long F,
                        float* alpha_out, double* ws, hipStream_t s) {
  k_alpha_partial<<<kRedBlocks, 256, 0, s>>>(first_s, keys_s, diff_base, F, (long long)n_base * F, ws);
  k_alpha_final<<<1, 64, 0, s>>>(ws, alpha_out);
  return hipGetLastError();
}

// sim[i][j] = sim[j][i] = <frame i, frame j> / (|frame i| |frame j|) in double, rounded once.  A workgroup
// owns 4 x 4 pairs (J <= I): 16 dot products and the 8 norms from 8 frames' values, each read once and widened once,
// where a workgroup per pair read two frames for every dot product (64 frames of 10 240: 26 us and 4 for the
// division, now 6.6 in all).  Threads take the same values of every frame in order, so a frame's norm is the same number
// in whichever workgroup it is taken.  Few workgroups wait for memory: a trip has four values of each of the eight
// frames in flight, next to each other where frames are made of whole aligned 16-byte pieces, else 512 apart (32 frames
// of 86 401: 201 us with one value a trip, 95 in two launches of a workgroup per pair, 67 now; of 86 400: 33).
constexpr int kSimTile = 4, kSimThreads = 512, kSimValues = 4;

// in lanes whose bit LANES is 0, a + that of the partner (lane + LANES), in the others b + that of the partner
template <int LANES> __device__ __forceinline__ double halves_swap(double a, double b) {
  unsigned al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
  if constexpr (LANES == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap(al, bl, false, false), hi = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    al = lo[0]; bl = lo[1]; ah = hi[0]; bh = hi[1];
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap(al, bl, false, false), hi = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    al = lo[0]; bl = lo[1]; ah = hi[0]; bh = hi[1];
  }
  return __hiloint2double((int)ah, (int)al) + __hiloint2double((int)bh, (int)bl);
}
template <int CTRL> __device__ __forceinline__ double dpp64(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <bool VEC>
__global__ __launch_bounds__(kSimThreads) void k_frame_similarity(const float* __restrict__ frames, int T, long long F,
                                                                  float* __restrict__ sim) {
  const int I = blockIdx.y, J = blockIdx.x;
  if (J > I) return;
  const float* row[2 * kSimTile];
#pragma unroll
  for (int r = 0; r < kSimTile; ++r) {                    // rows past the end: the last one again, never stored
    row[r] = frames + (size_t)min(I * kSimTile + r, T - 1) * F;
    row[kSimTile + r] = frames + (size_t)min(J * kSimTile + r, T - 1) * F;
  }
  constexpr int NACC = kSimTile * kSimTile + 2 * kSimTile;
  double acc[32] = {};                                    // 16 products, 8 norms, 8 unused
  auto add = [&](auto& x, int n) {                        // n values of every row
#pragma unroll
    for (int c = 0; c < n; ++c) {
      double d[2 * kSimTile];
#pragma unroll
      for (int r = 0; r < 2 * kSimTile; ++r) d[r] = (double)x[r][c];
#pragma unroll
      for (int i = 0; i < kSimTile; ++i)
#pragma unroll
        for (int j = 0; j < kSimTile; ++j) acc[i * kSimTile + j] = __builtin_fma(d[i], d[kSimTile + j], acc[i * kSimTile + j]);
#pragma unroll
      for (int r = 0; r < 2 * kSimTile; ++r) acc[16 + r] = __builtin_fma(d[r], d[r], acc[16 + r]);
    }
  };
  constexpr long long kTrip = kSimThreads * kSimValues;
  long long e = 0;
  f32x4 x[2 * kSimTile];
  for (; e + kTrip <= F; e += kTrip) {
#pragma unroll
    for (int r = 0; r < 2 * kSimTile; ++r) {
      if constexpr (VEC) {
        x[r] = *(const f32x4*)(row[r] + e + threadIdx.x * kSimValues);
      } else {
#pragma unroll
        for (int c = 0; c < kSimValues; ++c) x[r][c] = row[r][e + c * kSimThreads + threadIdx.x];
      }
    }
    add(x, kSimValues);
  }
  for (e += threadIdx.x; e < F; e += kSimThreads) {       // the last part of a trip, a value at a time
#pragma unroll
    for (int r = 0; r < 2 * kSimTile; ++r) x[r][0] = row[r][e];
    add(x, 1);
  }
  // 32 sums over 64 lanes: a lane hands half of its sums to its partner and takes the other half, five
  // times (lane bits 5 .. 1 choose sum bits 4 .. 0; within eight lanes 7 - lane is the partner of the other quad); what is left of each sum is in two lanes.  All of it register to
  // register: the 62 trips through LDS that it took were 1.2 us of the 7.7 of 64 frames of 10 240, 5.1 -> 3.7 at 2048.
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = halves_swap<32>(acc[k], acc[k + 16]);
#pragma unroll
  for (int k = 0; k < 8; ++k) acc[k] = halves_swap<16>(acc[k], acc[k + 8]);
  auto trade = [&](auto pattern, int half, int bit) {
    const bool up = lane & bit;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const double mine = up ? acc[k + half] : acc[k], give = up ? acc[k] : acc[k + half];
      acc[k] = mine + dpp64<decltype(pattern)::value>(give);
    }
  };
  trade(std::integral_constant<int, 0x128>{}, 4, 8);      // lane ^ 8: a row of 16 turned by 8
  trade(std::integral_constant<int, 0x141>{}, 2, 4);      // 7 - lane in each 8: the other quad
  trade(std::integral_constant<int, 0x4E>{}, 1, 2);       // lane ^ 2
  acc[0] += dpp64<0xB1>(acc[0]);                          // lane ^ 1
  __shared__ double part[kSimThreads / 64][32], total[32];
  if (!(lane & 1)) part[wave][lane >> 1] = acc[0];
  __syncthreads();
  if (threadIdx.x < NACC) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kSimThreads / 64; ++w) t += part[w][threadIdx.x];
    total[threadIdx.x] = t;
  }
  __syncthreads();
  if (threadIdx.x < kSimTile * kSimTile) {
    const int a = threadIdx.x / kSimTile, b = threadIdx.x % kSimTile, i = I * kSimTile + a, j = J * kSimTile + b;
    if (i >= T || j >= T) return;
    const double n = sqrt(total[16 + a] * total[16 + kSimTile + b]);
    const float v = (float)(total[threadIdx.x] / (n > 1e-300 ? n : 1e-300));
    sim[(size_t)i * T + j] = v;
    if (I != J) sim[(size_t)j * T + i] = v;               // a tile on the diagonal holds both halves
  }
}

hipError_t launch_frame_similarity(const float* frames, int T, long long F, float* sim, hipStream_t s) {
  if (T == 0) return hipSuccess;
  const dim3 grid(ceil_div(T, kSimTile), ceil_div(T, kSimTile));
  if (F % 4 == 0 && ((uintptr_t)frames & 15) == 0) k_frame_similarity<true><<<grid, kSimThreads, 0, s>>>(frames, T, F, sim);
  else k_frame_similarity<false><<<grid, kSimThreads, 0, s>>>(frames, T, F, sim);
  return hipGetLastError();
}

// ---------------------------------------------------------------- plain copy (key-step export)
__global__ void k_copy_f32(const float* __restrict__ in, float* __restrict__ out, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[i];
}

hipError_t launch_copy_f32(const float* in, float* out, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_copy_f32<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(in, out, n);
  return hipGetLastError();
}

}  // namespace fc
