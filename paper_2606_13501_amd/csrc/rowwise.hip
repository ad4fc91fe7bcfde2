// Memory-bound kernels of the DiT block: LayerNorm with adaLN modulation or a
// shared affine, per-head RMSNorm with sectioned rotary embedding on q and k,
// the standalone gated residual, and the timestep-conditioning chain
// (sinusoid -> Linear-SiLU -> Linear-SiLU -> Linear to the modulation vectors).
//
// Every kernel moves 16-byte vectors per lane with consecutive lanes on
// consecutive addresses; a row is held in registers between its statistics
// pass and its output pass so it is read from HBM exactly once.  The rows are
// streamed with non-temporal loads and stores (each byte is touched once, so
// keeping it in the caches only displaces other data): measured +4-7% on the
// LayerNorm and gated-residual kernels at 75,600 x 5,120.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace dit {

namespace {

template <typename T> struct Vec16;
template <> struct Vec16<bf16> { typedef bf16x8 type; static constexpr int n = 8; };
template <> struct Vec16<float> { typedef f32x4 type; static constexpr int n = 4; };

// ------------------------------------------------------------ LayerNorm
// out = (x - mean) / sqrt(var + eps) * mul + add, one wave per row.
//   modulate: mul = 1 + scale[req], add = shift[req] (fp32 vectors)
//   affine:   mul = gamma, add = beta (dtype vectors)
// NVL = 16-byte vectors per lane, a compile-time count so the row is held in
// exactly as many registers as it needs (occupancy hides the HBM latency).

// Mean and 1 / sqrt(var + eps) of the wave's row v (NVL vectors per lane).
// The squares are accumulated with explicit fused multiply-adds, so every
// kernel that calls this rounds the statistics the same way.
template <typename T, int NVL, typename V>
__device__ __forceinline__ void row_stats(const V (&v)[NVL], int lane, int nv, int hidden, float eps, float& mean,
                                          float& rstd) {
  constexpr int VN = Vec16<T>::n;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NVL; ++i)
#pragma unroll
    for (int e = 0; e < VN; ++e) sum += to_f<T>(v[i][e]);
  mean = wave_sum(sum) / hidden;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NVL; ++i) {
    if (lane + 64 * i < nv) {
#pragma unroll
      for (int e = 0; e < VN; ++e) {
        const float d = to_f<T>(v[i][e]) - mean;
        sq = fmaf(d, d, sq);
      }
    }
  }
  rstd = rsqrtf(wave_sum(sq) / hidden + eps);
}

template <typename T, int NVL>
__global__ __launch_bounds__(256) void layer_norm_affine_kernel(
    const T* __restrict__ x, T* __restrict__ out, int64_t n_rows, int hidden, float eps,
    const T* __restrict__ gamma, const T* __restrict__ beta) {
  typedef typename Vec16<T>::type V;
  constexpr int VN = Vec16<T>::n;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int nv = hidden / VN;
  const T* xr = x + row * hidden;
  V v[NVL];
#pragma unroll
  for (int i = 0; i < NVL; ++i) {
    const int c = lane + 64 * i;
    v[i] = c < nv ? __builtin_nontemporal_load(reinterpret_cast<const V*>(xr + c * VN)) : V{};
  }
  float mean, rstd;
  row_stats<T, NVL>(v, lane, nv, hidden, eps, mean, rstd);
  T* orow = out + row * hidden;
#pragma unroll
  for (int i = 0; i < NVL; ++i) {
    const int c = lane + 64 * i;
    if (c < nv) {
      const V g = *reinterpret_cast<const V*>(gamma + c * VN);
      const V b = *reinterpret_cast<const V*>(beta + c * VN);
      V o;
#pragma unroll
      for (int e = 0; e < VN; ++e)
        o[e] = from_f<T>(fmaf((to_f<T>(v[i][e]) - mean) * rstd, to_f<T>(g[e]), to_f<T>(b[e])));
      __builtin_nontemporal_store(o, reinterpret_cast<V*>(orow + c * VN));
    }
  }
}

// Modulated LayerNorm, WAVES rows per workgroup.  When all of them belong to
// one request (every workgroup but those across a request boundary), the
// request's 1 + scale and shift are first staged in LDS as fp32 (8 bytes per
// column), so they are read from L2 once per workgroup rather than once per
// row: at 75,600 x 5,120 the per-row reads were 40 KB of L2 traffic for
// every 10 KB row, and staging took the kernel from 70% to 75% of the HBM
// peak.  The other workgroups read the vectors of each row's request
// directly; both paths round identically.  The row is loaded after the
// staging: issued before it, the row loads held the staged reads back
// behind them and the kernel ran 20% slower.
template <typename T, int NVL, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void layer_norm_mod_kernel(
    const T* __restrict__ x, T* __restrict__ out, int64_t n_rows, int hidden, float eps,
    const float* __restrict__ shift, const float* __restrict__ scale, int64_t mod_stride, ReqTable req) {
  typedef typename Vec16<T>::type V;
  constexpr int VN = Vec16<T>::n;
  // hidden / 4 vectors of 1 + scale, then hidden / 4 of shift.  Source vector
  // j = G c + g (G = VN / 4 per 16-byte row vector c) is kept at g nv + c, so
  // the 64 lanes of a read, and of a staging write, touch 64 consecutive
  // vectors (no bank conflicts).
  constexpr int G = VN / 4;
  extern __shared__ f32x4 smod[];
  const int lane = threadIdx.x & 63;
  const int64_t r0 = (int64_t)blockIdx.x * WAVES;
  const int64_t row = r0 + (threadIdx.x >> 6);
  const int ra = find_req(req.cu, req.n_req, (int)r0);
  const bool staged = ra == find_req(req.cu, req.n_req, (int)(min(r0 + WAVES, n_rows) - 1));
  const int nv = hidden / VN, h4 = hidden / 4;
  if (staged) {   // uniform over the workgroup
    const f32x4* sc = reinterpret_cast<const f32x4*>(scale + (int64_t)ra * mod_stride);
    const f32x4* sh = reinterpret_cast<const f32x4*>(shift + (int64_t)ra * mod_stride);
    for (int at = threadIdx.x; at < h4; at += WAVES * 64) {   // consecutive LDS writes
      const int i = G * (at % nv) + at / nv;
      f32x4 m = sc[i];
#pragma unroll
      for (int u = 0; u < 4; ++u) m[u] = 1.0f + m[u];
      smod[at] = m;
      smod[h4 + at] = sh[i];
    }
    __syncthreads();
  }
  if (row >= n_rows) return;
  V v[NVL];
  {
    const T* xr = x + row * hidden;
#pragma unroll
    for (int i = 0; i < NVL; ++i) {
      const int c = lane + 64 * i;
      v[i] = c < nv ? __builtin_nontemporal_load(reinterpret_cast<const V*>(xr + c * VN)) : V{};
    }
  }
  float mean, rstd;
  row_stats<T, NVL>(v, lane, nv, hidden, eps, mean, rstd);
  const int r = staged ? ra : find_req(req.cu, req.n_req, (int)row);
  const f32x4* sc = reinterpret_cast<const f32x4*>(scale + (int64_t)r * mod_stride);
  const f32x4* sh = reinterpret_cast<const f32x4*>(shift + (int64_t)r * mod_stride);
  T* orow = out + row * hidden;
  auto emit = [&](auto&& mul_add) {
#pragma unroll
    for (int i = 0; i < NVL; ++i) {
      const int c = lane + 64 * i;
      if (c < nv) {
        V o;
#pragma unroll
        for (int e = 0; e < VN; e += 4) {
          f32x4 m4, a4;
          mul_add((c * VN + e) / 4, m4, a4);
#pragma unroll
          for (int u = 0; u < 4; ++u)
            o[e + u] = from_f<T>(fmaf((to_f<T>(v[i][e + u]) - mean) * rstd, m4[u], a4[u]));
        }
        __builtin_nontemporal_store(o, reinterpret_cast<V*>(orow + c * VN));
      }
    }
  };
  if (staged) {
    emit([&](int j, f32x4& m4, f32x4& a4) {
      const int at = (j % G) * nv + j / G;
      m4 = smod[at];
      a4 = smod[h4 + at];
    });
  } else {
    emit([&](int j, f32x4& m4, f32x4& a4) {
      m4 = sc[j];
      a4 = sh[j];
#pragma unroll
      for (int u = 0; u < 4; ++u) m4[u] = 1.0f + m4[u];
    });
  }
}

// ---------------------------------------------------- QK RMSNorm + rotary
// One wave per row, four rows per 256-thread block.  A head of head_dim
// values is LPH = head_dim / VN consecutive lanes (LPH divides 64), so every
// vector a lane touches sits at the same offset inside its head: the lane
// needs the same VN/2 rotary pairs and the same gain vector for all of them.
// Lane j computes the cos/sin of pair j (in double) and the lanes gather
// theirs by shuffles; a head's RMS statistic is a shuffle reduction over its
// LPH lanes.  q and k vectors of a pass (NV per lane each) are all loaded
// before any is computed on.
template <typename T, int NV>
__global__ __launch_bounds__(256) void qk_norm_rope_kernel(
    T* q, T* k, int64_t row_stride, int64_t n_rows, int n_heads, int head_dim, const T* __restrict__ g_q,
    const T* __restrict__ g_k, float eps, int rope, int sec0, int sec1, int sec2, float theta,
    RopeTable tab) {
  typedef typename Vec16<T>::type V;
  constexpr int VN = Vec16<T>::n;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int lph = head_dim / VN;
  const int hc = lane % lph;          // chunk index inside the head
  const int cpt = n_heads * lph;      // vectors per tensor
  T* base_ptr[2] = {q + row * row_stride, k ? k + row * row_stride : nullptr};
  const T* gain[2] = {g_q, g_k};
  float cr[VN / 2], sr[VN / 2];
  if (rope) {
    float cj = 1.f, sj = 0.f;
    const int j = lane;
    if (j < head_dim / 2) {
      const int r = find_req(tab.cu, tab.n_req, (int)row);
      const int g = tab.offset[r] + (int)row - tab.cu[r];
      const int pt = g / tab.grid_hw[r];
      const int ph = (g / tab.grid_w[r]) % tab.grid_h[r];
      const int pw = g % tab.grid_w[r];
      // pair j -> (section, index inside the section)
      int p, js, ds;
      if (j < sec0 / 2) { p = pt; js = j; ds = sec0; }
      else if (j < (sec0 + sec1) / 2) { p = ph; js = j - sec0 / 2; ds = sec1; }
      else { p = pw; js = j - (sec0 + sec1) / 2; ds = sec2; }
      const double ang = (double)p * exp(-2.0 * js / ds * log((double)theta));
      double sn, cn;
      sincos(ang, &sn, &cn);
      cj = (float)cn;
      sj = (float)sn;
    }
#pragma unroll
    for (int u = 0; u < VN / 2; ++u) {
      cr[u] = __shfl(cj, hc * (VN / 2) + u, 64);
      sr[u] = __shfl(sj, hc * (VN / 2) + u, 64);
    }
  }
  const int n_t = k ? 2 : 1;
  for (int b0 = 0; b0 < cpt; b0 += 64 * NV) {
    V v[2][NV];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = b0 + lane + 64 * i;
        v[t][i] = t < n_t && c < cpt ? __builtin_nontemporal_load(reinterpret_cast<const V*>(base_ptr[t] + (int64_t)c * VN)) : V{};
      }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t >= n_t) break;
      V g{};
      if (gain[t]) g = *reinterpret_cast<const V*>(gain[t] + hc * VN);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        if (b0 + 64 * i >= cpt) break;   // wave-uniform
        const int c = b0 + lane + 64 * i;
        float f[VN];
#pragma unroll
        for (int e = 0; e < VN; ++e) f[e] = to_f<T>(v[t][i][e]);
        if (gain[t]) {
          float sq = 0.f;
#pragma unroll
          for (int e = 0; e < VN; ++e) sq += f[e] * f[e];
          for (int o = lph / 2; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
          const float rs = rsqrtf(sq / head_dim + eps);
#pragma unroll
          for (int e = 0; e < VN; ++e) f[e] = f[e] * rs * to_f<T>(g[e]);
        }
        if (rope) {
#pragma unroll
          for (int u = 0; u < VN / 2; ++u) {
            const float a = f[2 * u], bb = f[2 * u + 1];
            f[2 * u] = a * cr[u] - bb * sr[u];
            f[2 * u + 1] = a * sr[u] + bb * cr[u];
          }
        }
        if (c < cpt) {
          V o;
#pragma unroll
          for (int e = 0; e < VN; ++e) o[e] = from_f<T>(f[e]);
          __builtin_nontemporal_store(o, reinterpret_cast<V*>(base_ptr[t] + (int64_t)c * VN));
        }
      }
    }
  }
}

// ------------------------------------------------------- gated residual
// out = x + gate[req] * (z + bias), one wave per row; the row's x and z
// vectors (NVL per lane) are all loaded before any is combined.
template <typename T, int NVL>
__global__ __launch_bounds__(256) void gated_residual_kernel(
    const T* x, const T* z, const T* __restrict__ bias, const float* __restrict__ gate,
    int64_t gate_stride, T* out, int64_t n_rows, int hidden, ReqTable req) {
  typedef typename Vec16<T>::type V;
  constexpr int VN = Vec16<T>::n;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int r = find_req(req.cu, req.n_req, (int)row);
  const float* g = gate + (int64_t)r * gate_stride;
  const int nv = hidden / VN;
  V xv[NVL], zv[NVL];
#pragma unroll
  for (int i = 0; i < NVL; ++i) {
    const int c = lane + 64 * i;
    xv[i] = c < nv ? __builtin_nontemporal_load(reinterpret_cast<const V*>(x + row * hidden + c * VN)) : V{};
    zv[i] = c < nv ? __builtin_nontemporal_load(reinterpret_cast<const V*>(z + row * hidden + c * VN)) : V{};
  }
#pragma unroll
  for (int i = 0; i < NVL; ++i) {
    const int c = lane + 64 * i;
    if (c < nv) {
      V bv{};
      if (bias) bv = *reinterpret_cast<const V*>(bias + c * VN);
      V o;
#pragma unroll
      for (int e = 0; e < VN; e += 4) {
        f32x4 g4 = *reinterpret_cast<const f32x4*>(g + c * VN + e);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          o[e + u] = from_f<T>(to_f<T>(xv[i][e + u]) + g4[u] * (to_f<T>(zv[i][e + u]) + to_f<T>(bv[e + u])));
      }
      __builtin_nontemporal_store(o, reinterpret_cast<V*>(out + row * hidden + c * VN));
    }
  }
}

// ------------------------------------------------------- conditioning
// The vectors that are inputs of a Linear of the chain are kept in an order in
// which its lanes read them in whole lines: in every whole group of 64 VN
// values (VN weights per 16-byte vector, one vector per lane), value
// VN lane + 4 h + j lies at 256 h + 4 lane + j.  With bf16 weights a lane
// needs 8 consecutive fp32 inputs, and its two 16-byte loads would each skip
// every other 16 bytes.  (fp32 weights, and the values after the last whole
// group: the plain order.)
template <typename T>
__device__ __forceinline__ int cond_at(int i, int n) {
  constexpr int VN = Vec16<T>::n, G = 64 * VN;
  if (VN == 4 || i - i % G + G > n) return i;
  const int k = i % G;
  return i - k + 256 * (k % VN / 4) + k / VN * 4 + k % 4;
}

// e[r] = [cos(t w_i), sin(t w_i)], w_i = 10000^(-i/half); computed in double.
template <typename T>
__global__ void timestep_embed_kernel(const float* __restrict__ t, float* __restrict__ e, int n_req,
                                      int freq_dim) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int half = freq_dim / 2;
  if (idx >= n_req * half) return;
  const int r = idx / half, i = idx - r * half;
  const double w = exp(-log(10000.0) * (double)i / (double)half);
  double sn, cn;
  sincos((double)t[r] * w, &sn, &cn);
  e[(int64_t)r * freq_dim + cond_at<T>(i, freq_dim)] = (float)cn;
  e[(int64_t)r * freq_dim + cond_at<T>(half + i, freq_dim)] = (float)sn;
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

// Sums of N values (a power of two up to 64) over the wave, all at once: lane
// l gets the sum of v[i], i the top log2(N) bits of l (so 64 / N lanes hold
// the same).  Each halving step exchanges half of the remaining values with
// the lane `o` away, so N sums take about N exchanges instead of 6 N; the
// pairs added are those of wave_sum, so the bits are the same.
template <int N, int O = 32>
__device__ __forceinline__ float wave_sums(float (&v)[N]) {
  if constexpr (O == 0) {
    return v[0];
  } else if constexpr (N == 1) {
    float w[1] = {v[0] + __shfl_xor(v[0], O, kWave)};
    return wave_sums<1, O / 2>(w);
  } else {
    float w[N / 2];
    const bool up = threadIdx.x & O;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      if constexpr (O == 32) {
        // swaps the upper half of the first with the lower half of the second
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + N / 2]), false, false);
        w[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      } else if constexpr (O == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + N / 2]), false, false);
        w[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      } else {
        w[i] = (up ? v[i + N / 2] : v[i]) + __shfl_xor(up ? v[i] : v[i + N / 2], O, kWave);
      }
    }
    return wave_sums<N / 2, O / 2>(w);
  }
}

// y[r][o] = act(sum_i W[o][i] x[r][i] + b[o]), x and y fp32.  The weights bound
// the time for few requests (the adaLN projection of one request at 30,720 x
// 5,120 bf16, 315 MB: 52.6 us, 6.0 TB/s); they are read once per RB requests
// (from the caches after the first time, where they fit).  A wave computes
// ROWS outputs for up to RB requests, so the inputs it reads from the caches
// (4 bytes per 2 of bf16 weights, request and wave) serve ROWS rows, and the
// sums over the wave are taken all at once.  With a row per wave and a tree
// per sum those took more time than the weights: 62.9 us for one request,
// 147.7 for six (now 78.1).  Two vectors of every row are in flight per lane.
// A lane sums its vectors of a row in order, the lanes meet in a tree: the
// same bits for every ROWS and RB, and as gemv_row_kernel.
//
// REST: code of its own for what is left over, i.e. a last group of at most 4
// requests (instead of its last request repeated up to RB) and the whole
// groups of 64 vectors after the last pair.  It costs registers, so it is used
// where it pays (see launch_gemv).
template <typename T, bool SILU_OUT, int ROWS, int RB, bool REST>
__global__ __launch_bounds__(256) void gemv_kernel(const T* __restrict__ W, const T* __restrict__ b,
                                                   const float* __restrict__ x, float* __restrict__ y,
                                                   int n_out, int n_in, int n_req) {
  typedef typename Vec16<T>::type V;
  constexpr int VN = Vec16<T>::n;
  typedef float fxv __attribute__((ext_vector_type(VN)));
  const int lane = threadIdx.x & 63;
  const int o0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * ROWS;
  if (o0 >= n_out) return;
  const int nv = n_in / VN;
  const T* wr[ROWS];   // rows past the last output repeat it
#pragma unroll
  for (int n = 0; n < ROWS; ++n) wr[n] = W + (int64_t)min(o0 + n, n_out - 1) * n_in;
  // requests r0 .. r0 + nr - 1, nr at most `size`
  auto group = [&](int r0, int nr, auto size) __attribute__((always_inline)) {
    constexpr int G = decltype(size)::value;
    float acc[ROWS][G] = {};
    // the vectors from c0 on, `steps` groups of 64.  FULL: every lane has its
    // vector (no per-lane tests, so the loads are not split by branches)
    auto run = [&](int c0, int n_vec, auto steps, auto full) __attribute__((always_inline)) {
      constexpr int S = decltype(steps)::value;
      constexpr bool kFull = decltype(full)::value;
      V wv[S][ROWS];
#pragma unroll
      for (int h = 0; h < S; ++h)
#pragma unroll
        for (int n = 0; n < ROWS; ++n) {
          const int c = c0 + 64 * h + lane;
          if (kFull || c < n_vec) wv[h][n] = *reinterpret_cast<const V*>(wr[n] + (int64_t)c * VN);
        }
#pragma unroll
      for (int h = 0; h < S; ++h) {
        const int c = c0 + 64 * h + lane;
        fxv xv[G];
#pragma unroll
        for (int rr = 0; rr < G; ++rr) {   // requests past the last one repeat it
          const float* xr = x + (int64_t)(r0 + min(rr, nr - 1)) * n_in;
          if (VN == 8 && (kFull || c0 + 64 * h + 64 <= n_vec)) {   // a whole group, in the order of cond_at
            const f32x4 lo = *reinterpret_cast<const f32x4*>(xr + (c0 + 64 * h) * VN + 4 * lane);
            const f32x4 hi = *reinterpret_cast<const f32x4*>(xr + (c0 + 64 * h) * VN + 256 + 4 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              xv[rr][e] = lo[e];
              xv[rr][VN - 4 + e] = hi[e];
            }
          } else if (kFull || c < n_vec) {
            xv[rr] = *reinterpret_cast<const fxv*>(xr + (int64_t)c * VN);
          }
        }
        if (kFull || c < n_vec) {
#pragma unroll
          for (int n = 0; n < ROWS; ++n)
#pragma unroll
            for (int rr = 0; rr < G; ++rr)
#pragma unroll
              for (int e = 0; e < VN; ++e) acc[n][rr] = fmaf(to_f<T>(wv[h][n][e]), xv[rr][e], acc[n][rr]);
        }
      }
    };
    constexpr std::integral_constant<int, 2> kTwo{};
    constexpr std::integral_constant<int, 1> kOne{};
    int c0 = 0;
    for (; c0 + 128 <= nv; c0 += 128) run(c0, nv, kTwo, std::true_type{});
    if constexpr (REST) {
      for (; c0 + 64 <= nv; c0 += 64) run(c0, nv, kOne, std::true_type{});
      if (c0 < nv) run(c0, nv, kOne, std::false_type{});
    } else {
      if (c0 < nv) run(c0, nv, kTwo, std::false_type{});
    }
    constexpr int N = ROWS * G;
    float v[N];
#pragma unroll
    for (int n = 0; n < ROWS; ++n)
#pragma unroll
      for (int rr = 0; rr < G; ++rr) v[n * G + rr] = acc[n][rr];
    float s = wave_sums<N>(v);
    const int n = lane / (64 / N) / G, rr = lane / (64 / N) % G, o = o0 + n;
    if (lane % (64 / N) == 0 && rr < nr && o < n_out) {
      s += b ? to_f<T>(b[o]) : 0.f;
      // (with SiLU: an input of the next Linear)
      y[(int64_t)(r0 + rr) * n_out + (SILU_OUT ? cond_at<T>(o, n_out) : o)] = SILU_OUT ? silu(s) : s;
    }
  };
  for (int r0 = 0; r0 < n_req; r0 += RB) {
    const int nr = min(RB, n_req - r0);
    if constexpr (REST && RB == 8) {
      if (nr == 1) { group(r0, nr, std::integral_constant<int, 1>{}); break; }
      if (nr == 2) { group(r0, nr, std::integral_constant<int, 2>{}); break; }
      if (nr <= 4) { group(r0, nr, std::integral_constant<int, 4>{}); break; }
    }
    group(r0, nr, std::integral_constant<int, RB>{});
  }
}

// The same product with a row per wave, for rows of at most 64 NVL vectors: a
// lane loads all of its NVL weight vectors first, so that they are in flight
// together, then each request's inputs, all at once.  A Linear of few outputs
// has too few waves for several rows per wave, and one request's Linear of a
// few microseconds waits for its loads once instead of once per two vectors.
// All groups of 64 vectors but the last are whole, so only that one is tested
// per lane: with a test of every group the loads are split by branches (the
// bf16 chain of one request at D = 640 11.3 us, now 10.1; at 768 11.0, 10.1).
template <typename T, bool SILU_OUT, int NVL>
__global__ __launch_bounds__(256) void gemv_row_kernel(const T* __restrict__ W, const T* __restrict__ b,
                                                       const float* __restrict__ x, float* __restrict__ y,
                                                       int n_out, int n_in, int n_req) {
  typedef typename Vec16<T>::type V;
  constexpr int VN = Vec16<T>::n;
  typedef float fxv __attribute__((ext_vector_type(VN)));
  const int lane = threadIdx.x & 63;
  const int o = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (o >= n_out) return;
  const T* wr = W + (int64_t)o * n_in;
  const int nv = n_in / VN;
  const float bo = b ? to_f<T>(b[o]) : 0.f;
  auto run = [&](auto full) __attribute__((always_inline)) {   // FULL: as in gemv_kernel
    constexpr bool kFull = decltype(full)::value;
    V wv[NVL];
#pragma unroll
    for (int u = 0; u < NVL; ++u) {
      const int c = lane + 64 * u;
      if (kFull || u < NVL - 1 || c < nv) wv[u] = *reinterpret_cast<const V*>(wr + c * VN);
    }
    for (int r = 0; r < n_req; ++r) {
      const float* xr = x + (int64_t)r * n_in;
      fxv xv[NVL];
#pragma unroll
      for (int u = 0; u < NVL; ++u) {
        const int c = lane + 64 * u;
        if (VN == 8 && (kFull || u < NVL - 1)) {   // a whole group, in the order of cond_at
          const f32x4 lo = *reinterpret_cast<const f32x4*>(xr + 64 * u * VN + 4 * lane);
          const f32x4 hi = *reinterpret_cast<const f32x4*>(xr + 64 * u * VN + 256 + 4 * lane);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            xv[u][e] = lo[e];
            xv[u][VN - 4 + e] = hi[e];
          }
        } else if (kFull || u < NVL - 1 || c < nv) {
          xv[u] = *reinterpret_cast<const fxv*>(xr + c * VN);
        }
      }
      float acc = 0.f;
#pragma unroll
      for (int u = 0; u < NVL; ++u)
        if (kFull || u < NVL - 1 || lane + 64 * u < nv) {
#pragma unroll
          for (int e = 0; e < VN; ++e) acc = fmaf(to_f<T>(wv[u][e]), xv[u][e], acc);
        }
      float sum = wave_sum(acc);
      if (lane == 0) {
        sum += bo;
        y[(int64_t)r * n_out + (SILU_OUT ? cond_at<T>(o, n_out) : o)] = SILU_OUT ? silu(sum) : sum;
      }
    }
  };
  if (nv == 64 * NVL) run(std::true_type{});
  else run(std::false_type{});
}

template <typename T, bool SILU_OUT>
bool launch_gemv_row(const T* W, const T* b, const float* x, float* y, int n_out, int n_in, int n_req, hipStream_t s) {
  const unsigned grid = (unsigned)((n_out + 3) / 4);
  switch ((n_in / Vec16<T>::n + 63) / 64) {
#define DIT_GEMV_ROW(NVL) \
  case NVL: gemv_row_kernel<T, SILU_OUT, NVL><<<grid, 256, 0, s>>>(W, b, x, y, n_out, n_in, n_req); return true;
    DIT_GEMV_ROW(1) DIT_GEMV_ROW(2) DIT_GEMV_ROW(3) DIT_GEMV_ROW(4) DIT_GEMV_ROW(5) DIT_GEMV_ROW(6)
    DIT_GEMV_ROW(7) DIT_GEMV_ROW(8) DIT_GEMV_ROW(9) DIT_GEMV_ROW(10) DIT_GEMV_ROW(11) DIT_GEMV_ROW(12)
    DIT_GEMV_ROW(13) DIT_GEMV_ROW(14) DIT_GEMV_ROW(15) DIT_GEMV_ROW(16)
#undef DIT_GEMV_ROW
    default: return false;
  }
}

// Which form, from the whole chain (two Linears D x D and one 6D x D) and the
// single Linears timed against each other, in us:
//  - one row per wave (gemv_row_kernel): one request, of fp32 weights (D = 384
//    9.1, with 2 and 4 rows 10.4; D = 4,096 94 against 115) or of a short bf16
//    Linear (D = 128 9.2, else 9.9); and the short fp32 ones of two requests
//    from 2,048 inputs on (3.8 against 4.1) and of three from 384 (D = 1,024
//    15.4 against 18.6).  At n_out = 2,048 in bf16 it no longer wins (the
//    chain 20.3 against 19.7).
//  - few outputs (below 2,048 for bf16, up to 2,048 for fp32): 2 rows, since 4
//    leave less than a wave per two SIMDs; with REST (nine requests at 1,536 x
//    1,536 5.5 against 6.4 us without, and against 9.9 with 4 rows).  From
//    3,072 on 4 rows win (three requests 5.3 against 5.8).
//  - one or two requests: 2 rows up to 8,192 outputs, where more waves count
//    (12.2 against 13.3 at 5,120 x 5,120), else 4.
//  - more: 4 rows; 8 where the reads of x bound it, for 5 and more requests
//    from 28,672 outputs on (6 requests, 4 and 8 rows, weights from the caches:
//    24,576 x 4,096 39.8 and 54.2, 27,648 x 4,608 47.3 and 53.4, 29,184 x 4,864
//    71.5 and 65.5, 30,720 x 5,120 81.8 and 73.7; weights from memory: 55.0 and
//    61.2, 69.9 and 68.2, 81.9 and 73.5, 85.6 and 77.1).
//  - fp32 with a small last group and up to 2,048 inputs: REST (nine requests
//    at D = 1,024 22.7 against 30.9); with larger weights its registers cost
//    more than the repeated requests (33 at D = 3,072: 345 against 274).
template <typename T, bool SILU_OUT>
void launch_gemv(const T* W, const T* b, const float* x, float* y, int n_out, int n_in, int n_req, hipStream_t s) {
  constexpr bool f32 = sizeof(T) == 4;
  const bool few = f32 ? n_out <= 2048 : n_out < 2048;
  const bool row = n_req == 1 ? f32 || few : f32 && few && (n_req == 2 ? n_in >= 2048 : n_req == 3 && n_in >= 384);
  if (row && launch_gemv_row<T, SILU_OUT>(W, b, x, y, n_out, n_in, n_req, s)) return;
  auto grid = [&](int rows) { return (unsigned)((n_out + 4 * rows - 1) / (4 * rows)); };
#define DIT_GEMV(ROWS, RB, REST) \
  gemv_kernel<T, SILU_OUT, ROWS, RB, REST><<<grid(ROWS), 256, 0, s>>>(W, b, x, y, n_out, n_in, n_req)
  if (few) {
    if (n_req == 1) DIT_GEMV(2, 1, true);
    else if (n_req == 2) DIT_GEMV(2, 2, true);
    else if (n_req <= 4) DIT_GEMV(2, 4, true);
    else DIT_GEMV(2, 8, true);
  } else if (n_req <= 2) {
    if (n_out <= 8192) {
      if (n_req == 1) DIT_GEMV(2, 1, false);
      else DIT_GEMV(2, 2, false);
    } else {
      if (n_req == 1) DIT_GEMV(4, 1, false);
      else DIT_GEMV(4, 2, false);
    }
  } else if (n_req <= 4) {
    DIT_GEMV(4, 4, false);
  } else if (f32 && n_in <= 2048 && n_req > 8 && (n_req - 1) % 8 < 4) {
    DIT_GEMV(4, 8, true);
  } else if (n_out >= 28672) {
    DIT_GEMV(8, 8, false);
  } else {
    DIT_GEMV(4, 8, false);
  }
#undef DIT_GEMV
}

template <typename T, int NVL>
hipError_t gres_nvl(const GatedResArgs& p, hipStream_t s) {
  gated_residual_kernel<T, NVL><<<(unsigned)((p.n_rows + 3) / 4), 256, 0, s>>>(
      (const T*)p.x, (const T*)p.z, (const T*)p.bias, p.gate, p.gate_stride, (T*)p.out, p.n_rows, p.hidden,
      p.req);
  return hipGetLastError();
}

// Rows of up to 1024 16-byte vectors (8192 bf16, 4096 fp32 values).
template <typename T>
hipError_t gres_typed(const GatedResArgs& p, hipStream_t s) {
  switch ((p.hidden / Vec16<T>::n + 63) / 64) {
    case 1: return gres_nvl<T, 1>(p, s);
    case 2: return gres_nvl<T, 2>(p, s);
    case 3: case 4: return gres_nvl<T, 4>(p, s);
    case 5: case 6: return gres_nvl<T, 6>(p, s);
    case 7: case 8: return gres_nvl<T, 8>(p, s);
    case 9: case 10: return gres_nvl<T, 10>(p, s);
    case 11: case 12: return gres_nvl<T, 12>(p, s);
    case 13: case 14: case 15: case 16: return gres_nvl<T, 16>(p, s);
    default: return hipErrorInvalidValue;
  }
}

constexpr int kLnModWaves = 4;   // rows of the modulated LayerNorm per workgroup

template <typename T, int NVL>
hipError_t ln_nvl(const LnArgs& p, hipStream_t s) {
  if (p.affine) {
    layer_norm_affine_kernel<T, NVL><<<(unsigned)((p.n_rows + 3) / 4), 256, 0, s>>>(
        (const T*)p.x, (T*)p.out, p.n_rows, p.hidden, p.eps, (const T*)p.gamma, (const T*)p.beta);
  } else {
    layer_norm_mod_kernel<T, NVL, kLnModWaves>
        <<<(unsigned)((p.n_rows + kLnModWaves - 1) / kLnModWaves), kLnModWaves * 64, (size_t)p.hidden * 8, s>>>(
            (const T*)p.x, (T*)p.out, p.n_rows, p.hidden, p.eps, p.shift, p.scale, p.mod_stride, p.req);
  }
  return hipGetLastError();
}

// Rows of up to 1024 16-byte vectors (8192 bf16, 4096 fp32 values).
template <typename T>
hipError_t ln_typed(const LnArgs& p, hipStream_t s) {
  const int nvl = (p.hidden / Vec16<T>::n + 63) / 64;
  switch (nvl) {
    case 1: return ln_nvl<T, 1>(p, s);
    case 2: return ln_nvl<T, 2>(p, s);
    case 3: return ln_nvl<T, 3>(p, s);
    case 4: return ln_nvl<T, 4>(p, s);
    case 5: return ln_nvl<T, 5>(p, s);
    case 6: return ln_nvl<T, 6>(p, s);
    case 7: return ln_nvl<T, 7>(p, s);
    case 8: return ln_nvl<T, 8>(p, s);
    case 9: case 10: return ln_nvl<T, 10>(p, s);
    case 11: case 12: return ln_nvl<T, 12>(p, s);
    case 13: case 14: return ln_nvl<T, 14>(p, s);
    case 15: case 16: return ln_nvl<T, 16>(p, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t cond_typed(const CondArgs& p, hipStream_t s) {
  if (p.w_t1) {
    const int half = p.freq_dim / 2;
    timestep_embed_kernel<T><<<(p.n_req * half + 255) / 256, 256, 0, s>>>(p.t, p.e, p.n_req, p.freq_dim);
    launch_gemv<T, true>((const T*)p.w_t1, (const T*)p.b_t1, p.e, p.a1, p.hidden, p.freq_dim, p.n_req, s);
    launch_gemv<T, true>((const T*)p.w_t2, (const T*)p.b_t2, p.a1, p.c, p.hidden, p.hidden, p.n_req, s);
  }
  if (p.w_ada) {
    const int n_out = p.n_mod * p.hidden;
    launch_gemv<T, false>((const T*)p.w_ada, (const T*)p.b_ada, p.c, p.mod, n_out, p.hidden, p.n_req, s);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_layer_norm(const LnArgs& p, hipStream_t s) {
  if (p.n_rows == 0) return hipSuccess;
  return p.dtype == DIT_BF16 ? ln_typed<bf16>(p, s) : ln_typed<float>(p, s);
}

namespace {

template <typename T, int NV>
void qk_nv(const NormRopeArgs& p, hipStream_t s) {
  qk_norm_rope_kernel<T, NV><<<(unsigned)((p.n_rows + 3) / 4), 256, 0, s>>>(
      (T*)p.q, (T*)p.k, p.row_stride, p.n_rows, p.n_heads, p.head_dim, (const T*)p.g_q, (const T*)p.g_k,
      p.eps, p.rope, p.sections[0], p.sections[1], p.sections[2], p.theta, p.tab);
}

template <typename T>
hipError_t qk_typed(const NormRopeArgs& p, hipStream_t s) {
  const int64_t nv = ((int64_t)p.n_heads * p.head_dim / Vec16<T>::n + 63) / 64;
  if (nv <= 1) qk_nv<T, 1>(p, s);
  else if (nv <= 2) qk_nv<T, 2>(p, s);
  else if (nv <= 3) qk_nv<T, 3>(p, s);
  else if (nv <= 4) qk_nv<T, 4>(p, s);
  else if (nv <= 6) qk_nv<T, 6>(p, s);
  else if (nv <= 8) qk_nv<T, 8>(p, s);
  else qk_nv<T, 10>(p, s);   // passes of 10 vectors per lane and tensor
  return hipGetLastError();
}

}  // namespace

hipError_t launch_qk_norm_rope(const NormRopeArgs& p, hipStream_t s) {
  if (p.n_rows == 0) return hipSuccess;
  return p.dtype == DIT_BF16 ? qk_typed<bf16>(p, s) : qk_typed<float>(p, s);
}

hipError_t launch_gated_residual(const GatedResArgs& p, hipStream_t s) {
  if (p.n_rows == 0) return hipSuccess;
  return p.dtype == DIT_BF16 ? gres_typed<bf16>(p, s) : gres_typed<float>(p, s);
}

hipError_t launch_conditioning(const CondArgs& p, hipStream_t s) {
  if (p.n_req == 0) return hipSuccess;
  return p.dtype == DIT_BF16 ? cond_typed<bf16>(p, s) : cond_typed<float>(p, s);
}

}  // namespace dit
