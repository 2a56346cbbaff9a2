// Token-local and per-step kernels of the DiT band step:
//   adaLN LayerNorm (LN without affine, then x(1 + scale) + shift),
//   conditioning (sinusoidal timestep MLP + label table -> adaLN vectors of
//   every block in one weight-streaming GEMV),
//   patch embedding of the band rows (+ the fixed position table),
//   final linear + unpatchify,
//   guidance + the scheduler update of §I (Lemma 1's eps coefficient).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace orch {

// ---------------------------------------------------------------------------
// adaLN LayerNorm: one wave per row, the row held in registers as float2
// (hidden % 128 == 0, hidden <= 2048).  The statistics are shifted sums
// sum(x - x0), sum((x - x0)^2) with x0 the row's first element (stable
// against a large mean), reduced together in one pass; shift and scale are
// loaded with the row, and the output is written as packed pairs.
template <typename T> struct Pair;
template <> struct Pair<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct Pair<bf16> { typedef __bf16 type __attribute__((ext_vector_type(2))); };

template <typename T>
__global__ __launch_bounds__(256) void ln_mod_kernel(const float* __restrict__ x, int rows, int H,
                                                     int rpb, const float* __restrict__ shift,
                                                     const float* __restrict__ scale,
                                                     int mod_stride, T* __restrict__ out) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int nv = H >> 7;
  const int b = row / rpb;
  const float2* xr = reinterpret_cast<const float2*>(x + (size_t)row * H);
  const float2* shr = reinterpret_cast<const float2*>(shift + (size_t)b * mod_stride);
  const float2* scr = reinterpret_cast<const float2*>(scale + (size_t)b * mod_stride);
  float2 v[16], sh[16], sc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (i < nv) {
      v[i] = xr[lane + 64 * i];
      sh[i] = shr[lane + 64 * i];
      sc[i] = scr[lane + 64 * i];
    }
  const float x0 = __shfl(v[0].x, 0, kWave);
  float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (i < nv) {
      const float a = v[i].x - x0, c = v[i].y - x0;
      s1 += a + c;
      s2 += a * a + c * c;
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s1 += __shfl_xor(s1, o, kWave);
    s2 += __shfl_xor(s2, o, kWave);
  }
  const float inv_h = 1.0f / (float)H;
  const float dmean = s1 * inv_h;
  const float var = fmaxf(s2 * inv_h - dmean * dmean, 0.0f);
  const float mean = x0 + dmean;
  const float rstd = 1.0f / sqrtf(var + 1e-6f);
  typedef typename Pair<T>::type P;
  P* o = reinterpret_cast<P*>(out + (size_t)row * H);
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (i < nv) {
      P w;
      w[0] = from_f<T>((v[i].x - mean) * rstd * (1.0f + sc[i].x) + sh[i].x);
      w[1] = from_f<T>((v[i].y - mean) * rstd * (1.0f + sc[i].y) + sh[i].y);
      o[lane + 64 * i] = w;
    }
}

// The same for a compile-time row length: two rows per wave (32 lanes each),
// 16-byte loads, NV float4 per lane (H = 128 NV).
template <typename T, int NV>
__global__ __launch_bounds__(256) void ln_mod_fixed_kernel(const float* __restrict__ x, int rows,
                                                           int rpb, const float* __restrict__ shift,
                                                           const float* __restrict__ scale,
                                                           int mod_stride, T* __restrict__ out) {
  constexpr int H = 128 * NV;
  const int row = blockIdx.x * 8 + (threadIdx.x >> 5);
  const int lane = threadIdx.x & 31;
  if (row >= rows) return;
  const int b = row / rpb;
  const float4* xr = reinterpret_cast<const float4*>(x + (size_t)row * H);
  const float4* shr = reinterpret_cast<const float4*>(shift + (size_t)b * mod_stride);
  const float4* scr = reinterpret_cast<const float4*>(scale + (size_t)b * mod_stride);
  float4 v[NV], sh[NV], sc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = xr[lane + 32 * i];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    sh[i] = shr[lane + 32 * i];
    sc[i] = scr[lane + 32 * i];
  }
  const float x0 = __shfl(v[0].x, 0, 32);
  float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const float a = v[i].x - x0, c = v[i].y - x0, d = v[i].z - x0, e = v[i].w - x0;
    s1 += (a + c) + (d + e);
    s2 += (a * a + c * c) + (d * d + e * e);
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    s1 += __shfl_xor(s1, o, 32);
    s2 += __shfl_xor(s2, o, 32);
  }
  constexpr float inv_h = 1.0f / (float)H;
  const float dmean = s1 * inv_h;
  const float var = fmaxf(s2 * inv_h - dmean * dmean, 0.0f);
  const float mean = x0 + dmean;
  const float rstd = 1.0f / sqrtf(var + 1e-6f);
  typedef T Q __attribute__((ext_vector_type(4)));
  Q* o = reinterpret_cast<Q*>(out + (size_t)row * H);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    Q w;
    w[0] = from_f<T>((v[i].x - mean) * rstd * (1.0f + sc[i].x) + sh[i].x);
    w[1] = from_f<T>((v[i].y - mean) * rstd * (1.0f + sc[i].y) + sh[i].y);
    w[2] = from_f<T>((v[i].z - mean) * rstd * (1.0f + sc[i].z) + sh[i].z);
    w[3] = from_f<T>((v[i].w - mean) * rstd * (1.0f + sc[i].w) + sh[i].w);
    o[lane + 32 * i] = w;
  }
}

template <typename T>
static void launch_ln_t(const float* x, int rows, int hidden, int rpb, const float* shift,
                        const float* scale, int mod_stride, T* out, hipStream_t s) {
  const bool al = ((uintptr_t)shift % 16 == 0) && ((uintptr_t)scale % 16 == 0) && mod_stride % 4 == 0;
  if (al && hidden == 1152) {
    hipLaunchKernelGGL((ln_mod_fixed_kernel<T, 9>), dim3(ceil_div(rows, 8)), dim3(256), 0, s, x,
                       rows, rpb, shift, scale, mod_stride, out);
  } else if (al && hidden == 384) {
    hipLaunchKernelGGL((ln_mod_fixed_kernel<T, 3>), dim3(ceil_div(rows, 8)), dim3(256), 0, s, x,
                       rows, rpb, shift, scale, mod_stride, out);
  } else {
    hipLaunchKernelGGL(ln_mod_kernel<T>, dim3(ceil_div(rows, 4)), dim3(256), 0, s, x, rows,
                       hidden, rpb, shift, scale, mod_stride, out);
  }
}

hipError_t launch_layernorm_modulate(const float* x, int rows, int hidden, int rpb,
                                     const float* shift, const float* scale, int mod_stride,
                                     void* out, int dtype, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (hidden % 128 != 0 || hidden > 2048) return hipErrorInvalidValue;
  if (dtype == kBF16)
    launch_ln_t<bf16>(x, rows, hidden, rpb, shift, scale, mod_stride, reinterpret_cast<bf16*>(out), s);
  else
    launch_ln_t<float>(x, rows, hidden, rpb, shift, scale, mod_stride, reinterpret_cast<float*>(out), s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Conditioning.
// 16 bytes of T as floats
template <typename T>
__device__ __forceinline__ void unpack16(const uint4& q, float* v) {
  const unsigned w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (sizeof(T) == 2) {
      v[2 * e] = __uint_as_float(w[e] << 16);
      v[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
    } else {
      v[e] = __uint_as_float(w[e]);
    }
  }
}

// t1[n] = SiLU(W1[n] . sinusoid(t) + b1[n]); sinusoid = [cos(t f_i), sin(t f_i)],
// f_i = 10000^(-i/half), evaluated in double.  One wave per output row, four rows
// a workgroup, whose threads share the sinusoid's evaluation (each wave for
// itself: 5.6 us at hidden 1152, now 4.9).
constexpr int kSinusoid = 1024;    // values held at a time

template <typename T>
__global__ __launch_bounds__(256) void temb1_kernel(const T* __restrict__ w1,
                                                    const float* __restrict__ b1, float t, int H,
                                                    int freq, float* __restrict__ t1) {
  __shared__ float sinusoid[kSinusoid];
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int half = freq / 2;
  const T* row = w1 + (size_t)min(n, H - 1) * freq;
  float acc = 0.0f;
  for (int k0 = 0; k0 < freq; k0 += kSinusoid) {
    const int m = min(freq - k0, kSinusoid);
    if (k0 > 0) __syncthreads();
    for (int j = threadIdx.x; j < m; j += 256) {
      const int k = k0 + j, i = k < half ? k : k - half;
      const double f = exp(-9.210340371976184 * (double)i / (double)half);  // ln(10000)
      const double a = (double)t * f;
      sinusoid[j] = (float)(k < half ? cos(a) : sin(a));
    }
    __syncthreads();
    for (int j = lane; j < m; j += 64) acc = fmaf(to_f<T>(row[k0 + j]), sinusoid[j], acc);
  }
  acc = wave_sum(acc);
  if (n < H && lane == 0) t1[n] = silu_f(acc + b1[n]);
}

// sc[b][n] = SiLU(W2[n] . t1 + b2[n] + table[label_b][n]).  One wave per row, in
// 16-byte chunks, every load of the row in flight before the first is used (2
// bytes a lane and load: 10.6 us at hidden 1152, now 4.7).
constexpr int kTemb2Chunks = 8;    // H <= 2048: 512 chunks of four floats, 64 lanes

template <typename T>
__global__ __launch_bounds__(256) void temb2_kernel(const T* __restrict__ w2,
                                                    const float* __restrict__ b2,
                                                    const float* __restrict__ t1,
                                                    const T* __restrict__ table, int H, int B,
                                                    int lab0, int lab1, float* __restrict__ sc) {
  constexpr int CH = 16 / sizeof(T);
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (n >= H) return;
  const uint4* row = reinterpret_cast<const uint4*>(w2 + (size_t)n * H);
  const int nck = H / CH;
  const float add0 = b2[n], y0 = to_f<T>(table[(size_t)lab0 * H + n]), y1 = to_f<T>(table[(size_t)lab1 * H + n]);
  uint4 q[kTemb2Chunks];
#pragma unroll
  for (int u = 0; u < kTemb2Chunks; ++u)
    if (lane + 64 * u < nck) q[u] = row[lane + 64 * u];
  float acc = 0.0f;
#pragma unroll
  for (int u = 0; u < kTemb2Chunks; ++u)
    if (lane + 64 * u < nck) {
      float wv[CH];
      unpack16<T>(q[u], wv);
#pragma unroll
      for (int e = 0; e < CH; ++e) acc = fmaf(wv[e], t1[(lane + 64 * u) * CH + e], acc);
    }
  acc = wave_sum(acc) + add0;
  if (lane == 0) {
    sc[n] = silu_f(acc + y0);
    if (B > 1) sc[H + n] = silu_f(acc + y1);
  }
}

// mod[b][n] = W_ada[n] . sc[b] + b_ada[n] for every adaLN row of every block:
// streams the whole adaLN weight once.  One lane per row: the weight is held
// in 64-row groups, 16-byte chunk k of the group's rows stored contiguously
// ([group][chunk][64 rows][16 B], see adaln_group_index), so a wave's load
// of chunk k is one contiguous KiB and no dot product crosses lanes.  sc
// (both guidance branches) sits in LDS and is read as a broadcast.
constexpr int kAdaGroup = 64;

template <bool NT>
__device__ __forceinline__ uint4 load16(const uint4* p) {
  if constexpr (!NT) return *p;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}

template <typename T, bool NT>
__global__ __launch_bounds__(256) void adaln_gemv_kernel(const T* __restrict__ w,
                                                         const float* __restrict__ bias,
                                                         const float* __restrict__ sc, int H,
                                                         int n_rows, int B,
                                                         float* __restrict__ mod) {
  constexpr int CH = 16 / sizeof(T);   // elements per 16-byte chunk
  constexpr int U = 8;                 // chunks in flight per lane
  __shared__ float4 xs[2 * 2048 / 4];  // sc[b][H], H <= 2048
  const int nck = H / CH;
  for (int i = threadIdx.x; i < 2 * H / 4; i += 256) {
    const int b = i / (H / 4);
    xs[i] = b < B ? reinterpret_cast<const float4*>(sc)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int group = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int n = group * kAdaGroup + lane;
  if (group * kAdaGroup >= n_rows) return;
  const uint4* wg = reinterpret_cast<const uint4*>(w) + (size_t)group * nck * kAdaGroup + lane;
  float a0 = 0.0f, a1 = 0.0f;
  for (int k0 = 0; k0 < nck; k0 += U) {
    uint4 q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = k0 + u < nck ? load16<NT>(wg + (size_t)(k0 + u) * kAdaGroup) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u;
      if (k < nck) {
        float wv[CH];
        unpack16<T>(q[u], wv);
#pragma unroll
        for (int e4 = 0; e4 < CH / 4; ++e4) {
          const float4 x0 = xs[(k * CH) / 4 + e4], x1 = xs[H / 4 + (k * CH) / 4 + e4];
          a0 = fmaf(wv[4 * e4 + 0], x0.x, a0); a1 = fmaf(wv[4 * e4 + 0], x1.x, a1);
          a0 = fmaf(wv[4 * e4 + 1], x0.y, a0); a1 = fmaf(wv[4 * e4 + 1], x1.y, a1);
          a0 = fmaf(wv[4 * e4 + 2], x0.z, a0); a1 = fmaf(wv[4 * e4 + 2], x1.z, a1);
          a0 = fmaf(wv[4 * e4 + 3], x0.w, a0); a1 = fmaf(wv[4 * e4 + 3], x1.w, a1);
        }
      }
    }
  }
  if (n < n_rows) {
    mod[n] = a0 + bias[n];
    if (B > 1) mod[(size_t)n_rows + n] = a1 + bias[n];
  }
}

template <typename T>
static hipError_t launch_cond_t(const CondParams& p, hipStream_t s) {
  hipLaunchKernelGGL(temb1_kernel<T>, dim3(ceil_div(p.hidden, 4)), dim3(256), 0, s,
                     reinterpret_cast<const T*>(p.w_t1), p.b_t1, p.t, p.hidden, p.freq_dim, p.t1);
  hipLaunchKernelGGL(temb2_kernel<T>, dim3(ceil_div(p.hidden, 4)), dim3(256), 0, s,
                     reinterpret_cast<const T*>(p.w_t2), p.b_t2, p.t1,
                     reinterpret_cast<const T*>(p.table), p.hidden, p.B, p.labels[0],
                     p.labels[1], p.sc);
  const int blocks = ceil_div(ceil_div(p.n_mod, kAdaGroup), 4);
  // Weights that the 256 MB cache behind the L2s cannot hold to the next step are
  // read past it.  Plain / non-temporal, us a call: 446 MB 91.5 / 79.2 (6.8 TB/s at
  // best for reads alone on this card), 319 MB 70.6 / 65.8, 223 MB 42.1 / 44.6, 127 MB
  // 33.6 / 39.8.
  const bool past = (size_t)p.n_mod * p.hidden * sizeof(T) > ((size_t)256 << 20);
  const auto gemv = past ? adaln_gemv_kernel<T, true> : adaln_gemv_kernel<T, false>;
  hipLaunchKernelGGL(gemv, dim3(blocks), dim3(256), 0, s, reinterpret_cast<const T*>(p.w_ada), p.b_ada, p.sc,
                     p.hidden, p.n_mod, p.B, p.mod);
  return hipGetLastError();
}

size_t adaln_group_index(size_t row, size_t col, int H, int esize) {
  const size_t ch = 16 / esize, nck = H / ch;
  const size_t g = row / kAdaGroup, l = row % kAdaGroup, k = col / ch;
  return ((g * nck + k) * kAdaGroup + l) * ch + col % ch;
}

hipError_t launch_conditioning(const CondParams& p, int dtype, hipStream_t s) {
  if (p.hidden % 8 != 0 || p.hidden > 2048 || p.B < 1 || p.B > 2) return hipErrorInvalidValue;
  return dtype == kBF16 ? launch_cond_t<bf16>(p, s) : launch_cond_t<float>(p, s);
}

// ---------------------------------------------------------------------------
// Patch embedding of the band: h[b][tok][n] = W[n] . patch(tok) + bias[n]
// + pos[global tok][n], patch vector ordered (channel, dy, dx).  The weight is
// held transposed, wt[k][n]; a thread owns four features (16-byte loads and
// stores) of kPatchTok tokens, whose position rows are all in flight at once.
// Bound by the rows it writes: 1664 tokens x 2 branches x 1152 took 15.9 us with
// one feature a thread, 9.1 us now (23 MB).
constexpr int kPatchTok = 4;  // tokens per thread

// (patch 2, 4 channels: a 16-element patch vector, index k = c*4 + dy*2 + dx)
__global__ __launch_bounds__(64) void patch_embed_kernel(PatchEmbedParams p) {
  const int q = blockIdx.y * 64 + threadIdx.x, Q = p.hidden / 4;  // feature quad
  if (q >= Q) return;
  const int n_tok = p.n_rows * p.grid, tok0 = blockIdx.x * kPatchTok;
  const float4* pos = reinterpret_cast<const float4*>(p.pos);
  const float4* w = reinterpret_cast<const float4*>(p.w);
  float4 acc[kPatchTok], ps[kPatchTok];
  const float4 bias = reinterpret_cast<const float4*>(p.b)[q];
#pragma unroll
  for (int u = 0; u < kPatchTok; ++u) {
    const int tok = min(tok0 + u, n_tok - 1);
    ps[u] = pos[((size_t)p.row_begin * p.grid + tok) * Q + q];
    acc[u] = bias;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float4 wk = w[(size_t)k * Q + q];
    const int c = k >> 2, dy = (k >> 1) & 1, dx = k & 1;
#pragma unroll
    for (int u = 0; u < kPatchTok; ++u) {
      const int tok = min(tok0 + u, n_tok - 1);
      const int i = tok / p.grid, j = tok - i * p.grid;
      const float x = p.x[((size_t)c * p.latent + (p.row_begin + i) * 2 + dy) * p.latent + j * 2 + dx];
      acc[u].x = fmaf(wk.x, x, acc[u].x);
      acc[u].y = fmaf(wk.y, x, acc[u].y);
      acc[u].z = fmaf(wk.z, x, acc[u].z);
      acc[u].w = fmaf(wk.w, x, acc[u].w);
    }
  }
#pragma unroll
  for (int u = 0; u < kPatchTok; ++u) {
    const int tok = tok0 + u;
    if (tok >= n_tok) break;
    // (h may be a caller's buffer on 4 bytes)
    typedef float row4 __attribute__((ext_vector_type(4), aligned(4)));
    const row4 o = {acc[u].x + ps[u].x, acc[u].y + ps[u].y, acc[u].z + ps[u].z, acc[u].w + ps[u].w};
    for (int b = 0; b < p.B; ++b) reinterpret_cast<row4*>(p.h)[((size_t)b * n_tok + tok) * Q + q] = o;
  }
}

hipError_t launch_patch_embed(const PatchEmbedParams& p, hipStream_t s) {
  const int n_tok = p.n_rows * p.grid;
  if (n_tok <= 0) return hipSuccess;
  if (p.patch != 2 || p.C != 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(patch_embed_kernel, dim3(ceil_div(n_tok, kPatchTok), ceil_div(p.hidden / 4, 64)),
                     dim3(64), 0, s, p);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Final linear + unpatchify; output vector ordered (dy, dx, channel) ->
// eps[b][c][i*p + dy][j*p + dx].
__device__ __forceinline__ void unpatchify_store(const FinalParams& p, int b, int tok, int o, float v) {
  const int pp = p.patch;
  const int c = o % p.out_ch;
  const int dxy = o / p.out_ch;
  const int dy = dxy / pp, dx = dxy - (dxy / pp) * pp;
  const int i = tok / p.grid, j = tok - (tok / p.grid) * p.grid;
  const int rows = p.n_rows * pp, W = p.grid * pp;
  p.eps[(((size_t)b * p.out_ch + c) * rows + i * pp + dy) * W + j * pp + dx] = v;
}

// bf16, 16 outputs: a wave takes 16 tokens x 16 outputs on v_mfma_f32_16x16x32_bf16,
// its operands straight from memory in 16-byte fragments (token, then output,
// lane & 15, channels 8 (lane >> 4) .. + 8), kFinalBatch steps of them in flight.
// (One token a wave in 2-byte loads: 17 us at 3328 tokens x 1152, now 6.8.)
constexpr int kFinalBatch = 12;

__global__ __launch_bounds__(64) void final_linear_mfma_kernel(FinalParams p) {
  const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
  const int total = p.B * p.n_tok, t0 = blockIdx.x * 16;
  const bf16* u = reinterpret_cast<const bf16*>(p.u) + (size_t)min(t0 + r16, total - 1) * p.hidden + 8 * g;
  const bf16* w = reinterpret_cast<const bf16*>(p.w) + (size_t)r16 * p.hidden + 8 * g;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int k0 = 0; k0 < p.hidden; k0 += 32 * kFinalBatch) {
    bf16x8 a[kFinalBatch], x[kFinalBatch];
#pragma unroll
    for (int s = 0; s < kFinalBatch; ++s)
      if (k0 + 32 * s < p.hidden) {
        a[s] = *reinterpret_cast<const bf16x8*>(w + k0 + 32 * s);
        x[s] = *reinterpret_cast<const bf16x8*>(u + k0 + 32 * s);
      }
#pragma unroll
    for (int s = 0; s < kFinalBatch; ++s)
      if (k0 + 32 * s < p.hidden) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], x[s], acc, 0, 0, 0);
  }
  // the lane holds outputs 4 g .. + 4 of token r16
  const int t = t0 + r16;
  if (t >= total) return;
  const int b = t / p.n_tok, tok = t - b * p.n_tok;
#pragma unroll
  for (int r = 0; r < 4; ++r) unpatchify_store(p, b, tok, 4 * g + r, acc[r] + p.b[4 * g + r]);
}

// fp32: one wave per (branch, token).
template <int NO>
__global__ __launch_bounds__(256) void final_linear_f32_kernel(FinalParams p) {
  const int wid = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wid >= p.B * p.n_tok) return;
  const int b = wid / p.n_tok, tok = wid - b * p.n_tok;
  const float* u = reinterpret_cast<const float*>(p.u) + (size_t)wid * p.hidden;
  const float* w = reinterpret_cast<const float*>(p.w);
  float acc[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) acc[o] = 0.0f;
  for (int k = lane; k < p.hidden; k += 64) {
    const float uv = u[k];
#pragma unroll
    for (int o = 0; o < NO; ++o) acc[o] = fmaf(w[(size_t)o * p.hidden + k], uv, acc[o]);
  }
#pragma unroll
  for (int o = 0; o < NO; ++o) acc[o] = wave_sum(acc[o]);
  if (lane < NO) {
    float v = 0.0f;
#pragma unroll
    for (int o = 0; o < NO; ++o)
      if (o == lane) v = acc[o];
    unpatchify_store(p, b, tok, lane, v + p.b[lane]);
  }
}

hipError_t launch_final_linear(const FinalParams& p, int dtype, hipStream_t s) {
  const int total = p.B * p.n_tok;
  if (total <= 0) return hipSuccess;
  if (p.out_ch * p.patch * p.patch != 16 || p.hidden % 128) return hipErrorInvalidValue;
  if (dtype == kBF16)
    hipLaunchKernelGGL(final_linear_mfma_kernel, dim3(ceil_div(total, 16)), dim3(64), 0, s, p);
  else
    hipLaunchKernelGGL((final_linear_f32_kernel<16>), dim3(ceil_div(total, 4)), dim3(256), 0, s, p);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Guidance + scheduler update: out = a x - b (eu + g (ec - eu)) + c z.
// out may be x itself (each element is read before it is written, by the
// same thread), so neither carries __restrict__.
__global__ __launch_bounds__(256) void update_vec4_kernel(const float* x, int ldx,
                                                          const float* __restrict__ ec,
                                                          const float* __restrict__ eu, float g,
                                                          const float* __restrict__ z, int ldz,
                                                          float a, float b, float c,
                                                          float* out, int ldo,
                                                          int rows, size_t cols4) {
  const size_t total = (size_t)rows * cols4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (size_t)gridDim.x * 256) {
    const size_t r = i / cols4, q = i - r * cols4;
    const float4 xv = reinterpret_cast<const float4*>(x + r * (size_t)ldx)[q];
    const float4 cv = reinterpret_cast<const float4*>(ec + r * cols4 * 4)[q];
    float4 e = cv;
    if (eu) {
      const float4 uv = reinterpret_cast<const float4*>(eu + r * cols4 * 4)[q];
      e.x = uv.x + g * (cv.x - uv.x);
      e.y = uv.y + g * (cv.y - uv.y);
      e.z = uv.z + g * (cv.z - uv.z);
      e.w = uv.w + g * (cv.w - uv.w);
    }
    float4 o;
    o.x = a * xv.x - b * e.x;
    o.y = a * xv.y - b * e.y;
    o.z = a * xv.z - b * e.z;
    o.w = a * xv.w - b * e.w;
    if (z) {
      const float4 zv = reinterpret_cast<const float4*>(z + r * (size_t)ldz)[q];
      o.x += c * zv.x;
      o.y += c * zv.y;
      o.z += c * zv.z;
      o.w += c * zv.w;
    }
    reinterpret_cast<float4*>(out + r * (size_t)ldo)[q] = o;
  }
}

__global__ __launch_bounds__(256) void update_scalar_kernel(const float* x, int ldx,
                                                            const float* __restrict__ ec,
                                                            const float* __restrict__ eu, float g,
                                                            const float* __restrict__ z, int ldz,
                                                            float a, float b, float c,
                                                            float* out, int ldo,
                                                            int rows, size_t cols) {
  const size_t total = (size_t)rows * cols;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (size_t)gridDim.x * 256) {
    const size_t r = i / cols, q = i - r * cols;
    float e = ec[r * cols + q];
    if (eu) {
      const float u = eu[r * cols + q];
      e = u + g * (e - u);
    }
    float o = a * x[r * (size_t)ldx + q] - b * e;
    if (z) o += c * z[r * (size_t)ldz + q];
    out[r * (size_t)ldo + q] = o;
  }
}

static bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

hipError_t launch_update(const float* x, int ldx, const float* ec, const float* eu, float g,
                         const float* z, int ldz, float a, float b, float c, float* out, int ldo,
                         int rows, size_t cols, hipStream_t s) {
  const size_t total = (size_t)rows * cols;
  if (total == 0) return hipSuccess;
  const bool vec = cols % 4 == 0 && ldx % 4 == 0 && ldo % 4 == 0 && (!z || ldz % 4 == 0) &&
                   al16(x) && al16(ec) && (!eu || al16(eu)) && (!z || al16(z)) && al16(out);
  const size_t work = vec ? total / 4 : total;
  const int blocks = (int)std::min<size_t>((work + 255) / 256, 8192);
  if (vec)
    hipLaunchKernelGGL(update_vec4_kernel, dim3(blocks), dim3(256), 0, s, x, ldx, ec, eu, g, z,
                       ldz, a, b, c, out, ldo, rows, cols / 4);
  else
    hipLaunchKernelGGL(update_scalar_kernel, dim3(blocks), dim3(256), 0, s, x, ldx, ec, eu, g, z,
                       ldz, a, b, c, out, ldo, rows, cols);
  return hipGetLastError();
}

}  // namespace orch
