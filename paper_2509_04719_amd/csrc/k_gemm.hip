// Projection GEMMs of the DiT block: y = A W^T + bias with fused epilogues
// (plain store, GELU, gated residual add into the fp32 residual stream, and
// the QKV scatter into the head-major Q buffer and the K / V^T buffer).
//
// bf16 path: MFMA tiles fed by direct-to-LDS loads (described at the kernels).
// fp32 path: 32x32x2 fp32 MFMAs (described at the kernel).  Shapes and pointers
// neither takes: a 64x64 SIMT tile with 4x4 outputs per thread.
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace orch {

// ---------------------------------------------------------------------------
// Epilogue.  A lane owns one output column n and, per call, four consecutive
// rows m..m+3 (the 32x32 MFMA accumulator layout).  Everything that depends
// on the column only is computed once per column in `Col`.
template <typename T, int EPI>
struct Epilogue {
  const EpiParams& ep;
  int M, N;

  struct Col {
    bool on;
    float bias;
    // QKV: destination of (branch 0, token 0), strides, factor (Q: q_scale)
    T* base;
    size_t bstride;
    int tstride;
    float mul = 1.0f;
    // RESIDUAL: gate pointer of branch 0
    const float* gate;
  };

  __device__ __forceinline__ int branch_of(int m) const {
    int b = 0;
    while (m >= (b + 1) * ep.rows_per_batch) ++b;
    return b;
  }

  __device__ __forceinline__ Col column(int n) const {
    Col c{};
    c.on = n < N;
    if (!c.on) return c;
    c.bias = ep.bias[n];
    if (EPI == kEpiResidual) c.gate = ep.gate + n;
    if (EPI == kEpiQkv) {
      const int which = n / ep.hidden;
      const int nn = n - which * ep.hidden;
      const int head = nn / ep.head_dim;
      const int dd = nn - head * ep.head_dim;
      const size_t ntot = (size_t)ep.kv_tokens;
      if (which == 0) {
        c.mul = ep.q_scale;
        c.base = reinterpret_cast<T*>(ep.q) + (size_t)head * ep.rows_per_batch * ep.head_dim + dd;
        c.bstride = (size_t)ep.heads * ep.rows_per_batch * ep.head_dim;
        c.tstride = ep.head_dim;
      } else if (which == 1) {
        c.base = reinterpret_cast<T*>(ep.kv) + ((size_t)head * ntot + ep.tok_offset) * ep.head_dim + dd;
        c.bstride = ep.kv_branch_stride;
        c.tstride = ep.head_dim;
      } else {
        c.base = reinterpret_cast<T*>(ep.kv) + ntot * ep.hidden +
                 ((size_t)head * ep.head_dim + dd) * ntot + ep.tok_offset;
        c.bstride = ep.kv_branch_stride;
        c.tstride = 1;
      }
    }
    return c;
  }

  __device__ __forceinline__ void store4(const Col& c, int m, int n, const float* v) const {
    if (!c.on) return;
    if (EPI == kEpiStore || EPI == kEpiGelu) {
      T* out = reinterpret_cast<T*>(ep.out) + n;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (m + r < M) {
          float y = v[r] + c.bias;
          if (EPI == kEpiGelu) y = gelu_fast(y);
          out[(size_t)(m + r) * N] = from_f<T>(y);
        }
      }
    } else if (EPI == kEpiResidual) {
      float* h = reinterpret_cast<float*>(ep.out) + n;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int mm = m + r;
        if (mm < M) h[(size_t)mm * N] += c.gate[(size_t)branch_of(mm) * ep.gate_stride] * (v[r] + c.bias);
      }
    } else {  // kEpiQkv
      const int b = branch_of(m);
      const int tok = m - b * ep.rows_per_batch;
      if (m + 3 < M && tok + 3 < ep.rows_per_batch) {
        T* dst = c.base + b * c.bstride + (size_t)tok * c.tstride;
        if (sizeof(T) == 2 && c.tstride == 1 && ((uintptr_t)dst & 7) == 0) {
          bf16x4 w;
#pragma unroll
          for (int r = 0; r < 4; ++r) w[r] = (bf16)((v[r] + c.bias) * c.mul);
          *reinterpret_cast<bf16x4*>(dst) = w;
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) dst[(size_t)r * c.tstride] = from_f<T>((v[r] + c.bias) * c.mul);
        }
      } else {
        for (int r = 0; r < 4; ++r) {
          const int mm = m + r;
          if (mm >= M) break;
          const int bb = branch_of(mm);
          const int tk = mm - bb * ep.rows_per_batch;
          c.base[bb * c.bstride + (size_t)tk * c.tstride] = from_f<T>((v[r] + c.bias) * c.mul);
        }
      }
    }
  }

  // GELU (tanh form) with tanh(u) = 1 - 2 / (exp(2u) + 1) on the fast exp;
  // used where the result is rounded to bf16.
  __device__ __forceinline__ static float gelu_fast(float x) {
    if (sizeof(T) == 4) return gelu_tanh_f(x);
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    const float e = __expf(2.0f * u);
    const float th = 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
    return 0.5f * x * (1.0f + th);
  }
};

// ---------------------------------------------------------------------------
// Epilogue of the MFMA GEMM.  The MFMAs produce transposed 32x32 blocks, so a
// lane holds C[m][n..n+3] (m = lane % 32 of the block, n = 8g + 4(lane / 32)).
// Each wave stages one 32-row strip of its tile at a time in a private LDS
// area (row stride TN + 4 floats, so the 16-byte writes of 16 rows land in
// distinct banks), then walks the strip in chunks along n: every global load
// and store is 16 bytes wide and a row's chunks are contiguous.  The QKV
// scatter writes Q and K rows the same way and walks V^T columns (8 tokens of
// one channel per lane).
template <int FM, int FN, int EPI>
struct StripEpilogue {
  static constexpr int TN = 32 * FN;
  static constexpr int LS = TN + 4;
  static constexpr int BYTES = 32 * LS * 4;  // LDS per wave

  const EpiParams& ep;
  int M, N;
  int split;   // kEpiPartial: this workgroup's k-split

  __device__ __forceinline__ int branch_of(int m) const {
    int b = 0;
    while (m >= (b + 1) * ep.rows_per_batch) ++b;
    return b;
  }

  // GELU, tanh form, as y * sigmoid(2u): 0.5 (1 + tanh(u)) = 1 / (1 + e^(-2u)),
  // u = sqrt(2/pi) (y + 0.044715 y^3), with e^(-2u) = exp2(y (c0 + c1 y^2))
  __device__ __forceinline__ static float act(float y) {
    if (EPI != kEpiGelu) return y;
    constexpr float c0 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
    constexpr float c1 = c0 * 0.044715f;
    const float e = __builtin_amdgcn_exp2f(y * fmaf(c1, y * y, c0));
    return y * __builtin_amdgcn_rcpf(1.0f + e);
  }

  // Operands of the epilogue loaded before the main loop, so their latency
  // hides behind the MFMAs: the bias of each store chunk, and for the gated
  // residual of one-strip tiles the fp32 h and gate rows as well.
  static constexpr int SIT = 32 * (TN / 8) / 64;       // store chunks per lane per strip
  static constexpr int RIT = 32 * (TN / 4) / 64;       // residual chunks per lane per strip
  static constexpr bool PRE_H = EPI == kEpiResidual && FM == 1 && RIT <= 8;
  // 8-channel bias chunks: one per store chunk, or a single one when every
  // chunk of a lane falls on the same columns (64 a multiple of TN / 8)
  static constexpr bool BIAS8 = EPI == kEpiStore || EPI == kEpiGelu || EPI == kEpiQkv;
  static constexpr int NB = (64 % (TN / 8) == 0) ? 1 : SIT;
  struct Pre {
    f32x4 b[BIAS8 ? NB : 1][2];
    float vb[EPI == kEpiQkv ? TN / 16 : 1];
    f32x4 h[PRE_H ? RIT : 1], g[PRE_H ? RIT : 1], rb[PRE_H ? RIT : 1];
  };

  // bias[nb]: that of column n0 (global memory, or the tile's in LDS)
  __device__ __forceinline__ void prefetch(Pre& pre, int lane, int m0, int n0, const float* bias, int nb) const {
    if constexpr (BIAS8) {
      constexpr int CH = TN / 8;
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int n = nb + ((q * 64 + lane) % CH) * 8;
        pre.b[q][0] = *reinterpret_cast<const f32x4*>(bias + n);
        pre.b[q][1] = *reinterpret_cast<const f32x4*>(bias + n + 4);
      }
    }
    if constexpr (EPI == kEpiQkv) {
#pragma unroll
      for (int q = 0; q < TN / 16; ++q) pre.vb[q] = bias[nb + q * 16 + (lane >> 2)];
    }
    if constexpr (PRE_H) {
      constexpr int CH = TN / 4;
      const float* hb = reinterpret_cast<const float*>(ep.out);
#pragma unroll
      for (int q = 0; q < RIT; ++q) {
        const int f = q * 64 + lane, m = m0 + f / CH, n = n0 + (f % CH) * 4;
        const bool in = m < M;
        const int mm = in ? m : M - 1;
        pre.h[q] = *reinterpret_cast<const f32x4*>(hb + (size_t)mm * N + n);
        pre.g[q] = *reinterpret_cast<const f32x4*>(ep.gate + (size_t)branch_of(mm) * ep.gate_stride + n);
        pre.rb[q] = *reinterpret_cast<const f32x4*>(ep.bias + n);
      }
    }
  }

  // rows [mr, mr + 32) x columns [n0, n0 + TN) of C, staged in strip
  __device__ __forceinline__ void rows_store(const float* strip, int lane, int mr, int n0,
                                             const Pre& pre) const {
    constexpr int CH = TN / 8, IT = 32 * CH / 64;
    bf16* out = reinterpret_cast<bf16*>(ep.out);
#pragma unroll
    for (int q = 0; q < IT; ++q) {
      const int f = q * 64 + lane, row = f / CH, c = f % CH;
      const int m = mr + row, n = n0 + c * 8;
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(strip + row * LS + c * 8);
      const f32x4 x1 = *reinterpret_cast<const f32x4*>(strip + row * LS + c * 8 + 4);
      if (m < M) {
        const f32x4 b0 = pre.b[NB == 1 ? 0 : q][0];
        const f32x4 b1 = pre.b[NB == 1 ? 0 : q][1];
        bf16x8 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o[r] = from_f<bf16>(act(x0[r] + b0[r]));
          o[4 + r] = from_f<bf16>(act(x1[r] + b1[r]));
        }
        *reinterpret_cast<bf16x8*>(out + (size_t)m * N + n) = o;
      }
    }
  }

  __device__ __forceinline__ void rows_residual(const float* strip, int lane, int mr, int n0,
                                                const Pre& pre) const {
    constexpr int CH = TN / 4, IT = 32 * CH / 64;
    float* hb = reinterpret_cast<float*>(ep.out);
    f32x4 x[IT], hv[IT];
    // all loads first (or prefetched): the stores below may alias them as far
    // as the compiler knows, so this keeps at most one round trip per strip
#pragma unroll
    for (int q = 0; q < IT; ++q) {
      const int f = q * 64 + lane, row = f / CH, c = f % CH;
      const int m = mr + row, n = n0 + c * 4;
      x[q] = *reinterpret_cast<const f32x4*>(strip + row * LS + c * 4);
      if constexpr (PRE_H) hv[q] = pre.h[q];
      else hv[q] = m < M ? *reinterpret_cast<const f32x4*>(hb + (size_t)m * N + n) : f32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int q = 0; q < IT; ++q) {
      const int f = q * 64 + lane, row = f / CH, c = f % CH;
      const int m = mr + row, n = n0 + c * 4;
      if (m < M) {
        f32x4 g, b;
        if constexpr (PRE_H) {
          g = pre.g[q];
          b = pre.rb[q];
        } else {
          g = *reinterpret_cast<const f32x4*>(ep.gate + (size_t)branch_of(m) * ep.gate_stride + n);
          b = *reinterpret_cast<const f32x4*>(ep.bias + n);
        }
        f32x4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = hv[q][r] + g[r] * (x[q][r] + b[r]);
        *reinterpret_cast<f32x4*>(hb + (size_t)m * N + n) = y;
      }
    }
  }

  __device__ __forceinline__ void rows_qkv(const float* strip, int lane, int mr, int n0,
                                           const Pre& pre) const {
    const int hd = ep.head_dim, hidden = ep.hidden, rpb = ep.rows_per_batch;
    const size_t ntot = (size_t)ep.kv_tokens;
    bf16* qb = reinterpret_cast<bf16*>(ep.q);
    bf16* kvb = reinterpret_cast<bf16*>(ep.kv);
    // Q and K: 8 channels of one head per lane (head_dim % 8 == 0)
    if (n0 < 2 * hidden) {
      constexpr int CH = TN / 8, IT = 32 * CH / 64;
#pragma unroll
      for (int q = 0; q < IT; ++q) {
        const int f = q * 64 + lane, row = f / CH, c = f % CH;
        const int m = mr + row, n = n0 + c * 8;
        if (m >= M || n >= 2 * hidden) continue;
        const f32x4 x0 = *reinterpret_cast<const f32x4*>(strip + row * LS + c * 8);
        const f32x4 x1 = *reinterpret_cast<const f32x4*>(strip + row * LS + c * 8 + 4);
        const f32x4 b0 = pre.b[NB == 1 ? 0 : q][0];
        const f32x4 b1 = pre.b[NB == 1 ? 0 : q][1];
        const int b = branch_of(m), tok = m - b * rpb;
        const int which = n >= hidden, nn = n - which * hidden;
        const float mul = which ? 1.0f : ep.q_scale;
        const int head = (int)__umulhi((unsigned)nn, ep.hd_magic), dd = nn - head * hd;
        bf16* dst = which == 0 ? qb + (((size_t)b * ep.heads + head) * rpb + tok) * hd + dd
                               : kvb + b * ep.kv_branch_stride + ((size_t)head * ntot + ep.tok_offset + tok) * hd + dd;
        bf16x8 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o[r] = from_f<bf16>((x0[r] + b0[r]) * mul);
          o[4 + r] = from_f<bf16>((x1[r] + b1[r]) * mul);
        }
        *reinterpret_cast<bf16x8*>(dst) = o;
      }
    }
    // V^T [head][d][token]: 8 consecutive tokens of one channel per lane;
    // four lanes cover the strip's 32 tokens (64 contiguous bytes).  Token
    // groups 2 and 3 read their tokens rotated by four (8 LS = 32 mod 64 banks
    // would put them on the banks of groups 0 and 1; 4 LS = 16 mod 64 moves
    // them to the free ones), then swap the halves back.
    static_assert((4 * LS) % 64 == 16, "conflict-free V^T reads");
    if (n0 + TN > 2 * hidden) {
      constexpr int IT = TN * 4 / 64;
#pragma unroll
      for (int q = 0; q < IT; ++q) {
        const int col = q * 16 + (lane >> 2), grp = lane & 3;
        const int n = n0 + col;
        if (n < 2 * hidden) continue;
        const int rot = (grp >> 1) * 4;
        float v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float x = strip[(grp * 8 + ((t + rot) & 7)) * LS + col];   // token t ^ rot
          v[t] = x;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float a = v[t], b = v[t + 4];
          v[t] = rot ? b : a;
          v[t + 4] = rot ? a : b;
        }
        const float bias = pre.vb[q];
        const int nn = n - 2 * hidden, head = (int)__umulhi((unsigned)nn, ep.hd_magic), dd = nn - head * hd;
        bf16* vt = kvb + ntot * hidden + ((size_t)head * hd + dd) * ntot + ep.tok_offset;
        const int m = mr + grp * 8;
        const int b = m < M ? branch_of(m) : 0, tok = m - b * rpb;
        bf16* dst = vt + b * ep.kv_branch_stride + tok;
        if (m + 7 < M && tok + 7 < rpb && ((uintptr_t)dst & 15) == 0) {
          bf16x8 o;
#pragma unroll
          for (int t = 0; t < 8; ++t) o[t] = from_f<bf16>(v[t] + bias);
          *reinterpret_cast<bf16x8*>(dst) = o;
        } else {
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int mm = m + t;
            if (mm < M) {
              const int bb = branch_of(mm);
              vt[bb * ep.kv_branch_stride + (mm - bb * rpb)] = from_f<bf16>(v[t] + bias);
            }
          }
        }
      }
    }
  }

  // a k-split's partial sums, fp32 rows of ws[split]
  __device__ __forceinline__ void rows_partial(const float* strip, int lane, int mr, int n0) const {
    constexpr int CH = TN / 4, IT = 32 * CH / 64;
    float* wb = ep.ws + (size_t)split * M * N;
#pragma unroll
    for (int q = 0; q < IT; ++q) {
      const int f = q * 64 + lane, row = f / CH, c = f % CH;
      const int m = mr + row, n = n0 + c * 4;
      if (m < M)
        *reinterpret_cast<f32x4*>(wb + (size_t)m * N + n) = *reinterpret_cast<const f32x4*>(strip + row * LS + c * 4);
    }
  }

  // the wave's tile: rows [m0, m0 + 32 FM), columns [n0, n0 + TN)
  __device__ __forceinline__ void run(const f32x16 (&acc)[FM][FN], float* strip, int lane, int m0,
                                      int n0, const Pre& pre) const {
    const int lr = lane & 31, h = lane >> 5;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(strip + lr * LS + j * 32 + 8 * g + 4 * h) =
              f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
      if constexpr (EPI == kEpiStore || EPI == kEpiGelu) rows_store(strip, lane, m0 + 32 * i, n0, pre);
      else if constexpr (EPI == kEpiResidual) rows_residual(strip, lane, m0 + 32 * i, n0, pre);
      else if constexpr (EPI == kEpiPartial) rows_partial(strip, lane, m0 + 32 * i, n0);
      else rows_qkv(strip, lane, m0 + 32 * i, n0, pre);
    }
  }
};

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM.
//
// BM x BN x BK block tile over WM x WN waves; each wave owns a (BM/WM) x
// (BN/WN) block of v_mfma_f32_32x32x16_bf16 accumulators in fp32.  Operands go
// global -> LDS with the direct-to-LDS load (16 bytes per lane, 1 KB per wave
// instruction, no register staging) into a ring of S stages.  LDS rows are
// 2*BK bytes, unpadded; the 16-byte chunks of row r are XOR-swizzled by
// (r / Q) % CPR so that a fragment read (16 lanes = 16 rows at one logical
// chunk) touches 64 distinct banks.  One barrier per k-tile; the loads of
// tile kt+S-1 are interleaved with the MFMAs of tile kt.
// Compile-time layout of one configuration.
template <int BM, int BN, int BK, int WM, int WN, int S>
struct GemmGeo {
  static constexpr int NW = WM * WN;
  static constexpr int TM = BM / WM, TN = BN / WN;  // wave tile
  static constexpr int FM = TM / 32, FN = TN / 32;  // 32x32 blocks per wave
  static constexpr int CPR = BK / 8;                // 16-byte chunks per row
  static constexpr int RPL = 1024 / (2 * BK);       // rows per wave-level load
  static constexpr int Q = 128 / BK;                // rows per 256-byte bank sweep
  static constexpr int IA = BM / (NW * RPL), IB = BN / (NW * RPL);
  static constexpr int LPT = IA + IB;               // loads per lane per k-tile
  static constexpr int STAGE = (BM + BN) * BK * 2;  // bytes per stage
  static constexpr int KK = BK / 16;                // MFMA k-steps per k-tile
  // next-tile loads issued per k-step: all in the first with two stages (they
  // get one tile of compute to land), else spread over the k-steps
  static constexpr int LPK = S == 2 ? LPT : (LPT + KK - 1) / KK;
  static_assert(NW == 4 || NW == 8, "four or eight waves");
  static_assert(BK == 32 || BK == 64, "k-tile");
  static_assert(FM >= 1 && FN >= 1 && TM % 32 == 0 && TN % 32 == 0, "wave tile");
  static_assert(BM % (NW * RPL) == 0 && BN % (NW * RPL) == 0, "rows per wave");
  static_assert(S >= 2 && S <= 8 && LPT * (S - 1) < 64, "pipeline depth");
  static_assert(S * STAGE <= 160 * 1024, "LDS");
};

// Which tile a workgroup takes: workgroup b is in split b / T of T = tiles_m x
// tiles_n tiles; inside a split XCD-major, then groups of 8 tile rows,
// column-major inside.
struct TileAt {
  int split, m, n;
  __device__ __forceinline__ TileAt(int tiles_m, int tiles_n) {
    const int T = tiles_m * tiles_n;
    split = __builtin_amdgcn_readfirstlane(blockIdx.x / T);
    int pid = blockIdx.x - split * T;
    const int per = T / 8;
    if (pid < per * 8) pid = (pid & 7) * per + (pid >> 3);
    constexpr int GROUP = 8;
    const int gid = pid / (GROUP * tiles_n);
    const int first_m = gid * GROUP;
    const int gsz = min(tiles_m - first_m, GROUP);
    m = first_m + (pid % (GROUP * tiles_n)) % gsz;
    n = (pid % (GROUP * tiles_n)) / gsz;
  }
};

template <int BM, int BN, int BK, int WM, int WN, int S, int EPI>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_kernel(const bf16* __restrict__ A,
                                                        const bf16* __restrict__ W, int M, int N,
                                                        int K, int ldk, int tiles_m, int tiles_n,
                                                        EpiParams ep) {
  using G = GemmGeo<BM, BN, BK, WM, WN, S>;
  constexpr int FM = G::FM, FN = G::FN, KK = G::KK, IA = G::IA, LPT = G::LPT, LPK = G::LPK;

  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // K is this workgroup's k extent, ldk the row stride of A and W: with a
  // k-split, split s takes keys [s K, (s + 1) K)
  const TileAt at(tiles_m, tiles_n);
  const int split = at.split;
  const int m0 = at.m * BM, n0 = at.n * BN;

  // byte offset of this lane's source chunk in each wave-level load: load j
  // covers tile rows (j * NW + wave) * RPL .. + RPL - 1 (A rows first, then
  // W rows); A rows past M re-read row M - 1
  const int prow = lane / G::CPR;
  const int pchunk = lane % G::CPR;
  unsigned off[LPT];
#pragma unroll
  for (int j = 0; j < LPT; ++j) {
    const int i = j < IA ? j : j - IA;
    const int r = (i * G::NW + wave) * G::RPL + prow;
    const int lchunk = pchunk ^ ((r / G::Q) % G::CPR);
    const unsigned row = j < IA ? (unsigned)min(m0 + r, M - 1) : (unsigned)(n0 + r);
    off[j] = (row * (unsigned)ldk + lchunk * 8) * 2u;
  }
  const char* gA = reinterpret_cast<const char*>(A + (size_t)split * K);
  const char* gW = reinterpret_cast<const char*>(W + (size_t)split * K);

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // fragment read offsets: row = wave tile row + lrow, logical chunk 2 kk + h
  const int lrow = lane & 31;
  const int h = lane >> 5;
  int koff[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) koff[kk] = ((2 * kk + h) ^ ((lrow / G::Q) % G::CPR)) * 16;
  const int arow = (wm * G::TM + lrow) * BK * 2;
  const int brow = BM * BK * 2 + (wn * G::TN + lrow) * BK * 2;

  const int KT = K / BK;  // >= S - 1 (checked by the launcher)

  // load j of k-tile kt into stage st
  auto dma = [&](auto jc, int kt_, int st_) {
    constexpr int j = decltype(jc)::value;
    constexpr int i = j < IA ? j : j - IA;
    constexpr int part = j < IA ? 0 : BM * BK * 2;
    char* dst = smem + st_ * G::STAGE + part + (i * G::NW + wave) * G::RPL * BK * 2;
    const char* src = (j < IA ? gA : gW) + (unsigned)kt_ * (BK * 2) + off[j];
    __builtin_amdgcn_global_load_lds((const ORCH_GLB void*)src, (ORCH_LDS void*)dst, 16, 0, 0);
  };

  // the MFMAs of stage st; with issue, the loads of tile ikt into stage ist
  // go between them.  Emission order is fixed slot by slot (a scheduling
  // fence after each): MFMA e of k-step kk, then its share of the reads of
  // k-step kk+1's fragments, then its share of the next tile's loads.
  auto compute = [&](int st, auto issue_c, int ikt, int ist) {
    constexpr bool ISSUE = decltype(issue_c)::value;
    constexpr int NM = FM * FN, ND = FM + FN;
    const char* base = smem + st * G::STAGE;
    bf16x8 a[2][FM], b[2][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
      a[0][i] = *reinterpret_cast<const bf16x8*>(base + arow + i * 32 * BK * 2 + koff[0]);
#pragma unroll
    for (int j = 0; j < FN; ++j)
      b[0][j] = *reinterpret_cast<const bf16x8*>(base + brow + j * 32 * BK * 2 + koff[0]);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, KK>([&](auto kkc) {
      constexpr int kk = decltype(kkc)::value;
      constexpr int cur = kk & 1;
      constexpr int nd = kk + 1 < KK ? ND : 0;
      constexpr int l0 = cmin(kk * LPK, LPT), nl = ISSUE ? cmin(kk * LPK + LPK, LPT) - l0 : 0;
      static_for<0, NM>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        constexpr int i = e / FN, j = e % FN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[cur][j], a[cur][i], acc[i][j], 0, 0, 0);
        static_for<e * nd / NM, (e + 1) * nd / NM>([&](auto dc) {
          constexpr int d = decltype(dc)::value;
          if constexpr (d < FM)
            a[cur ^ 1][d] = *reinterpret_cast<const bf16x8*>(base + arow + d * 32 * BK * 2 + koff[kk + 1]);
          else
            b[cur ^ 1][d - FM] =
                *reinterpret_cast<const bf16x8*>(base + brow + (d - FM) * 32 * BK * 2 + koff[kk + 1]);
        });
        static_for<l0 + e * nl / NM, l0 + (e + 1) * nl / NM>([&](auto jc) { dma(jc, ikt, ist); });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };

  // epilogue operands first: the oldest loads, covered by the main loop
  using E = StripEpilogue<FM, FN, EPI>;
  const E epi{ep, M, N, split};
  typename E::Pre pre;
  epi.prefetch(pre, lane, m0 + wm * G::TM, n0 + wn * G::TN, ep.bias, n0 + wn * G::TN);

#pragma unroll
  for (int s = 0; s < S - 1; ++s) static_for<0, LPT>([&](auto jc) { dma(jc, s, s); });
  int kt = 0;
  for (; kt + S - 1 < KT; ++kt) {
    wait_vmcnt<(S - 2) * LPT>();
    lds_barrier();
    compute(kt % S, std::true_type{}, kt + S - 1, (kt + S - 1) % S);
  }
  // drain: the last S-1 tiles, nothing more to issue
  static_for<0, S - 2>([&](auto rc) {
    wait_vmcnt<(S - 2 - decltype(rc)::value) * LPT>();
    lds_barrier();
    compute(kt % S, std::false_type{}, 0, 0);
    ++kt;
  });
  wait_vmcnt<0>(); lds_barrier(); compute(kt % S, std::false_type{}, 0, 0);

  // epilogue: the stage buffers become per-wave staging strips
  static_assert(G::NW * E::BYTES <= S * G::STAGE, "epilogue staging fits the stage buffers");
  lds_barrier();
  epi.run(acc, reinterpret_cast<float*>(smem + wave * E::BYTES), lane, m0 + wm * G::TM, n0 + wn * G::TN,
          pre);
}

// ---------------------------------------------------------------------------
// The 256 x 256 tile in phases: eight waves (2 x 4, 128 x 64 outputs each), k-tiles
// of 64 in two LDS stages.  A k-tile takes four phases, one for each quarter
// (i, j) of the wave's tile: 64 rows (half i of A) x 32 columns (half j of W),
// eight MFMAs, in the order (0,0) (0,1) (1,1) (1,0).  Between its MFMAs a phase
// reads the fragments of the next one (each half has registers of its own, W's
// two halves swapping sets every k-tile) and loads one half-tile two k-tiles
// ahead into the stage just read:
//
//   phase  MFMAs  reads        loads
//   P0     A0 W0  W1(kt)       A0(kt + 2)
//   P1     A0 W1  A1(kt)       W0(kt + 2)
//   P2     A1 W1  A0(kt + 1)   W1(kt + 2)
//   P3     A1 W0  W0(kt + 1)   A1(kt + 2)
//
// A barrier before P0 and one before P2: each publishes the two halves read
// until the next (loaded six or more phases earlier: vmcnt(8) leaves the four
// younger half-tiles in flight) and frees the two read since the last.  So no
// MFMA waits for an LDS round trip behind a barrier, and a load has 1.5 k-tiles to
// land; gemm_bf16_kernel reads a k-tile's first fragments after its barrier and
// loads one k-tile ahead.
// k runs in the same order as there, 16 at a time: the same bits.
namespace ph {
constexpr int BM = 256, BN = 256, BK = 64, KK = 4, HALF = 128 * BK * 2, LDS = 8 * HALF + BN * 4;
enum { kA0 = 0, kA1 = 1, kW0 = 2, kW1 = 3 };
// half x of stage st: A's four in the first 64 KB, W's in the second (read
// offsets within 16 bits of one base each)
constexpr int at(int x, int st) { return ((x & 2) * 2 + st * 2 + (x & 1)) * HALF; }
}  // namespace ph

template <int EPI>
__global__ __launch_bounds__(512) void gemm_bf16_phased_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                               int M, int N, int K, int tiles_m, int tiles_n, EpiParams ep) {
  // (device-only types: the host pass needs the launch stub alone)
#if defined(__HIP_DEVICE_COMPILE__)
  using namespace ph;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const TileAt ta(tiles_m, tiles_n);
  const int m0 = ta.m * BM, n0 = ta.n * BN;

  // Half X's row r is row 128 (r / 64) + 64 i + r % 64 of A's tile, 64 (r / 32) +
  // 32 j + r % 32 of W's: each wave's 128 x 64 outputs are contiguous.  Load l of
  // a half fills rows 8 l .. + 8, this wave's are l = 2 wave, 2 wave + 1; chunk c
  // of row r lies at c ^ (r / 2 % 8).  A rows past M re-read row M - 1.
  unsigned off[4][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = (2 * wave + q) * 8 + (lane >> 3);
    const unsigned ch = (unsigned)((lane & 7) ^ ((r >> 1) & 7)) * 16u;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      off[kA0 + x][q] = (unsigned)min(m0 + 128 * (r >> 6) + 64 * x + (r & 63), M - 1) * (unsigned)K * 2u + ch;
      off[kW0 + x][q] = (unsigned)(n0 + 64 * (r >> 5) + 32 * x + (r & 31)) * (unsigned)K * 2u + ch;
    }
  }
  // (buffer loads: the k-tile is a scalar offset, the lane's offset constant; the
  // launcher keeps both matrices under 2 GiB)
  const __amdgpu_buffer_rsrc_t rA = buffer_rsrc(A, (size_t)M * K * 2);
  const __amdgpu_buffer_rsrc_t rW = buffer_rsrc(W, (size_t)N * K * 2);
  // load q of half x of k-tile kt into stage st
  auto load = [&](int x, int q, int st, int kt) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(x < kW0 ? rA : rW,
                                             (ORCH_LDS void*)(smem + at(x, st) + (2 * wave + q) * 1024), 16, off[x][q],
                                             (unsigned)kt * (BK * 2), 0, 0);
  };

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // (two LDS bases per k-step, the rest in the read's 16-bit offset; the empty asm
  // keeps the compiler from moving the 64 KB out of W's)
  int a_rd[KK], w_rd[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int ko = ((2 * kk + h) ^ ((lr >> 1) & 7)) * 16;
    a_rd[kk] = (64 * wm + lr) * BK * 2 + ko;
    w_rd[kk] = at(kW0, 0) + (32 * wn + lr) * BK * 2 + ko;
    asm volatile("" : "+v"(w_rd[kk]));
  }
  bf16x8 fa[2][2 * KK], fw[2][KK];   // A halves (two 32-row blocks), W halves
  // fragment e of a half: k-step e / 2, block e % 2 of A; k-step e of W
  auto read_a = [&](int x, int st, int e) __attribute__((always_inline)) {
    fa[x][e] = *reinterpret_cast<const bf16x8*>(smem + a_rd[e >> 1] + at(kA0 + x, st) + (e & 1) * 32 * BK * 2);
  };
  auto read_w = [&](int x, int st, int set, int e) __attribute__((always_inline)) {
    fw[set][e] = *reinterpret_cast<const bf16x8*>(smem + w_rd[e] + (at(kW0 + x, st) - at(kW0, 0)));
  };
  // at most `ahead` loads in flight, every fragment read arrived, then the barrier
  auto sync = [&](auto ahead_c) __attribute__((always_inline)) {
    wait_vmcnt<decltype(ahead_c)::value>();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // quarter (i, j) from W's register set; f(e) follows MFMA e
  auto quarter = [&](auto ic, auto jc, auto set_c, auto&& f) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value, j = decltype(jc)::value, set = decltype(set_c)::value;
    static_for<0, 2 * KK>([&](auto ec) {
      constexpr int e = decltype(ec)::value, b = e & 1;
      acc[2 * i + b][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[set][e >> 1], fa[i][e], acc[2 * i + b][j], 0, 0, 0);
      f(e);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using E = StripEpilogue<4, 2, EPI>;
  const E epi{ep, M, N, 0};
  typename E::Pre pre;
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // k-tile kt in stage ST (its W0 in set ST).  LEFT: k-tiles after it, 2: two or
  // more, so the loads go on
  auto ktile = [&](auto st_c, auto left_c, int kt) __attribute__((always_inline)) {
    constexpr int ST = decltype(st_c)::value, LEFT = decltype(left_c)::value;
    constexpr bool L = LEFT == 2;
    using S0 = std::integral_constant<int, ST>;
    using S1 = std::integral_constant<int, ST ^ 1>;
    sync(std::integral_constant<int, LEFT == 0 ? 0 : 8>{});
    quarter(I0{}, I0{}, S0{}, [&](int e) __attribute__((always_inline)) {
      if (e < KK) read_w(1, ST, ST ^ 1, e);
      if (L && (e & 3) == 3) load(kA0, e >> 2, ST, kt + 2);
    });
    quarter(I0{}, I1{}, S1{}, [&](int e) __attribute__((always_inline)) {
      read_a(1, ST, e);
      if (L && (e & 3) == 3) load(kW0, e >> 2, ST, kt + 2);
    });
    if constexpr (LEFT > 0) sync(std::integral_constant<int, L ? 8 : 4>{});
    quarter(I1{}, I1{}, S1{}, [&](int e) __attribute__((always_inline)) {
      if (LEFT > 0) read_a(0, ST ^ 1, e);
      if (L && (e & 3) == 3) load(kW1, e >> 2, ST, kt + 2);
    });
    quarter(I1{}, I0{}, S0{}, [&](int e) __attribute__((always_inline)) {
      if (LEFT > 0 && e < KK) read_w(0, ST ^ 1, ST ^ 1, e);
      if (L && (e & 3) == 3) load(kA1, e >> 2, ST, kt + 2);
    });
  };

  const int KT = K / BK;   // even (checked by the launcher)
  // the tile's bias first, past the stages (it is cold in a step, and there is no
  // register for it to wait in)
  if (wave == 0)
    __builtin_amdgcn_global_load_lds((const ORCH_GLB void*)(ep.bias + n0 + 4 * lane), (ORCH_LDS void*)(smem + 8 * HALF),
                                     16, 0, 0);
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
    for (const int x : {kA0, kW0, kW1, kA1})
      for (int q = 0; q < 2; ++q) load(x, q, kt, kt);
  wait_vmcnt<12>();
  lds_barrier();
#pragma unroll
  for (int e = 0; e < 2 * KK; ++e) read_a(0, 0, e);
#pragma unroll
  for (int e = 0; e < KK; ++e) read_w(0, 0, 0, e);
  int kt = 0;
  for (; kt + 2 < KT; kt += 2) {
    ktile(I0{}, std::integral_constant<int, 2>{}, kt);
    ktile(I1{}, std::integral_constant<int, 2>{}, kt + 1);
  }
  ktile(I0{}, I1{}, kt);
  ktile(I1{}, I0{}, kt + 1);

  static_assert(8 * E::BYTES <= 8 * HALF, "epilogue staging fits the stages");
  lds_barrier();
  epi.prefetch(pre, lane, m0 + wm * 128, n0 + wn * 64, reinterpret_cast<const float*>(smem + 8 * HALF), wn * 64);
  epi.run(acc, reinterpret_cast<float*>(smem + wave * E::BYTES), lane, m0 + wm * 128, n0 + wn * 64, pre);
#endif
}

// ---------------------------------------------------------------------------
// bf16 GEMM for few output tiles: four waves, (BM / 32) x (BN / 32) blocks of
// 32 x 32 outputs x KG groups that share the k (group g takes the stages g, g + KG,
// ...; their sums meet in LDS, added in group order).  A stage is U k-tiles of 64,
// laid out and swizzled as in gemm_bf16_kernel; a ring of S per group.  k runs in
// the same order as there with one group: the same bits.
template <int BM, int BN, int KG, int U, int S>
struct GemmSmallGeo {
  static constexpr int NWG = 4 / KG, WN = BN / 32;
  static constexpr int TILE = (BM + BN) * 128;            // bytes of a k-tile
  static constexpr int STAGE = U * TILE;
  static constexpr int LPT = (BM + BN) / 8 / NWG;         // 1 KB loads per wave and k-tile
  static constexpr int LDS = KG * S * STAGE;
  static_assert((BM / 32) * (BN / 32) == NWG, "a 32 x 32 block per wave");
  static_assert((BM + BN) / 8 % NWG == 0 && (S - 1) * U * LPT < 64, "whole loads");
  static_assert((KG - 1) * NWG * 4096 <= LDS && LDS <= 160 * 1024, "LDS");
};

template <int BM, int BN, int KG, int U, int S, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_small_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                              int M, int N, int K, int tiles_n, EpiParams ep) {
  using G = GemmSmallGeo<BM, BN, KG, U, S>;
  constexpr int LPT = G::LPT;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = wave % G::NWG, kg = wave / G::NWG;
  // row-major tiles, an eighth of them in a row on each XCD
  int w = blockIdx.x;
  const int per = gridDim.x / 8;
  if (w < per * 8) w = (w & 7) * per + (w >> 3);
  const int m0 = w / tiles_n * BM, n0 = w % tiles_n * BN;
  const int mw = m0 + wg / G::WN * 32, nw = n0 + wg % G::WN * 32;
  char* ring = smem + kg * S * G::STAGE;

  using E = StripEpilogue<1, 1, EPI>;
  const E epi{ep, M, N, 0};
  typename E::Pre pre;
  if (kg == 0) epi.prefetch(pre, lane, mw, nw, ep.bias, nw);

  // load i of a k-tile: rows 8 (wg LPT + i) .. + 8 (A first, then W); A rows past
  // M re-read row M - 1
  unsigned off[LPT];
  bool isa[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int r0 = (wg * LPT + i) * 8, r = r0 + (lane >> 3);
    isa[i] = r0 < BM;
    off[i] = ((isa[i] ? (unsigned)min(m0 + r, M - 1) : (unsigned)(n0 + r - BM)) * (unsigned)K +
              ((lane & 7) ^ ((r >> 1) & 7)) * 8) * 2u;
  }
  const char* gA = reinterpret_cast<const char*>(A);
  const char* gW = reinterpret_cast<const char*>(W);
  // this group's t-th stage
  auto issue = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < LPT; ++i)
        __builtin_amdgcn_global_load_lds(
            (const ORCH_GLB void*)((isa[i] ? gA : gW) + (unsigned)((kg + KG * t) * U + u) * 128 + off[i]),
            (ORCH_LDS void*)(ring + t % S * G::STAGE + u * G::TILE + (wg * LPT + i) * 1024), 16, 0, 0);
  };
  const int arow = (wg / G::WN * 32 + lr) * 128, wrow = (BM + wg % G::WN * 32 + lr) * 128;
  int koff[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) koff[c] = ((2 * c + h) ^ ((lr >> 1) & 7)) * 16;
  f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;

  // groups differ by at most one stage; all meet every barrier
  const int ST = K / (64 * U), mine = (ST - kg + KG - 1) / KG, NIT = (ST + KG - 1) / KG;
#pragma unroll
  for (int t = 0; t < S - 1; ++t)
    if (t < mine) issue(t);
  for (int t = 0; t < NIT; ++t) {
    if (t + S - 2 < mine) wait_vmcnt<(S - 2) * U * LPT>();
    else wait_vmcnt<0>();
    lds_barrier();
    if (t + S - 1 < mine) issue(t + S - 1);
    if (t >= mine) continue;
    const char* base = ring + t % S * G::STAGE;
    bf16x8 a[U][4], b[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a[u][c] = *reinterpret_cast<const bf16x8*>(base + u * G::TILE + arow + koff[c]);
        b[u][c] = *reinterpret_cast<const bf16x8*>(base + u * G::TILE + wrow + koff[c]);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[u][c], a[u][c], acc[0][0], 0, 0, 0);
  }
  lds_barrier();
  if constexpr (KG > 1) {
    if (kg > 0) {
      float* part = reinterpret_cast<float*>(smem + ((kg - 1) * G::NWG + wg) * 4096) + lane;
#pragma unroll
      for (int r = 0; r < 16; ++r) part[r * 64] = acc[0][0][r];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g) {
      const float* part = reinterpret_cast<const float*>(smem + (g * G::NWG + wg) * 4096) + lane;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][0][r] += part[r * 64];
    }
  }
  // (the strips lie past the groups' sums)
  constexpr int SUMS = (KG - 1) * G::NWG * 4096;
  static_assert(SUMS + G::NWG * E::BYTES <= G::LDS, "strips fit the ring");
  epi.run(acc, reinterpret_cast<float*>(smem + SUMS + wg * E::BYTES), lane, mw, nw, pre);
}

// ---------------------------------------------------------------------------
// fp32 GEMM on v_mfma_f32_32x32x2_f32 (fp32 products and sums; 154 TFLOP/s in a
// large library product, twice the vector unit without packed instructions).
// A workgroup is four waves: (BM / 32) x (BN / 32) blocks of 32 x 32 outputs x KG
// groups that share the k-tiles.  k-tiles of 32 (128-byte rows) go straight
// into LDS, a ring of S stages per group, 16-byte chunks XOR-swizzled by row as
// in the bf16 kernel.  A fragment read gives a lane four consecutive k of its
// row, one for each of four MFMAs: MFMA e of chunk pair c adds k = 8 c + e and
// 8 c + 4 + e.
//
// Every configuration adds in the same order, that K alone fixes: four sums, of the
// k-tiles 4 i, 4 i + 1, 4 i + 2 and 4 i + 3, added as ((0 + 1) + 2) + 3.  Group g of KG
// holds the sums g, g + KG, ... (its k-tiles g, g + KG, ... in turn); the others'
// meet group 0's in LDS.  So a row's result does not depend on how many rows
// the call has.
template <int BM, int BN, int KG, int S>
struct GemmF32Geo {
  static constexpr int BK = 32, NWG = 4 / KG;             // waves per group
  static constexpr int SUMS = 4 / KG;                     // sums per group
  static constexpr int WN = BN / 32;
  static constexpr int STAGE = (BM + BN) * BK * 4;
  static constexpr int LPT = (BM + BN) / 8 / NWG;         // 1 KB loads per wave and k-tile
  static constexpr int LDS = KG * S * STAGE;
  static_assert((BM / 32) * (BN / 32) == NWG, "a 32 x 32 block per wave");
  static_assert((BM + BN) / 8 % NWG == 0, "whole loads");
  static_assert((KG - 1) * NWG * SUMS * 4096 <= LDS, "the groups' sums fit the ring");
};

template <int BM, int BN, int KG, int S, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                       int M, int N, int K, int tiles_n, EpiParams ep) {
  using G = GemmF32Geo<BM, BN, KG, S>;
  constexpr int LPT = G::LPT, SUMS = G::SUMS;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = wave % G::NWG, kg = wave / G::NWG;
  const int m0 = (int)blockIdx.x / tiles_n * BM, n0 = (int)blockIdx.x % tiles_n * BN;
  char* ring = smem + kg * S * G::STAGE;

  // load j of a stage: rows 8 j .. + 8 (A first, then W); rows past the matrix
  // re-read its last one
  const char* src[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int r = (wg * LPT + i) * 8 + (lane >> 3);
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    const float* row = r < BM ? A + (size_t)min(m0 + r, M - 1) * K : W + (size_t)min(n0 + r - BM, N - 1) * K;
    src[i] = reinterpret_cast<const char*>(row + ch * 4);
  }
  // this group's t-th k-tile into stage st
  auto issue = [&](int t, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i)
      __builtin_amdgcn_global_load_lds((const ORCH_GLB void*)(src[i] + (size_t)(kg + KG * t) * (G::BK * 4)),
                                       (ORCH_LDS void*)(ring + st * G::STAGE + (wg * LPT + i) * 1024), 16, 0, 0);
  };
  const int arow = (wg / G::WN * 32 + lr) * 128, brow = (BM + wg % G::WN * 32 + lr) * 128;
  int koff[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) koff[c] = ((2 * c + h) ^ ((lr >> 1) & 7)) * 16;
  f32x16 acc[SUMS];
#pragma unroll
  for (int u = 0; u < SUMS; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[u][r] = 0.0f;

  const int KT = K / G::BK, mine = (KT - kg + KG - 1) / KG;   // this group's k-tiles
  // its t-th k-tile landed and every read of the stage before done, for every wave;
  // the next load
  auto turn = [&](int t) __attribute__((always_inline)) {
    if (t + S - 2 < mine) wait_vmcnt<(S - 2) * LPT>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    if (t + S - 1 < mine) issue(t + S - 1, (t + S - 1) % S);
  };
  auto add = [&](int t, f32x16& sum) __attribute__((always_inline)) {
    const char* base = ring + t % S * G::STAGE;
    f32x4 a[4], b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      a[c] = *reinterpret_cast<const f32x4*>(base + arow + koff[c]);
      b[c] = *reinterpret_cast<const f32x4*>(base + brow + koff[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][e], b[c][e], sum, 0, 0, 0);
  };
#pragma unroll
  for (int t = 0; t < S - 1; ++t)
    if (t < mine) issue(t, t);
  // four k-tiles a turn, one for each sum; then the last KT % 4, where a group may
  // be short (all meet every barrier)
  int t = 0;
  for (; KG * (t + SUMS) <= KT; t += SUMS) {
    static_for<0, SUMS>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      turn(t + u);
      add(t + u, acc[u]);
    });
  }
  static_for<0, SUMS>([&](auto uc) {
    constexpr int u = decltype(uc)::value;
    if (KG * (t + u) < KT) {
      turn(t + u);
      if (t + u < mine) add(t + u, acc[u]);
    }
  });
  if constexpr (KG > 1) {
    __syncthreads();
    if (kg > 0) {
      float* part = reinterpret_cast<float*>(smem + ((kg - 1) * G::NWG + wg) * SUMS * 4096) + lane;
#pragma unroll
      for (int u = 0; u < SUMS; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[(16 * u + r) * 64] = acc[u][r];
    }
    __syncthreads();
    if (kg > 0) return;
  }
#pragma unroll
  for (int j = 1; j < 4; ++j) {
    const int g = j % KG, u = j / KG;    // sum j: group g's u-th
    if (g == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][r] += acc[u][r];
    } else {
      const float* part = reinterpret_cast<const float*>(smem + ((g - 1) * G::NWG + wg) * SUMS * 4096) + lane;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][r] += part[(16 * u + r) * 64];
    }
  }
  // a lane holds column lr, rows 8 g + 4 h .. + 4
  const Epilogue<float, EPI> epi{ep, M, N};
  const int n = n0 + wg % G::WN * 32 + lr;
  const auto col = epi.column(n);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float v[4] = {acc[0][4 * g], acc[0][4 * g + 1], acc[0][4 * g + 2], acc[0][4 * g + 3]};
    epi.store4(col, m0 + wg / G::WN * 32 + 8 * g + 4 * h, n, v);
  }
}

// ---------------------------------------------------------------------------
// SIMT GEMM (shapes and pointers the matrix-core kernels do not take)
namespace simt_gemm {
constexpr int BM = 64, BN = 64, BK = 16;
}

template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_simt_kernel(const T* __restrict__ A,
                                                        const T* __restrict__ W, int M, int N,
                                                        int K, EpiParams ep) {
  using namespace simt_gemm;
  __shared__ float sA[BK][BM + 4];
  __shared__ float sB[BK][BN + 4];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int idx = tid + 256 * e;
      int r = idx >> 4, kk = idx & 15;
      int gk = k0 + kk;
      int gm = m0 + r, gn = n0 + r;
      sA[kk][r] = (gm < M && gk < K) ? to_f<T>(A[(size_t)gm * K + gk]) : 0.f;
      sB[kk][r] = (gn < N && gk < K) ? to_f<T>(W[(size_t)gn * K + gk]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sA[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = sB[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  const Epilogue<T, EPI> epi{ep, M, N};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = n0 + tx * 4 + j;
    float v[4] = {acc[0][j], acc[1][j], acc[2][j], acc[3][j]};
    epi.store4(epi.column(n), m0 + ty * 4, n, v);
  }
}

// ---------------------------------------------------------------------------
// Tile selection.  ORCH_GEMM_TILE=<index> forces a configuration (tuning): a row
// of kTiles, then of kSmall.
struct TileCfg {
  int bm, bn, bk, waves, stages;
  float eff;  // measured relative throughput of the shape on a full machine
};
static const TileCfg kTiles[] = {
    {256, 256, 64, 8, 2, 1.17f},
    {256, 192, 64, 8, 2, 1.00f},
    {128, 128, 64, 8, 4, 0.75f},
    {128, 64, 64, 4, 2, 0.30f},  // fallback: any N % 64 == 0, K % 64 == 0
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr int kFallbackTile = kNumTiles - 1;

static int forced_tile() {
  const char* s = getenv("ORCH_GEMM_TILE");
  return s ? atoi(s) : -1;
}

static bool tile_fits(const TileCfg& t, int N, int K) {
  return N % t.bn == 0 && K % t.bk == 0 && K / t.bk >= t.stages - 1;
}

// Pick the configuration with the least estimated time: whole rounds of tiles
// over the 256 CUs times the tile area, divided by the tile's relative
// throughput per CU.  The throughputs were measured on the DiT-XL projection
// shapes (K = 1152 and 4608, M from 768 to 20480).  A round of K = 1152 takes 31 to
// 35 us with 256x256 tiles, 27 to 29 with 256x192 and 12 with 128x128: 1152 -> 4608
// takes 195 us in 6 rounds of 256x256 and 231 us in 8 rounds of 256x192 at M = 20480,
// 121 (4) and 136 us (5) at 12288, 86 and 88 us (3 each) at 8192; the 128x128
// tile wins when 256-row tiles would leave most CUs idle.  The rating of 256x256
// holds for both of its loops: where only the plain one runs (K an odd multiple of
// 64), 256x256 against 256x192 is 20.8 / 24.7 us at 16896 x 192 -> 1536, 52.2 / 56.4 at
// 12288 x 320 -> 4608, 201 / 220 at 20480 x 1088 -> 4608.
static int pick_tile(int M, int N, int K, int f) {
  if (f >= 0 && f < kNumTiles && tile_fits(kTiles[f], N, K)) return f;
  int best = kFallbackTile;
  float best_cost = 0.0f;
  for (int c = 0; c < kNumTiles; ++c) {
    const TileCfg& t = kTiles[c];
    if (!tile_fits(t, N, K)) continue;
    const int tiles = ceil_div(M, t.bm) * (N / t.bn);
    const float cost = (float)ceil_div(tiles, 256) * t.bm * t.bn / t.eff;
    if (best_cost == 0.0f || cost < best_cost) {
      best = c;
      best_cost = cost;
    }
  }
  return best;
}

bool gemm_uses_mfma(int N, int K, int dtype) {
  return dtype == kBF16 && N % 64 == 0 && K % 64 == 0;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// The MFMA kernel moves 16-byte chunks of every operand and output; shapes
// or pointers that do not allow that take the SIMT kernel.
static bool mfma_path_ok(const void* A, const void* W, int N, int K, int epi, const EpiParams& ep,
                         int dtype) {
  if (!gemm_uses_mfma(N, K, dtype) || !aligned16(A) || !aligned16(W) || !aligned16(ep.bias))
    return false;
  if (epi == kEpiResidual) return aligned16(ep.out) && aligned16(ep.gate) && ep.gate_stride % 4 == 0;
  if (epi == kEpiQkv)
    return aligned16(ep.q) && aligned16(ep.kv) && ep.head_dim % 8 == 0 && ep.kv_branch_stride % 8 == 0 &&
           ep.hidden < 65536;
  return aligned16(ep.out);
}

template <int BM, int BN, int BK, int WM, int WN, int S, int EPI>
static void launch_tile(const void* A, const void* W, int M, int N, int K, const EpiParams& ep0,
                        hipStream_t s, int splits = 1) {
  const int tm = ceil_div(M, BM), tn = N / BN;
  constexpr int lds = S * GemmGeo<BM, BN, BK, WM, WN, S>::STAGE;
  EpiParams ep = ep0;
  // head = umulhi(channel, ceil(2^32 / head_dim)): exact for channels < 2^16
  if (EPI == kEpiQkv) ep.hd_magic = (unsigned)((0x100000000ull + ep.head_dim - 1) / ep.head_dim);
  auto kern = gemm_bf16_kernel<BM, BN, BK, WM, WN, S, EPI>;
  static bool attr = [&] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    return true;
  }();
  (void)attr;
  hipLaunchKernelGGL(kern, dim3(tm * tn * splits), dim3(64 * WM * WN), lds, s,
                     reinterpret_cast<const bf16*>(A), reinterpret_cast<const bf16*>(W), M, N,
                     K / splits, K, tm, tn, ep);
}

// Sum of the k-splits' partials, then the caller's epilogue (bias, GELU,
// gated residual or the QKV scatter): four rows of one column per thread, the
// splits added in order.
template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_split_reduce_kernel(int splits, int M, int N,
                                                                EpiParams ep) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  const int m = blockIdx.y * 4;
  if (n >= N) return;
  const Epilogue<T, EPI> epi{ep, M, N};
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int sp = 0; sp < splits; ++sp) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (m + r < M) v[r] += ep.ws[((size_t)sp * M + m + r) * N + n];
  }
  epi.store4(epi.column(n), m, n, v);
}

// K-split of a GEMM whose tiles leave most of the machine idle (at most 128
// tiles for 256 CUs): splits s with s * tiles <= 256, at least 8 k-tiles per
// split, s dividing the k-tiles and the partials fitting the workspace.
// (Splits that take more than one round, e.g. 144 tiles in three splits, or
// 378 in two, measured slower than no split: the partials' round trip
// through HBM costs more than the idle CUs.)
static int split_plan(int M, int N, int K, const TileCfg& t, size_t ws_elems) {
  const int tiles = ceil_div(M, t.bm) * (N / t.bn);
  const int kt = K / t.bk;
  if (tiles > 128) return 1;
  int sp = cmin(256 / tiles, kt / 8);
  while (sp > 1 && (kt % sp != 0 || (size_t)sp * M * N > ws_elems)) --sp;
  return sp;
}

template <int EPI>
static void launch_phased(const void* A, const void* W, int M, int N, int K, const EpiParams& ep0, hipStream_t s) {
  EpiParams ep = ep0;
  if (EPI == kEpiQkv) ep.hd_magic = (unsigned)((0x100000000ull + ep.head_dim - 1) / ep.head_dim);
  auto kern = gemm_bf16_phased_kernel<EPI>;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, ph::LDS);
  (void)attr;
  const int tm = ceil_div(M, ph::BM), tn = N / ph::BN;
  hipLaunchKernelGGL(kern, dim3(tm * tn), dim3(512), ph::LDS, s, reinterpret_cast<const bf16*>(A),
                     reinterpret_cast<const bf16*>(W), M, N, K, tm, tn, ep);
}

template <int EPI>
static void launch_tile_cfg(int c, const void* A, const void* W, int M, int N, int K,
                            const EpiParams& ep, hipStream_t s, int splits) {
  switch (c) {
    case 0:
      // More than one round: the phased kernel (1152 -> 4608, M = 20480: 229 -> 210
      // us).  In a single round the plain loop: there the phased kernel is 2 us
      // faster by itself (M = 3328 in a step: 38.4 -> 36.5 us), but the
      // attention after it loses as much (71.9 -> 73.5 us) and the step 1%.  (A
      // k-split is one round at most: split_plan.)
      if constexpr (EPI != kEpiPartial) {
        if (K % 128 == 0 && ceil_div(M, ph::BM) * (N / ph::BN) > 256 && (size_t)cmax(M, N) * K < (size_t)1 << 30) {
          launch_phased<EPI>(A, W, M, N, K, ep, s);
          break;
        }
      }
      launch_tile<256, 256, 64, 2, 4, 2, EPI>(A, W, M, N, K, ep, s, splits);
      break;
    case 1: launch_tile<256, 192, 64, 4, 2, 2, EPI>(A, W, M, N, K, ep, s, splits); break;
    case 2: launch_tile<128, 128, 64, 4, 2, 4, EPI>(A, W, M, N, K, ep, s, splits); break;
    default: launch_tile<128, 64, 64, 2, 2, 2, EPI>(A, W, M, N, K, ep, s, splits); break;
  }
}

template <int BM, int BN, int KG, int U, int S, int EPI>
static void launch_small_tile(const void* A, const void* W, int M, int N, int K, const EpiParams& ep0, hipStream_t s) {
  using G = GemmSmallGeo<BM, BN, KG, U, S>;
  EpiParams ep = ep0;
  if (EPI == kEpiQkv) ep.hd_magic = (unsigned)((0x100000000ull + ep.head_dim - 1) / ep.head_dim);
  auto kern = gemm_bf16_small_kernel<BM, BN, KG, U, S, EPI>;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS);
  (void)attr;
  hipLaunchKernelGGL(kern, dim3(ceil_div(M, BM) * (N / BN)), dim3(256), G::LDS, s, reinterpret_cast<const bf16*>(A),
                     reinterpret_cast<const bf16*>(W), M, N, K, N / BN, ep);
}

// Whether and how to use the small kernel: the configuration with the least
// estimated time, if that is below the estimate of the tile and k-split chosen
// otherwise.  Estimates in us over the k-tiles of 64, fitted to M from 32 to 3328
// at the DiT projections of hidden 384, 768 and 1152 and checked from 8 rows and K =
// 64 on:
//   small  2.5 + max(KT' b, KT c WGs / 256): KT' the k-tiles rounded up to whole turns
//          of the groups, b a lone workgroup's k-tile (a group's turn, shared by the
//          groups), c what a CU
//          needs per workgroup's k-tile when several share it (about 54 B per
//          ns and CU of operands from L2, the same for all of them); one
//          workgroup per CU (LDS): 2.5 + KT' b rounds + 1.5 per further round
//   128^2  4.5 + 0.42 KT / splits a round, plus 5 and 8 B of partials per split
//          and output at 6 TB/s with a k-split
// Measured, us before -> after: hidden 384, M = 96: qkv 5.3 -> 3.6, out-proj 6.5 -> 3.7,
// fc1 6.3 -> 3.8, fc2 12.1 -> 5.5 (k-split and reduction before); hidden 1152, M =
// 384: 14.7 -> 11.7, 13.5 -> 7.4, 16.1 -> 13.0, 25.2 -> 18.6; M = 768: out-proj 15.2 -> 9.1,
// while qkv and fc1 stay (11.6 against 19.8, 13.3 against 23.4).
struct SmallCfg {
  int bm, bn, groups, k;   // k: K is a multiple of it
  bool one;                // one workgroup per CU
  float b, c;
};
static const SmallCfg kSmall[] = {
    {32, 32, 4, 64, true, 0.125f, 0.0f}, {32, 32, 4, 64, false, 0.165f, 0.21f}, {32, 64, 2, 64, false, 0.205f, 0.25f},
    {64, 64, 1, 128, true, 0.28f, 0.0f}, {64, 64, 1, 128, false, 0.33f, 0.38f},
};

static int pick_small(int M, int N, int K, const TileCfg& t, int splits, bool fixed_order, int f) {
  constexpr int n = sizeof(kSmall) / sizeof(kSmall[0]);
  if (f >= 0) return f >= kNumTiles && f < kNumTiles + n && K % kSmall[f - kNumTiles].k == 0 ? f - kNumTiles : -1;
  const int kt = K / 64;
  const int rounds = ceil_div(ceil_div(M, t.bm) * (N / t.bn) * splits, 256);
  if (t.bm != 128 || rounds > 1) return -1;
  float best = 4.5f + 0.42f * kt / splits + (splits > 1 ? 5.0f + splits * ((float)M * N * 8e-6f / 6.0f) : 0.0f);
  int pick = -1;
  for (int i = 0; i < n; ++i) {
    const SmallCfg& c = kSmall[i];
    if (K % c.k || (fixed_order && c.groups > 1)) continue;
    const int wgs = ceil_div(M, c.bm) * (N / c.bn), r = ceil_div(wgs, 256);
    const float alone = ceil_div(kt, c.groups) * c.groups * c.b, shared = kt * c.c * wgs / 256.0f;
    const float us = 2.5f + (c.one ? alone * r + 1.5f * (r - 1) : alone > shared ? alone : shared);
    if (us < best) {
      best = us;
      pick = i;
    }
  }
  return pick;
}

template <int EPI>
static void launch_small(int c, const void* A, const void* W, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  switch (c) {
    case 0: launch_small_tile<32, 32, 4, 1, 4, EPI>(A, W, M, N, K, ep, s); break;
    case 1: launch_small_tile<32, 32, 4, 1, 2, EPI>(A, W, M, N, K, ep, s); break;
    case 2: launch_small_tile<32, 64, 2, 1, 3, EPI>(A, W, M, N, K, ep, s); break;
    case 3: launch_small_tile<64, 64, 1, 2, 4, EPI>(A, W, M, N, K, ep, s); break;
    default: launch_small_tile<64, 64, 1, 2, 2, EPI>(A, W, M, N, K, ep, s); break;
  }
}

template <int BM, int BN, int KG, int S, int EPI>
static void launch_f32_tile(const void* A, const void* W, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  using G = GemmF32Geo<BM, BN, KG, S>;
  auto kern = gemm_f32_kernel<BM, BN, KG, S, EPI>;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS);
  (void)attr;
  const int tn = ceil_div(N, BN);
  hipLaunchKernelGGL(kern, dim3(ceil_div(M, BM) * tn), dim3(256), G::LDS, s, reinterpret_cast<const float*>(A),
                     reinterpret_cast<const float*>(W), M, N, K, tn, ep);
}

// The split of the four waves (the same bits in each).  A 32 x 32 block is one
// wave's chain of K / 2 MFMAs (64 cycles each), so with few blocks the key groups
// shorten it, and with some thousands the two-group tile still spreads them more
// evenly; with more, the 64 x 64 tile loads half the bytes per product.  Measured us
// for (64, 64, 1) / (32, 64, 2) / (32, 32, 4): 96 x 1536 -> 384 (36 blocks) 35 / 20 /
// 14; 1000 x 1536 -> 384 (384) 38 / 24 / 25; 1000 x 384 -> 1152 (1152) 18.6 / 15.7 /
// 18.5; 2000 x 3072 -> 768 (1512) 117 / 95 / 111; 4096 x 4608 -> 1152 (4608) 410 /
// 390 / 442; 4096 x 1152 -> 4608 (18432) 375 / 401 / 530.  (The 64 x 64 SIMT tile:
// 1000 x 384 -> 1152 42 us.)
template <int EPI>
static void launch_f32(const void* A, const void* W, int M, int N, int K, const EpiParams& ep, hipStream_t s) {
  const long long blocks = (long long)ceil_div(M, 32) * ceil_div(N, 32);
  if (blocks > 8192) launch_f32_tile<64, 64, 1, 3, EPI>(A, W, M, N, K, ep, s);
  else if (blocks > 512) launch_f32_tile<32, 64, 2, 2, EPI>(A, W, M, N, K, ep, s);
  else launch_f32_tile<32, 32, 4, 2, EPI>(A, W, M, N, K, ep, s);
}

template <int EPI>
static hipError_t launch_gemm_epi(const void* A, const void* W, int M, int N, int K,
                                  const EpiParams& ep, int dtype, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
  if (mfma_path_ok(A, W, N, K, EPI, ep, dtype)) {
    const int f = forced_tile(), c = pick_tile(M, N, K, f);
    const int sp = ep.ws && aligned16(ep.ws) ? split_plan(M, N, K, kTiles[c], ep.ws_elems) : 1;
    // a workspace smaller than the plan's is no leave to share K
    const bool fixed = ep.fixed_order || (ep.ws && sp < split_plan(M, N, K, kTiles[c], (size_t)-1));
    const int sm = pick_small(M, N, K, kTiles[c], sp, fixed, f);
    if (sm >= 0) {
      launch_small<EPI>(sm, A, W, M, N, K, ep, s);
    } else if (sp > 1) {
      launch_tile_cfg<kEpiPartial>(c, A, W, M, N, K, ep, s, sp);
      hipLaunchKernelGGL((gemm_split_reduce_kernel<bf16, EPI>), dim3(ceil_div(N, 256), ceil_div(M, 4)),
                         dim3(256), 0, s, sp, M, N, ep);
    } else {
      launch_tile_cfg<EPI>(c, A, W, M, N, K, ep, s, 1);
    }
  } else if (dtype == kF32 && K % 32 == 0 && aligned16(A) && aligned16(W)) {
    launch_f32<EPI>(A, W, M, N, K, ep, s);
  } else {
    dim3 grid(ceil_div(N, simt_gemm::BN), ceil_div(M, simt_gemm::BM));
    if (dtype == kBF16)
      hipLaunchKernelGGL((gemm_simt_kernel<bf16, EPI>), grid, dim3(256), 0, s,
                         reinterpret_cast<const bf16*>(A), reinterpret_cast<const bf16*>(W), M,
                         N, K, ep);
    else
      hipLaunchKernelGGL((gemm_simt_kernel<float, EPI>), grid, dim3(256), 0, s,
                         reinterpret_cast<const float*>(A), reinterpret_cast<const float*>(W),
                         M, N, K, ep);
  }
  return hipGetLastError();
}

size_t gemm_split_workspace_elems(int M, int N, int K, int dtype) {
  if (M <= 0 || !gemm_uses_mfma(N, K, dtype)) return 0;
  const int f = forced_tile(), c = pick_tile(M, N, K, f);
  if (!tile_fits(kTiles[c], N, K)) return 0;
  const int sp = split_plan(M, N, K, kTiles[c], (size_t)-1);
  if (sp > 1) return (size_t)sp * M * N;
  // waves that share K need no room, but a caller's leave: 16 bytes
  const int sm = pick_small(M, N, K, kTiles[c], 1, false, f);
  return sm >= 0 && kSmall[sm].groups > 1 ? 4 : 0;
}

hipError_t launch_gemm(const void* A, const void* W, int M, int N, int K, int epi,
                       const EpiParams& ep, int dtype, hipStream_t s) {
  switch (epi) {
    case kEpiStore: return launch_gemm_epi<kEpiStore>(A, W, M, N, K, ep, dtype, s);
    case kEpiGelu: return launch_gemm_epi<kEpiGelu>(A, W, M, N, K, ep, dtype, s);
    case kEpiResidual: return launch_gemm_epi<kEpiResidual>(A, W, M, N, K, ep, dtype, s);
    case kEpiQkv: return launch_gemm_epi<kEpiQkv>(A, W, M, N, K, ep, dtype, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace orch
