// Attention of a band's queries over the whole image's keys/values (fresh and
// stale, as in k_attention.hip) for the head dimensions and types that kernel
// does not take: bf16 heads of 32, 80, 96 and 128 channels, and fp32 heads of
// every size.
//
// Flash style on the matrix cores, a wave per 32 queries, 32 keys at a time.
// The scores are formed transposed, S^T = K Q^T, so a lane owns one query
// column; O^T = V^T P^T takes the probabilities straight from the score
// registers:
//   fp32  v_mfma_f32_32x32x2_f32.  Its two k of an instruction are the keys
//         8g + e and 8g + 4 + e that score register 4g + e holds in the two
//         lane halves, so P needs no movement at all.
//   bf16  v_mfma_f32_32x32x16_bf16, the K rows permuted in LDS (bits 2 and 3
//         of the row swapped) so that a lane's eight scores of a 16-key chunk
//         are consecutive keys.  Scores are scaled in fp32 (Q is not rounded
//         again) and the probabilities are split p = hi + lo in two bf16, two
//         MFMAs for each V^T fragment: 16 significant bits of p reach the PV
//         product, so rounding the output to bf16 stays the only error that
//         shows (2-norm against float64 1.7e-3; with p rounded once 2.4e-3).
//         hi is p's top 16 bits and lo what is left of p (1 + 2^-23), so both are
//         positive (down to p = 2^-103) and an infinite V gives hi V + lo V = V,
//         not a NaN.
// K tiles ([32 keys][d]) and V^T tiles ([d][32 keys]) go global -> LDS with the
// direct-to-LDS load into a ring of stages, one barrier per iteration, their
// 16-byte chunks swizzled by row so that 16 rows at one chunk hit distinct banks.
//
// Measured: bf16, 16 (branch, head) x 1000 queries x 4096 keys, d = 128: 37.9 ms
// in the scalar kernel (one thread per query), 65 us here, 516 TFLOP/s counting
// every product once (the split P makes it 775 on the matrix cores).  Bound by a
// wave's own chain of MFMAs, exponentials and conversions: at this shape each
// SIMD holds one wave.
//
// A workgroup is four waves, QG query groups x KG key groups: key group g takes
// the key tiles g, g + KG, ..., and the groups' parts of a query meet in LDS at
// the end.  Splitting the keys inside the workgroup is what fills the chip
// where the queries alone do not.  With PARTS = 2 a group walks its keys as two
// groups would, one after the other: the same bits as twice the groups.
#include <cfloat>

#include "common.h"
#include "kernels.h"

namespace orch {

namespace gen_attn {
constexpr int BKV = 32;
constexpr float kUp = 1.0f + 0x1p-23f;

constexpr int gcd_(int a, int b) { return b == 0 ? a : gcd_(b, a % b); }

template <typename T, int D, int KG, int PARTS = 1>
struct Geo {
  static constexpr int EPC = 16 / (int)sizeof(T);     // elements per 16-byte chunk
  static constexpr int KPC = 2 * EPC;                 // contraction depth per fragment pair
  static constexpr int NC = D / KPC;                  // K fragments per lane
  static constexpr int NX = BKV / KPC;                // V^T fragments per lane and 32-row tile
  static constexpr int KCH = D / EPC;                 // chunks per K row
  static constexpr int VCH = BKV / EPC;               // chunks per V^T row
  static constexpr int KP = 16 / gcd_(KCH, 16);       // rows between rotations
  static constexpr int VP = 16 / gcd_(VCH, 16);
  static constexpr int DT = (D + 31) / 32;            // 32-row tiles of O^T
  static constexpr int TB = BKV * D * (int)sizeof(T); // bytes of a K tile, and of a V^T tile
  static constexpr int NL = 2 * TB / 1024;            // 1 KB loads per tile pair
  static constexpr int STAGE = 2 * TB + (DT * 32 - D) * BKV * (int)sizeof(T);
  static constexpr int S = 3;
  static constexpr int QG = 4 / KG;
  static constexpr int PART = (DT * 16 + 2) * 256;    // a wave's O, max and sum
  static constexpr int LDS = KG * S * STAGE;
  static constexpr bool FITS = LDS <= 160 * 1024;
  static_assert(PARTS == 1 || PARTS == 2, "parts");
  static_assert(D % KPC == 0 && TB % 1024 == 0, "whole fragments and loads");
  static_assert((KG - 1) * PARTS * QG * PART <= LDS, "parts fit the ring");
};

// Chunk ch of a row of CH chunks lies at position swizzle(ch, row): XOR where
// CH is a power of two, else rotated, one step every P rows.
template <int CH, int P>
__device__ __forceinline__ int swizzle(int ch, int row) {
  return (CH & (CH - 1)) == 0 ? ch ^ (row / P % CH) : (ch + row / P) % CH;
}
template <int CH, int P>
__device__ __forceinline__ int unswizzle(int pos, int row) {
  return (CH & (CH - 1)) == 0 ? pos ^ (row / P % CH) : (pos + CH - row / P % CH) % CH;
}
__device__ __forceinline__ int kperm(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }
}  // namespace gen_attn

template <typename T, int D, int KG, int PARTS>
__global__ __launch_bounds__(256, D * sizeof(T) >= 384 ? 1 : 2) void attn_general_kernel(AttnParams p) {
  using namespace gen_attn;
  using G = Geo<T, D, KG, PARTS>;
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int QG = G::QG, S = G::S, EPC = G::EPC, ES = (int)sizeof(T);
  constexpr int LPW = (G::NL + QG - 1) / QG;          // loads per wave and tile
  typedef T frag __attribute__((ext_vector_type(EPC)));

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, lc = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qg = wave % QG, kg = wave / QG;

  // workgroups in the order (branch, head, query tile), an eighth of them in a
  // row on each XCD, so the query tiles that read the same K/V share an L2
  const int n_qt = (p.n_q + 32 * QG - 1) / (32 * QG);
  const int NWG = gridDim.x;
  int w = blockIdx.x;
  if (w < NWG / 8 * 8) w = (w & 7) * (NWG / 8) + (w >> 3);
  const int pair = w / n_qt, q0 = (w - pair * n_qt) * 32 * QG + 32 * qg;
  const int b = pair / p.heads, head = pair - b * p.heads;
  const int n_kv = p.n_kv, fb = p.fresh_begin, nf = p.n_fresh;
  const int fn = nf > 0 ? p.fresh_n : n_kv;
  const size_t H = (size_t)p.heads * D;
  const T* ks = reinterpret_cast<const T*>(p.kv_stale) + b * p.stale_bs + (size_t)head * n_kv * D;
  const T* vs = reinterpret_cast<const T*>(p.kv_stale) + b * p.stale_bs + n_kv * H + (size_t)head * D * n_kv;
  const T *kf = ks, *vf = vs;
  if (nf > 0) {
    kf = reinterpret_cast<const T*>(p.kv_fresh) + b * p.fresh_bs + ((size_t)head * fn + p.fresh_off) * D;
    vf = reinterpret_cast<const T*>(p.kv_fresh) + b * p.fresh_bs + fn * H + (size_t)head * D * fn + p.fresh_off;
  }

  char* ring = smem + kg * S * G::STAGE;
  // V^T rows [D, 32 DT): zero, never written by the loads
  if constexpr (G::DT * 32 > D) {
    constexpr int W4 = (G::DT * 32 - D) * BKV * ES / 4;
    for (int i = threadIdx.x; i < KG * S * W4; i += 256)
      reinterpret_cast<unsigned*>(smem + (i / W4) * G::STAGE + 2 * G::TB)[i % W4] = 0u;
    __syncthreads();
  }

  // Load slot i of this wave is the tile pair's 1 KB load j = qg + QG i (K
  // first, then V^T; past the last one again an earlier slot, the same bytes to
  // the same place, so that every wave counts LPW loads); the lane fetches
  // chunk ch of row `row` (K: the row's key is kperm(row) in bf16).  off: its
  // element offset from the tile's first key in the stale buffer.
  auto load_of = [&](int i) __attribute__((always_inline)) {
    return qg + QG * i < G::NL ? qg + QG * i : qg + QG * (i - 1);
  };
  auto row_of = [&](int j, int ln) __attribute__((always_inline)) {
    return j < G::NL / 2 ? (j * 64 + ln) / G::KCH : ((j - G::NL / 2) * 64 + ln) / G::VCH;
  };
  auto chunk_of = [&](int j, int ln, int row) __attribute__((always_inline)) {
    return j < G::NL / 2 ? unswizzle<G::KCH, G::KP>(j * 64 + ln - row * G::KCH, row)
                         : unswizzle<G::VCH, G::VP>((j - G::NL / 2) * 64 + ln - row * G::VCH, row);
  };
  unsigned off[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int j = load_of(i), row = row_of(j, lane), ch = chunk_of(j, lane, row);
    off[i] = (unsigned)((j < G::NL / 2 ? (F32 ? row : kperm(row)) * D : row * n_kv) + ch * EPC);
  }
  auto issue = [&](int t, int st) __attribute__((always_inline)) {
    const int n0 = t * BKV;
    auto load = [&](const T* src, int j) __attribute__((always_inline)) {
      __builtin_amdgcn_global_load_lds((const ORCH_GLB void*)src, (ORCH_LDS void*)(ring + st * G::STAGE + j * 1024),
                                       16, 0, 0);
    };
    if (n0 + BKV <= fb || n0 >= fb + nf) {
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        const int j = load_of(i);
        load((j < G::NL / 2 ? ks + (size_t)n0 * D : vs + n0) + off[i], j);
      }
    } else {
      // a tile with fresh keys, perhaps across the band's edge: a chunk's keys
      // are all fresh or all stale.  (The empty asm keeps the lane's rows and
      // chunks from being held in registers through the loop.)
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        const int j = load_of(i), row = row_of(j, ln), e = chunk_of(j, ln, row) * EPC;
        const bool isk = j < G::NL / 2;
        const int n = n0 + (isk ? (F32 ? row : kperm(row)) : e);
        const bool fresh = (unsigned)(n - fb) < (unsigned)nf;
        load(isk ? (fresh ? kf + (size_t)(n - fb) * D : ks + (size_t)n * D) + e
                 : (fresh ? vf + (size_t)row * fn + (n - fb) : vs + (size_t)row * n_kv + n), j);
      }
    }
  };

  // this lane's query (B operand): channels KPC c + EPC h .. + EPC
  const int qrow = min(q0 + lc, p.n_q - 1);
  const T* qp = reinterpret_cast<const T*>(p.q) + (((size_t)b * p.heads + head) * p.n_q + qrow) * D;
  frag qf[G::NC];
#pragma unroll
  for (int c = 0; c < G::NC; ++c) qf[c] = *reinterpret_cast<const frag*>(qp + G::KPC * c + EPC * h);
  const float scale = p.q_scaled ? 1.0f : 1.4426950408889634f / sqrtf((float)D);  // log2(e) / sqrt(d)

  // fragment reads (A operand: row lane & 31, chunk 2 c + h); with XOR the
  // chunk's offset is one XOR of the first one's
  constexpr bool KX = (G::KCH & (G::KCH - 1)) == 0;
  int k_rd[KX ? 1 : G::NC];
#pragma unroll
  for (int c = 0; c < (KX ? 1 : G::NC); ++c) k_rd[c] = (lc * G::KCH + swizzle<G::KCH, G::KP>(2 * c + h, lc)) * 16;
  const int v_rd = G::TB + (lc * G::VCH + swizzle<G::VCH, G::VP>(h, lc)) * 16;
  auto k_at = [&](int c) __attribute__((always_inline)) { return KX ? k_rd[0] ^ (32 * c) : k_rd[c]; };
  auto v_at = [&](int x, int t) __attribute__((always_inline)) { return (v_rd ^ (32 * x)) + t * 32 * G::VCH * 16; };
  static_assert(32 / G::VP % G::VCH == 0, "the swizzle repeats every 32 rows");
  static_assert(G::TB % (16 * G::VCH) == 0, "V^T rows start at multiples of their size");

  f32x16 o[G::DT];
#pragma unroll
  for (int t = 0; t < G::DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  // (the lowest finite number, not -infinity: where every score of a tile is
  // -infinity, exp2(score - max) is then 0 and not the NaN of inf - inf)
  float m_run = -FLT_MAX, l_run = 0.0f;
  auto is_huge = [](float m) __attribute__((always_inline)) { return fabsf(m) > 0x1p20f && fabsf(m) <= FLT_MAX; };
  bool huge = true;   // of any query of the wave

  const f32x16 zero16 = {};
  // one K fragment's MFMAs of the score chain
  auto qk = [&](const frag& k, int c, f32x16& sc) __attribute__((always_inline)) {
    if constexpr (F32) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sc = __builtin_amdgcn_mfma_f32_32x32x2f32(k[e], qf[c][e], c == 0 && e == 0 ? zero16 : sc, 0, 0, 0);
    } else {
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, qf[c], c == 0 ? zero16 : sc, 0, 0, 0);
    }
  };
  // the largest of a query's 32 scores, in log2 units
  auto query_max = [&](const f32x16& v) __attribute__((always_inline)) {
    float mx = fmaxf(fmaxf(v[0], v[1]), v[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) mx = fmaxf(fmaxf(mx, v[r]), v[r + 1]);
    return max_xhalf(fmaxf(mx, v[15])) * scale;
  };
  // Softmax and PV product of the tile in stage st (scores sc, their max mx);
  // with NEXT, the scores of the tile in stage nst, into sn, and mx becomes
  // their max.  A lone wave on its SIMD has to cover its own VALU work, so the
  // emission order is fixed slot by slot (a scheduling fence after each): the
  // next tile's score MFMAs between the first EPC probabilities, then the PV
  // MFMAs of each EPC keys between the next EPC probabilities, the last ones
  // before the next max.
  auto tile = [&](auto next_c, int st, f32x16& sc, float& mx, int nst, f32x16& sn) __attribute__((always_inline)) {
    constexpr bool NEXT = decltype(next_c)::value;
    const char* base = ring + st * G::STAGE;
    // Running max, raised only where a query's scores pass it by 8 in log2
    // units (each query decides for itself, so its sums do not depend on its
    // neighbours); probabilities then reach 2^8, in fp32.
    const bool up = !(mx <= m_run + 8.0f);
    if (__builtin_expect(__any(up), 0)) {
      const float mn = up ? mx : m_run;
      const float alpha = up ? __builtin_amdgcn_exp2f(m_run - mn) : 1.0f;
      m_run = mn;
      huge = __any(is_huge(mn));
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < G::DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
    }
    // Past 2^20 the rounding of max = score * scale is no longer small against 1,
    // and the fused score * scale - max below would show it (scores of the lowest
    // finite number: an exponent of +-2^102 where 0 is meant).  There the
    // difference is taken of the rounded product, so that equal scores cancel.
    float m_sub = m_run;
    if (__builtin_expect(huge, 0)) {
#pragma clang fp contract(off)
      const bool big = is_huge(m_run);
      const float inv = 1.0f / scale;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float s = sc[r] * scale;
        sc[r] = big ? (s - m_run) * inv : sc[r];
      }
      m_sub = big ? 0.0f : m_run;
    }
    frag kn[NEXT ? G::NC : 1], v[2][G::DT], hi[2], lo[2];
    if constexpr (NEXT) {
#pragma unroll
      for (int c = 0; c < G::NC; ++c) kn[c] = *reinterpret_cast<const frag*>(ring + nst * G::STAGE + k_at(c));
    }
#pragma unroll
    for (int t = 0; t < G::DT; ++t) v[0][t] = *reinterpret_cast<const frag*>(base + v_at(0, t));
    __builtin_amdgcn_sched_barrier(0);
    // probability e of key chunk x, and the one before it into the sum and the
    // MFMA operands (an exponential's result is not ready at once)
    float sum = 0.0f, pv[EPC];
    auto take = [&](auto xc, int e) __attribute__((always_inline)) {
      constexpr int x = decltype(xc)::value;
      sum += pv[e];
      if constexpr (F32) {
        hi[x & 1][e] = pv[e];
      } else {
        const unsigned top = __float_as_uint(pv[e]) & 0xffff0000u;
        hi[x & 1][e] = __builtin_bit_cast(bf16, (unsigned short)(top >> 16));
        lo[x & 1][e] = (bf16)fmaf(pv[e], kUp, -__uint_as_float(top));
      }
    };
    auto prob = [&](auto xc, int e) __attribute__((always_inline)) {
      constexpr int x = decltype(xc)::value;
      pv[e] = __builtin_amdgcn_exp2f(fmaf(sc[EPC * x + e], scale, -m_sub));
      if (e > 0) take(xc, e - 1);
      if (e == EPC - 1) take(xc, e);
    };
    static_for<0, EPC>([&](auto gc) {
      constexpr int g = decltype(gc)::value;
      if constexpr (NEXT)
        static_for<g * G::NC / EPC, (g + 1) * G::NC / EPC>([&](auto cc) { qk(kn[decltype(cc)::value], decltype(cc)::value, sn); });
      prob(std::integral_constant<int, 0>{}, g);
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<0, G::NX>([&](auto xc) {
      constexpr int x = decltype(xc)::value, cur = x & 1;
      if constexpr (x + 1 < G::NX) {
#pragma unroll
        for (int t = 0; t < G::DT; ++t) v[cur ^ 1][t] = *reinterpret_cast<const frag*>(base + v_at(x + 1, t));
      }
      constexpr int NM = (F32 ? 4 : 2) * G::DT;    // O^T tile m % DT, part m / DT (hi, lo; or key e)
      static_for<0, EPC>([&](auto gc) {
        constexpr int g = decltype(gc)::value;
        static_for<g * NM / EPC, (g + 1) * NM / EPC>([&](auto mc) {
          constexpr int m = decltype(mc)::value, t = m % G::DT, q = m / G::DT;
          if constexpr (F32) o[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[cur][t][q], hi[cur][q], o[t], 0, 0, 0);
          else o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[cur][t], q ? lo[cur] : hi[cur], o[t], 0, 0, 0);
        });
        if constexpr (x + 1 < G::NX) prob(std::integral_constant<int, (x + 1 < G::NX ? x + 1 : 0)>{}, g);
        else if constexpr (NEXT && g == 0) mx = query_max(sn);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    l_run += sum;
  };

  // Key group kg's tiles kg, kg + KG, ...; the groups' counts differ by at most
  // one (launcher: at least one tile each), and a group that is one short loads
  // and scores its last tile again, so that all waves meet the same barriers, and
  // leaves it out (a probability of zero would not do: 0 V is a NaN where V is
  // infinite).  At the top of iteration i tile
  // i's scores are formed and tile i + 1 is waited for; the barrier also frees
  // the stage of tile i - 1 for tile i + 2.
  const int nt = n_kv / BKV, NIT = (nt + KG - 1) / KG;
  const bool full = kg + KG * (NIT - 1) < nt;
  // (two parts: the tiles kg, kg + 2 KG, ..., `first` of them, then kg + KG, kg + 3 KG, ...)
  const int first = (nt - kg + 2 * KG - 1) / (2 * KG);
  auto tile_at = [&](int i) __attribute__((always_inline)) {
    const int j = full || i + 1 < NIT ? i : NIT - 2;
    if constexpr (PARTS == 1) return kg + KG * j;
    else return kg + (j < first ? 2 * KG * j : KG + 2 * KG * (j - first));
  };
  f32x16 o_first[PARTS == 2 ? G::DT : 1];
  float m_first = 0.0f, l_first = 0.0f;
  f32x16 s0, s1;
  issue(tile_at(0), 0);
  if (1 < NIT) issue(tile_at(1), 1);
  if (1 < NIT) wait_vmcnt<LPW>();
  else wait_vmcnt<0>();
  lds_barrier();
#pragma unroll
  for (int c = 0; c < G::NC; ++c) qk(*reinterpret_cast<const frag*>(ring + k_at(c)), c, s0);
  float mx = query_max(s0);
  auto iterate = [&](int i, f32x16& sc, f32x16& sn) __attribute__((always_inline)) {
    wait_vmcnt<0>();
    lds_barrier();
    if (i + 2 < NIT) issue(tile_at(i + 2), (i + 2) % S);
    tile(std::true_type{}, i % S, sc, mx, (i + 1) % S, sn);
    if constexpr (PARTS == 2) {
      if (i + 1 == first) {
        m_first = m_run;
        l_first = l_run;
        m_run = -FLT_MAX;
        l_run = 0.0f;
        huge = true;
#pragma unroll
        for (int t = 0; t < G::DT; ++t) {
          o_first[t] = o[t];
          o[t] = zero16;
        }
      }
    }
  };
  auto last = [&](int i, f32x16& sc) __attribute__((always_inline)) {
    if (full) tile(std::false_type{}, i % S, sc, mx, 0, sc);
  };
  int i = 0;
  for (; i + 2 < NIT; i += 2) {
    iterate(i, s0, s1);
    iterate(i + 1, s1, s0);
  }
  if (i + 1 < NIT) {
    iterate(i, s0, s1);
    last(i + 1, s1);
  } else {
    last(i, s0);
  }

  l_run += __shfl_xor(l_run, 32, kWave);
  if constexpr (PARTS == 2) l_first += __shfl_xor(l_first, 32, kWave);
  // The parts of a query, [register][lane], merged by key group 0 in the order of
  // their first tiles: part j is group j % KG's, its j / KG-th.
  f32x16 om[G::DT];
  float m = PARTS == 2 ? m_first : m_run, l = PARTS == 2 ? l_first : l_run;
#pragma unroll
  for (int t = 0; t < G::DT; ++t) om[t] = PARTS == 2 ? o_first[PARTS == 2 ? t : 0] : o[t];
  auto merge = [&](float m2, float l2, auto&& o2) __attribute__((always_inline)) {
    const float mn = fmaxf(m, m2);
    const float f1 = __builtin_amdgcn_exp2f(m - mn), f2 = __builtin_amdgcn_exp2f(m2 - mn);
    m = mn;
    l = l * f1 + l2 * f2;
#pragma unroll
    for (int t = 0; t < G::DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) om[t][r] = om[t][r] * f1 + o2(t, r) * f2;
  };
  if constexpr (KG > 1) {
    lds_barrier();
    if (kg > 0) {
      auto put = [&](int j, float m2, float l2, const f32x16* o2) __attribute__((always_inline)) {
        float* part = reinterpret_cast<float*>(smem + (((kg - 1) * PARTS + j) * QG + qg) * G::PART) + lane;
#pragma unroll
        for (int t = 0; t < G::DT; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) part[(16 * t + r) * 64] = o2[t][r];
        part[G::DT * 1024] = m2;
        part[G::DT * 1024 + 64] = l2;
      };
      put(0, m, l, om);
      if constexpr (PARTS == 2) put(1, m_run, l_run, o);
    }
    __syncthreads();
    if (kg > 0) return;
  }
#pragma unroll
  for (int j = 1; j < KG * PARTS; ++j) {
    if (j % KG == 0) {
      merge(m_run, l_run, [&](int t, int r) __attribute__((always_inline)) { return o[t][r]; });
    } else {
      const float* part = reinterpret_cast<const float*>(smem + ((j % KG - 1) * PARTS + j / KG) * QG * G::PART + qg * G::PART) + lane;
      merge(part[G::DT * 1024], part[G::DT * 1024 + 64],
            [&](int t, int r) __attribute__((always_inline)) { return part[(16 * t + r) * 64]; });
    }
  }
  // a lane holds channels 32 t + 8 g + 4 h .. + 4 of its query
  if (q0 + lc < p.n_q) {
    const float inv = 1.0f / l;
    T* orow = reinterpret_cast<T*>(p.out) + ((size_t)b * p.n_q + q0 + lc) * H + (size_t)head * D;
    typedef T quad __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int t = 0; t < G::DT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d = 32 * t + 8 * g + 4 * h;
        if (32 * t + 8 * g + 8 <= D) {
          quad v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = from_f<T>(om[t][4 * g + e] * inv);
          *reinterpret_cast<quad*>(orow + d) = v;
        }
      }
  }
}

// ---------------------------------------------------------------------------
// Shapes the kernel takes: whole 32-key tiles, 16-byte chunks of Q, K and V^T
// all fresh or all stale, element offsets inside a head in 31 bits.
bool attention_general_ok(const AttnParams& p, int dtype) {
  const int epc = dtype == kBF16 ? 8 : 4;
  auto a16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  if (dtype == kBF16 && !(p.d == 32 || p.d == 64 || p.d == 80 || p.d == 96 || p.d == 128)) return false;
  if (p.n_kv % gen_attn::BKV || (long long)p.n_kv * p.d >= (1ll << 31)) return false;
  if (!a16(p.q) || !a16(p.kv_stale) || !a16(p.out) || p.stale_bs % epc) return false;
  return p.n_fresh == 0 ||
         (a16(p.kv_fresh) && p.fresh_bs % epc == 0 && p.fresh_begin % epc == 0 && p.n_fresh % epc == 0 &&
          p.fresh_n % epc == 0 && p.fresh_off % epc == 0 && (long long)p.fresh_n * p.d < (1ll << 31));
}

template <typename T, int D, int KG, int PARTS = 1>
static hipError_t launch_kg(const AttnParams& p, hipStream_t s) {
  using G = gen_attn::Geo<T, D, KG, PARTS>;
  auto kern = attn_general_kernel<T, D, KG, PARTS>;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(ceil_div(p.n_q, 32 * G::QG) * p.heads * p.B), dim3(256), G::LDS, s, p);
  return hipGetLastError();
}

// bf16 heads of 64 channels: the other kernel's 128-query tiles leave CUs idle
// where queries are few and walk all keys in one chain where those are too few
// to cut (or merge the parts in a second launch).  Measured here / there, us: 6
// heads, 96 queries x 256 keys 5.2 / 7.2, x 576 7.3 / 10.8, x 1024 9.3 / 11.5, x 2304
// 16.2 / 16.0; 24 (branch, head) x 576 queries (432 waves) x 1024 keys 14.3 / 17.1; 32 x
// 576 queries (576 waves) x 576 keys 12.9 / 11.7.
bool attention_general_better(const AttnParams& p, int dtype) {
  return dtype == kBF16 && p.d == 64 && !p.fixed_order && p.n_kv <= 1024 &&
         (long long)ceil_div(p.n_q, 32) * p.heads * p.B <= 512 && attention_general_ok(p, dtype);
}

// Key groups per workgroup.  A wave of 32 queries is bound by its own chain
// (0.8 us per 32 keys at d = 128), so the keys are split as far as all
// workgroups stay resident at once; past that a split only shares each K/V tile
// among fewer queries.  Measured with 1 / 2 / 4 groups, us: bf16 d = 80 (two
// workgroups of two groups a CU, one of four), 256 waves x 1024 keys 26.3 / 15.7 /
// 12.2; 512 waves 27.4 / 17.4 / 23.5; 1024 waves 29.8 / 25.7 / 44.9; 2048 waves 44.7 /
// 47.5 / 87.0; d = 128 (one of two groups), 512 waves 31.7 / 21.7, 1024 waves 35.7 /
// 42.4.
// fp32 takes the same groups whatever the number of queries, so that the order of a
// query's sums is fixed by its keys: four at d = 32 (or two of two parts each, once
// four are not resident), else two (one at d = 128, where two do not fit).  d =
// 72 with 1 / 2 groups: 512 waves 93 / 53, 1024 waves 96 / 103.
template <typename T, int D, int KG>
static bool resident(const AttnParams& p) {
  using G = gen_attn::Geo<T, D, KG>;
  return G::FITS && p.n_kv / gen_attn::BKV >= KG &&   // a tile for every group
         (long long)ceil_div(p.n_q, 32 * G::QG) * p.heads * p.B <= 256 * (160 * 1024 / G::LDS);
}

template <typename T, int D>
static hipError_t launch_d(const AttnParams& p, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    if constexpr (gen_attn::Geo<T, D, 4>::FITS)
      if (!p.fixed_order && resident<T, D, 4>(p)) return launch_kg<T, D, 4>(p, s);
    if (!p.fixed_order && resident<T, D, 2>(p)) return launch_kg<T, D, 2>(p, s);
  } else if constexpr (gen_attn::Geo<T, D, 2>::FITS) {
    const int nt = p.n_kv / gen_attn::BKV;
    if constexpr (gen_attn::Geo<T, D, 4>::FITS)
      if (nt >= 4) return resident<T, D, 4>(p) ? launch_kg<T, D, 4>(p, s) : launch_kg<T, D, 2, 2>(p, s);
    if (nt >= 2) return launch_kg<T, D, 2>(p, s);
  }
  return launch_kg<T, D, 1>(p, s);
}

// Whether waves share a query's keys at this shape, if the call leaves them free to.
bool attention_general_shares(int B, int heads, int n_q, int n_kv, int d, int dtype) {
  AttnParams p{};
  p.B = B; p.heads = heads; p.n_q = n_q; p.n_kv = n_kv; p.d = d;
  if (dtype != kBF16 || !attention_general_ok(p, dtype)) return false;
  switch (d) {
    case 32: return resident<bf16, 32, 2>(p);
    case 64: return attention_general_better(p, dtype) || (!attention_uses_mfma(d, n_kv, dtype) && resident<bf16, 64, 2>(p));
    case 80: return resident<bf16, 80, 2>(p);
    case 96: return resident<bf16, 96, 2>(p);
    case 128: return resident<bf16, 128, 2>(p);
  }
  return false;
}

hipError_t launch_attention_general(const AttnParams& p, int dtype, hipStream_t s) {
  if (dtype == kBF16) {
    switch (p.d) {
      case 32: return launch_d<bf16, 32>(p, s);
      case 64: return launch_d<bf16, 64>(p, s);
      case 80: return launch_d<bf16, 80>(p, s);
      case 96: return launch_d<bf16, 96>(p, s);
      case 128: return launch_d<bf16, 128>(p, s);
    }
  } else {
    switch (p.d) {
      case 32: return launch_d<float, 32>(p, s);
      case 64: return launch_d<float, 64>(p, s);
      case 72: return launch_d<float, 72>(p, s);
      case 80: return launch_d<float, 80>(p, s);
      case 96: return launch_d<float, 96>(p, s);
      case 128: return launch_d<float, 128>(p, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace orch
