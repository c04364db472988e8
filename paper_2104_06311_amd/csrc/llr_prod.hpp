// Exact and max-log LLRs from the factors of a product constellation, one thread per symbol;
// also every constellation of up to 16 points (one factor if it has no more).
//
// With x_l = (x_A(l_A), x_B(l_B), ...) over disjoint groups of label bits and coordinates
// (prep.hip finds and verifies them on every call), exp(-c ||y - x_l||^2) is a product over
// the groups, the sums over the other groups cancel from S0 / S1, and the LLRs of a group's
// bits need its own points only: 2 x 16 for 256-QAM instead of 256, 2 x 8 for the 4D product
// of two 8-PSK instead of 64.
//
// Per group and symbol: squared distances of its 2^MF <= 16 points in difference form, then
//   max-log:              L_b = cnat (min_{b=1} d2 - min_{b=0} d2), FP64 distances;
//   exact, M <= 16, and groups of up to 4 points: FP64 distances; per label subset the smallest
//     (FP64) and the FP32 sum of 2^-(c (d2 - min)), L_b = cnat (min1 - min0) + ln (sum0 / sum1), the
//     logarithm in FP64 for M <= 16 (not for 4-point groups of products in two and four dimensions, see
//     subset_llr);
//   exact, 8 and 16 points of M >= 32 (where the general path's scores are FP32): FP32
//     distances, one exponential per point relative to the nearest, the subset sums by a tree,
//     L_b = ln (S0 / S1).  A bit whose smaller sum fell below 2^-100 takes its subsets' smallest
//     distances in FP64 and their sums relative to them.
// A symbol of M >= 32 whose distances reach too far for FP32 (in_range) is marked, and demapped in FP64
// altogether by rest_columns; so is every symbol of a call whose c or points are outside the FP32 form's
// range (all_symbols).
// A non-finite received value gives NaN LLRs, as on the general path.
//
// Bound by memory for up to 4 points a factor (4e6 symbols of 16-QAM, a whole call: 207.7 ->
// 26.9 us, 3.6e12 B/s of its 24 bytes a symbol) and by vector instructions, about 4.4 cycles
// each, for 16 (1e6 symbols of 256-QAM: 71.3 -> 36.9 us).  LLRs are no further from 64-bit ones
// than before (relative 2-norm 2.5e-8 and 5.7e-8 against 2.5e-8 and 2.6e-7).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "fp64_form.hpp"
#include "gmi_terms.hpp"
#include "llr_kernels.hpp"

namespace md {
namespace prodk {

constexpr int kProdThreads = 256;
constexpr float kLn2f = 0.69314718055994530942f;

typedef const __attribute__((address_space(4))) int ConstInt;        // uniform: scalar loads
typedef const __attribute__((address_space(4))) double ConstDouble;
typedef const __attribute__((address_space(4))) float ConstFloat;

// A symbol's received vector in registers (two or four coordinates), read by a coordinate that is
// the same for the whole wavefront.
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float pick(float2v v, int co) { return co ? v.y : v.x; }
__device__ __forceinline__ float pick(float4v v, int co) {
  const float lo = (co & 1) ? v.y : v.x, hi = (co & 1) ? v.w : v.z;
  return (co & 2) ? hi : lo;
}
template <class V>
__device__ __forceinline__ V load_row(const float* __restrict__ p) {
  V v;
  __builtin_memcpy(&v, p, sizeof(V));      // 4-byte aligned
  return v;
}

struct ProdTables {
  ConstInt* fd;         // the factor's description
  ConstDouble* td;
  ConstFloat* tf;
};

__device__ __forceinline__ double min_r(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float min_r(float a, float b) { return fminf(a, b); }

// Squared distances of the group's points; `nonfinite` collects 0 * y (NaN for inf and NaN).  Groups of
// two and four points take several coordinates at a time: one by one each waited for its index, then
// for its points (M = 2, D = 30, 1000 symbols: 29 us a call, 25 so).
template <int MF, class R>
__device__ __forceinline__ void distances(const ProdTables& T, const float* __restrict__ row, R (&d2)[1 << MF],
                                          float* nonfinite) {
  constexpr int U = MF == 1 ? 8 : (MF == 2 ? 4 : 1);
  const int df = T.fd[1];
  auto coords = [&](int i, auto first, auto count) {
    constexpr int C = decltype(count)::value;
    int co[C];
    float yf[C];
    R x[C][1 << MF];
#pragma unroll
    for (int u = 0; u < C; ++u) co[u] = T.fd[8 + i + u];
#pragma unroll
    for (int u = 0; u < C; ++u) {
      yf[u] = row[co[u]];
#pragma unroll
      for (int p = 0; p < (1 << MF); ++p) {
        if constexpr (sizeof(R) == 8) x[u][p] = T.td[16 * co[u] + p];
        else x[u][p] = T.tf[16 * co[u] + p];
      }
    }
#pragma unroll
    for (int u = 0; u < C; ++u) {
      *nonfinite = fmaf(yf[u], 0.0f, *nonfinite);
      const R y = static_cast<R>(yf[u]);
#pragma unroll
      for (int p = 0; p < (1 << MF); ++p) {
        const R diff = y - x[u][p];
        if (decltype(first)::value && u == 0) d2[p] = diff * diff;
        else d2[p] = fma(diff, diff, d2[p]);
      }
    }
  };
  typedef std::integral_constant<int, 1> One;
  coords(0, std::true_type{}, One{});
  int i = 1;
  if constexpr (U > 1)
    for (; i + U <= df; i += U) coords(i, std::false_type{}, std::integral_constant<int, U>{});
  for (; i < df; ++i) coords(i, std::false_type{}, One{});
}

// Smallest distance of the label-0 and label-1 subset of bit b.
template <int MF, class R>
__device__ __forceinline__ void subset_min(const R (&d2)[1 << MF], int b, R* m0, R* m1) {
  R a[2] = {d2[0], d2[1 << b]};
#pragma unroll
  for (int p = 1; p < (1 << MF); ++p)
    if (p != (1 << b)) a[(p >> b) & 1] = min_r(a[(p >> b) & 1], d2[p]);
  *m0 = a[0];
  *m1 = a[1];
}

// Exact LLR of bit b with every subset relative to its own smallest distance (whose term is 1:
// a subset of one point needs no exponential, one of two points a single one).  Differences are
// scaled in FP64 and rounded last: neither they nor c need lie in the FP32 range, and the smallest
// distance's own term is 1 however large c times it is.
//
// LOG64: the logarithm in FP64 (some 17 instructions; its 1e-10 is far below the sums' 6e-8).  FP32
// logarithms add about what two FP32 sums carry: 8-PSK at 2 dB 3.34e-8 (relative 2-norm) against 3.24e-8,
// an unstructured M = 4 at -4 dB 5.98e-8 against 5.33e-8; but they take 26 us of 4e6 16-QAM symbols where
// FP64 ones take 34, and the sums of a 4-point group are of two terms instead of 8: 3.30e-8 at 2 dB,
// 3.90e-8 over all 16 points with FP64 logarithms.
// mn: the subsets' smallest distances.
template <int MF, bool LOG64>
__device__ __forceinline__ float subset_llr(const double (&d2)[1 << MF], int b, double c, double cnat, double (&mn)[2]) {
  subset_min<MF>(d2, b, &mn[0], &mn[1]);
  // (a point that is not finite, M = 2: NaN, as a sum of its terms would be)
  if constexpr (MF == 1) return static_cast<float>(fma(cnat, mn[1] - mn[0], 0.0 * (mn[0] + mn[1])));
  float s[2] = {0.0f, 0.0f};
  if constexpr (MF == 2) {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int p = v << b, o = p | (2 >> b);       // the subset's two points
      s[v] = 1.0f + __builtin_amdgcn_exp2f(static_cast<float>(-c * fabs(d2[p] - d2[o])));
    }
  } else {
#pragma unroll
    for (int p = 0; p < (1 << MF); ++p)
      s[(p >> b) & 1] += __builtin_amdgcn_exp2f(static_cast<float>(c * (mn[(p >> b) & 1] - d2[p])));
  }
  double lg;
  if constexpr (LOG64) lg = fp64::log_ratio<9, MF == 2>(s[0], s[1]);
  else lg = static_cast<double>(kLn2f * (__builtin_amdgcn_logf(s[0]) - __builtin_amdgcn_logf(s[1])));
  return static_cast<float>(fma(cnat, mn[1] - mn[0], lg));
}

enum { PROD_MAXLOG = 0, PROD_DOUBLE = 1, PROD_FLOAT = 2 };
// FP32 distances for factors of 8 and 16 points in PROD_FLOAT; with fewer the exponentials they
// save are few, and FP64 costs as little.
template <int MODE, int MF>
constexpr bool kFloat = MODE == PROD_FLOAT && MF >= 3;
template <int MODE, int MF>
using Real = typename std::conditional<kFloat<MODE, MF>, float, double>::type;

// How far a symbol's factors reach, in base-2 units: the sum of their nearest points' scores, and the
// largest distance from there to a subset's best point (FP32 form: where a sum fell below 2^-100).
struct Reach {
  float top = 0.0f, beyond = 0.0f;
};
// FP32 distances carry 3 roundings of their score, which must stay small beside 1 for the nearest
// points; and beyond 575 units the general path's FP32 windows end as well.  Not for NaN or infinity.
__device__ __forceinline__ bool in_range(const Reach& r) { return r.top <= 256.0f && r.top + r.beyond <= 575.0f; }

// The LLR of bit b when one of its sums is too small: FP64 smallest distances (dist64(p): the
// distance of point p), FP32 sums relative to the FP32 ones (rounded scores: good within in_range).
template <int MF, class F>
__device__ __forceinline__ float wide_llr(const float (&d2)[1 << MF], int b, float cf, double cnat, F dist64, float top,
                                          Reach& reach) {
  float mf[2];
  subset_min<MF>(d2, b, &mf[0], &mf[1]);
  const float cm[2] = {cf * mf[0], cf * mf[1]};
  reach.beyond = fmaxf(reach.beyond, fmaxf(cm[0], cm[1]) - top);
  double mn[2] = {INFINITY, INFINITY};
  float s[2] = {0.0f, 0.0f};
#pragma unroll
  for (int p = 0; p < (1 << MF); ++p) {
    const int v = (p >> b) & 1;
    mn[v] = fmin(mn[v], dist64(p));
    s[v] += __builtin_amdgcn_exp2f(fmaf(-cf, d2[p], cm[v]));
  }
  const float lg = kLn2f * (__builtin_amdgcn_logf(s[0]) - __builtin_amdgcn_logf(s[1]));
  return static_cast<float>(cnat * (mn[1] - mn[0]) + static_cast<double>(lg));
}

// The LLRs of a factor's bits from its squared distances (LOG64: see subset_llr).
template <int MODE, int MF, bool LOG64, class F>
__device__ __forceinline__ void llr_from_distances(const Real<MODE, MF> (&d2)[1 << MF], double c, double cnat,
                                                   float (&L)[MF], F dist64, Reach& reach) {
  constexpr int MP = 1 << MF;
  if constexpr (MODE == PROD_MAXLOG) {
#pragma unroll
    for (int b = 0; b < MF; ++b) {
      double m0, m1;
      subset_min<MF>(d2, b, &m0, &m1);
      // (NaN points are left out, also when a subset has no others: infinitely far)
      L[b] = static_cast<float>(cnat * (fmin(m1, INFINITY) - fmin(m0, INFINITY)));
    }
  } else if constexpr (!kFloat<MODE, MF>) {
    double near = 0.0, far = 0.0;
#pragma unroll
    for (int b = 0; b < MF; ++b) {
      double mn[2];
      L[b] = subset_llr<MF, LOG64>(d2, b, c, cnat, mn);
      if (MODE == PROD_FLOAT) {
        if (b == 0) near = fmin(mn[0], mn[1]);
        far = fmax(far, fmax(mn[0], mn[1]));
      }
      __builtin_amdgcn_sched_barrier(0);       // one bit's temporaries at a time (registers)
    }
    if (MODE == PROD_FLOAT) {
      reach.top += static_cast<float>(c * near);
      reach.beyond = fmaxf(reach.beyond, static_cast<float>(c * (far - near)));
    }
  } else {
    const float cf = static_cast<float>(c);
    float dmin = d2[0];
#pragma unroll
    for (int p = 1; p < MP; ++p) dmin = fminf(dmin, d2[p]);
    const float top = cf * dmin;
    float v[MP];
#pragma unroll
    for (int p = 0; p < MP; ++p) v[p] = __builtin_amdgcn_exp2f(fmaf(-cf, d2[p], top));
    // level b: v[k] sums the 2^b consecutive labels of block k, so bit b of a label is the
    // parity of its block index
#pragma unroll
    for (int b = 0; b < MF; ++b) {
      const int cnt = MP >> b;
      float a0 = v[0], a1 = v[1];
#pragma unroll
      for (int k = 2; k < cnt; k += 2) {
        a0 += v[k];
        a1 += v[k + 1];
      }
      L[b] = fminf(a0, a1) >= 0x1p-100f ? kLn2f * __builtin_amdgcn_logf(a0 * __builtin_amdgcn_rcpf(a1))
                                        : wide_llr<MF>(d2, b, cf, cnat, dist64, top, reach);
#pragma unroll
      for (int k = 0; k < cnt / 2; ++k) v[k] = v[2 * k] + v[2 * k + 1];
    }
    reach.top += top;
  }
}

// Stores a factor's LLRs into the symbol's row: consecutive columns from `last` on (the usual
// layout) by one store, others one by one.
template <int MF>
__device__ __forceinline__ void store_llrs(const float (&L)[MF], ConstInt* fd, bool run, int last,
                                           float* __restrict__ lrow) {
  if (run) {
    float out[MF];
#pragma unroll
    for (int i = 0; i < MF; ++i) out[MF - 1 - i] = L[i];
    __builtin_memcpy(lrow + last, out, sizeof(out));
  } else {
#pragma unroll
    for (int i = 0; i < MF; ++i) lrow[fd[3 + i]] = L[i];
  }
}

// The loss term of a factor's bits.
template <int MF>
__device__ __forceinline__ float loss_of(const float (&L)[MF], ConstInt* fd, int m, uint32_t lab) {
  float t = 0.0f;
#pragma unroll
  for (int i = 0; i < MF; ++i) t += softplus_bits(((lab >> (m - 1 - fd[3 + i])) & 1u) ? L[i] : -L[i]);
  return t;
}

// One factor of a symbol, any shape.
template <int MODE, int MF, bool GMI>
__device__ __forceinline__ float factor_llr(const ProdTables& T, const float* __restrict__ row, int m, double c, double cnat,
                                            float* __restrict__ lrow, uint32_t lab, float* nonfinite, Reach& reach) {
  Real<MODE, MF> d2[1 << MF];
  distances<MF>(T, row, d2, nonfinite);
  float L[MF];
  auto dist64 = [&](int p) {
    double r = 0.0;
    for (int i = 0; i < T.fd[1]; ++i) {
      const int co = T.fd[8 + i];
      const double diff = static_cast<double>(row[co]) - T.td[16 * co + p];
      r = fma(diff, diff, r);
    }
    return r;
  };
  llr_from_distances<MODE, MF, MODE == PROD_DOUBLE>(d2, c, cnat, L, dist64, reach);
  store_llrs<MF>(L, T.fd, T.fd[7] != 0, T.fd[2 + MF], lrow);
  return GMI ? loss_of<MF>(L, T.fd, m, lab) : 0.0f;
}

// The factors as prepare() wrote them (layout in common.hpp).
struct ProdArgs {
  const int* prod;
  const double* ptab;
  const float* ptabf;
};

struct SymbolArgs {
  const float* y;
  float* llr;
  const uint32_t *gmi_tx, *gmi_labels;
  float* gmi_terms;
  uint64_t* left;         // one bit per symbol
  int* any_left;          // set when a bit is
  int64_t N;
  int m, D;
  double c, cnat;
  float start;            // 0, or NaN when the labels are broken
  bool fp32_ok;           // the FP32 form may be used
};

template <bool GMI>
__device__ __forceinline__ uint32_t sent_label(const SymbolArgs& A, int64_t n, float* term) {
  if constexpr (!GMI) return 0u;
  const uint32_t t = A.gmi_tx[n];
  const bool ok = t < (1u << A.m);
  *term = ok ? 0.0f : __builtin_nanf("");
  return A.gmi_labels[ok ? t : 0u];
}

// Marks the symbols left to rest_columns, one bit each (a wavefront's 64 symbols are one aligned run);
// returns the loss term, NaN where it will be taken from the final LLRs.  *some: whether any was marked.
__device__ __forceinline__ float mark_left(const SymbolArgs& A, int64_t n, const Reach& reach, float nonfinite, float term,
                                           bool* some) {
  const bool out = !(A.fp32_ok && in_range(reach)) && nonfinite == 0.0f;
  const uint64_t mask = __ballot(out);
  if ((n & 63) == 0) A.left[n >> 6] = mask;
  *some = *some || mask != 0;
  return out ? __builtin_nanf("") : term;
}

template <bool GMI>
__device__ __forceinline__ void finish_symbol(const SymbolArgs& A, int64_t n, float nonfinite, float term) {
  if (!(nonfinite == 0.0f)) {
    for (int k = 0; k < A.m; ++k) A.llr[n * A.m + k] = __builtin_nanf("");
    term = __builtin_nanf("");
  }
  if constexpr (GMI) A.gmi_terms[n] = term;
}

// All symbols of the thread when the constellation is NF factors of MF bits and DF coordinates
// each, DT = NF DF coordinates in all: points, columns and coordinates are read once, ahead of
// the loop (scalar registers).  Reading them per symbol and factor, in a chain of dependent
// scalar loads, made the kernel take 49 instead of 24 us for 4e6 symbols of 16-QAM, and staging
// the rows through LDS 54 us.
template <int MODE, int MF, int NF, int DF, bool GMI>
__device__ __forceinline__ void fixed_symbols(const ProdTables& T0, ConstInt* head, const SymbolArgs& A) {
  constexpr int DT = NF * DF, MP = 1 << MF;
  typedef Real<MODE, MF> R;
  R tab[NF][DF][MP];
  int co[NF][DF], last[NF];
  ConstInt* fd[NF];
  bool run = true;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    fd[f] = head + kProdHead + kProdFactor * f;
    last[f] = fd[f][2 + MF];
    run = run && fd[f][7] != 0;
#pragma unroll
    for (int i = 0; i < DF; ++i) {
      co[f][i] = fd[f][8 + i];
#pragma unroll
      for (int p = 0; p < MP; ++p) {
        if constexpr (sizeof(R) == 8) tab[f][i][p] = T0.td[16 * co[f][i] + p];
        else tab[f][i][p] = T0.tf[16 * co[f][i] + p];
      }
    }
  }
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kProdThreads;
  int64_t n = static_cast<int64_t>(blockIdx.x) * kProdThreads + threadIdx.x;
  typedef typename std::conditional<DT == 2, float2v, float4v>::type Row;
  Row next = {};
  if (n < A.N) next = load_row<Row>(A.y + n * DT);
  bool some = false;
  for (; n < A.N; n += stride) {
    const Row yv = next;
    if (n + stride < A.N) next = load_row<Row>(A.y + (n + stride) * DT);
    float nonfinite = A.start, term = 0.0f;
#pragma unroll
    for (int d = 0; d < DT; ++d) nonfinite = fmaf(yv[d], 0.0f, nonfinite);
    const uint32_t lab = sent_label<GMI>(A, n, &term);
    Reach reach;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      R d2[MP];
#pragma unroll
      for (int i = 0; i < DF; ++i) {
        const R yd = static_cast<R>(pick(yv, co[f][i]));
#pragma unroll
        for (int p = 0; p < MP; ++p) {
          const R diff = yd - tab[f][i][p];
          d2[p] = i == 0 ? diff * diff : fma(diff, diff, d2[p]);
        }
      }
      float L[MF];
      auto dist64 = [&](int p) {
        double r = 0.0;
#pragma unroll
        for (int i = 0; i < DF; ++i) {
          const double diff = static_cast<double>(pick(yv, co[f][i])) - T0.td[16 * co[f][i] + p];
          r = fma(diff, diff, r);
        }
        return r;
      };
      constexpr bool log64 = MODE == PROD_DOUBLE && (NF == 1 || MF > 2);
      llr_from_distances<MODE, MF, log64>(d2, A.c, A.cnat, L, dist64, reach);
      store_llrs<MF>(L, fd[f], run, last[f], A.llr + n * A.m);
      if constexpr (GMI) term += loss_of<MF>(L, fd[f], A.m, lab);
    }
    if constexpr (MODE == PROD_FLOAT) term = mark_left(A, n, reach, nonfinite, term, &some);
    finish_symbol<GMI>(A, n, nonfinite, term);
  }
  if (some) *A.any_left = 1;
}

// Whether constellations of m label bits in two or four coordinates come here: MB = 0, the product kernel
// (M <= 16 exact; products of 128 to kProdMaxM points; max-log both), or the kernel for 2^MB points.
template <int MODE, int MB>
constexpr bool comes_here(int m) {
  if (MB != 0) return m == MB;
  return (MODE != PROD_FLOAT && (1 << m) <= kSmallM) || (MODE != PROD_DOUBLE && m >= 7 && (1 << m) <= kProdMaxM);
}

// False: no loop of its own for this shape.
template <int MODE, int NF, int DF, bool GMI, int MB, int MF = 1>
__device__ __forceinline__ bool fixed_shape(int mf, const ProdTables& T, ConstInt* head, const SymbolArgs& A) {
  if constexpr (comes_here<MODE, MB>(NF * MF))
    if (mf == MF) {
      fixed_symbols<MODE, MF, NF, DF, GMI>(T, head, A);
      return true;
    }
  if constexpr (MF < kProdMaxBits) return fixed_shape<MODE, NF, DF, GMI, MB, MF + 1>(mf, T, head, A);
  return false;
}

// GMI: also the loss term of every symbol (NaN for a transmitted index outside the labels).
// DT = 2 and 4: the even shapes of two and four coordinates (QAM; its 4D products, and those of
// planes; 2D constellations of up to 16 points) take the loop above, everything else the general
// one.
template <int MODE, bool GMI, int DT, int MB>
__device__ __forceinline__ void all_symbols(const ProdArgs& G, const int* __restrict__ flags, SymbolArgs A) {
  ConstInt* fl = reinterpret_cast<ConstInt*>(reinterpret_cast<uint64_t>(flags));
  A.start = fl[0] != 0 ? __builtin_nanf("") : 0.0f;
  // The FP32 form: while an FP32 squared distance that overflows means a score of 2^28 and more, and
  // one that underflows a score below 2^-28; and, from 128 points on, not for constellations the
  // general path would leave to its FP64 kernel (flags[2]).
  A.fp32_ok = A.c >= 1e-30 && A.c <= 1e30 && (MB != 0 || fl[2] == 0);
  ConstInt* head = reinterpret_cast<ConstInt*>(reinterpret_cast<uint64_t>(G.prod));
  ProdTables T;
  T.td = reinterpret_cast<ConstDouble*>(reinterpret_cast<uint64_t>(G.ptab));
  T.tf = reinterpret_cast<ConstFloat*>(reinterpret_cast<uint64_t>(G.ptabf));
  const int nf = head[0], nconst = head[1];
  if constexpr (DT != 0) {
    const int mf = head[kProdHead];
    bool even = nconst == 0 && DT % nf == 0;
    for (int f = 0; f < nf; ++f)
      even = even && head[kProdHead + kProdFactor * f] == mf && head[kProdHead + kProdFactor * f + 1] * nf == DT;
    if constexpr (DT == 2) {
      if (even && nf == 2 && fixed_shape<MODE, 2, 1, GMI, MB>(mf, T, head, A)) return;
      if (even && nf == 1 && fixed_shape<MODE, 1, 2, GMI, MB>(mf, T, head, A)) return;
    } else {
      if (even && nf == 4 && fixed_shape<MODE, 4, 1, GMI, MB>(mf, T, head, A)) return;
      if (even && nf == 2 && fixed_shape<MODE, 2, 2, GMI, MB>(mf, T, head, A)) return;
    }
  }
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kProdThreads;
  bool some = false;
  for (int64_t n = static_cast<int64_t>(blockIdx.x) * kProdThreads + threadIdx.x; n < A.N; n += stride) {
    const float* row = A.y + n * A.D;
    float* lrow = A.llr + n * A.m;
    float nonfinite = A.start, term = 0.0f;
    const uint32_t lab = sent_label<GMI>(A, n, &term);
    Reach reach;
    for (int i = 0; i < nconst; ++i) nonfinite = fmaf(row[head[2 + i]], 0.0f, nonfinite);
    for (int f = 0; f < nf; ++f) {
      T.fd = head + kProdHead + kProdFactor * f;
      switch (T.fd[0]) {
        case 1: term += factor_llr<MODE, 1, GMI>(T, row, A.m, A.c, A.cnat, lrow, lab, &nonfinite, reach); break;
        case 2: term += factor_llr<MODE, 2, GMI>(T, row, A.m, A.c, A.cnat, lrow, lab, &nonfinite, reach); break;
        case 3: term += factor_llr<MODE, 3, GMI>(T, row, A.m, A.c, A.cnat, lrow, lab, &nonfinite, reach); break;
        default: term += factor_llr<MODE, 4, GMI>(T, row, A.m, A.c, A.cnat, lrow, lab, &nonfinite, reach); break;
      }
    }
    if constexpr (MODE == PROD_FLOAT) term = mark_left(A, n, reach, nonfinite, term, &some);
    finish_symbol<GMI>(A, n, nonfinite, term);
  }
  if (some) *A.any_left = 1;
}

// ------------------------------------------------------------------ symbols left
// The symbols that reach too far for the forms with FP32 sums (the general path's FP64 kernel took
// them), one lane per symbol and LLR, all in FP64: distances, exponentials, sums and logarithm.  A block takes
// chunks of up to 1024 symbols and lists the marked ones in LDS; a wavefront's LLRs are of one column,
// so points are scalar loads.  Called by kernels that the general path launches after its first one and that
// would have nothing to do.
//
// Apart from the kernel that marks them because their 16 distances and 64 exponentials in FP64 took its
// registers (134 instead of 91) and made it 14 to 22 % slower where no symbol is left; and one lane per LLR
// because a call of a few thousand symbols waits for the longest chain.
constexpr int kRestMasks = 16;                 // 64-symbol masks of the largest chunk
struct RestList {
  unsigned short item[kRestMasks * 64];
  int count;
};

// Wavefront 0 lists the marked symbols of the masks m0 .. m0 + masks - 1: one mask per lane, places by
// a prefix sum.  The block meets at a barrier afterwards.
__device__ __forceinline__ void list_left(const uint64_t* __restrict__ left, int64_t m0, int64_t nmask, int masks,
                                          RestList& list) {
  if (threadIdx.x >= 64) return;
  uint64_t mk = (static_cast<int>(threadIdx.x) < masks && m0 + threadIdx.x < nmask) ? left[m0 + threadIdx.x] : 0;
  const int own = __popcll(mk);
  int at = own;
#pragma unroll
  for (int o = 1; o < kRestMasks; o <<= 1) {
    const int up = __shfl_up(at, o, 64);
    if (static_cast<int>(threadIdx.x) >= o) at += up;
  }
  if (threadIdx.x == kRestMasks - 1) list.count = at;
  at -= own;
  for (; mk; mk &= mk - 1)
    list.item[at++] = static_cast<unsigned short>(64 * threadIdx.x + __ffsll(static_cast<unsigned long long>(mk)) - 1);
}
// Masks a block takes at a time, so that `blocks` blocks share nmask of them.
inline int rest_masks(int64_t nmask, int64_t blocks) {
  const int64_t k = (nmask + blocks - 1) / blocks;
  return static_cast<int>(k < 1 ? 1 : (k > kRestMasks ? kRestMasks : k));
}

// Smallest distance of the subset (bit b = v) and the sum of 2^-(c (d2 - min)).
template <int MF>
__device__ __forceinline__ void subset_sum(const ProdTables& T, const float* __restrict__ row, int b, int v, double c,
                                           double* mn, double* sum) {
  constexpr int H = 1 << (MF - 1);
  double d2[H];
#pragma unroll
  for (int j = 0; j < H; ++j) d2[j] = 0.0;
  const int df = T.fd[1], low = (1 << b) - 1;
#pragma unroll 1
  for (int i = 0; i < df; ++i) {
    const int co = T.fd[8 + i];
    const double y = static_cast<double>(row[co]);
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const double diff = y - T.td[16 * co + (((j & ~low) << 1) | (v << b) | (j & low))];
      d2[j] = fma(diff, diff, d2[j]);
    }
  }
  double a = d2[0], s = 0.0;
#pragma unroll
  for (int j = 1; j < H; ++j) a = fmin(a, d2[j]);
#pragma unroll
  for (int j = 0; j < H; ++j) s += fp64::exp2_neg(c * (d2[j] - a));
  *mn = a;
  *sum = s;
}
template <int MF>
__device__ __forceinline__ float column_llr(const ProdTables& T, const float* __restrict__ row, int b, double c, double cnat) {
  double mn[2], sum[2];
  subset_sum<MF>(T, row, b, 0, c, &mn[0], &sum[0]);
  subset_sum<MF>(T, row, b, 1, c, &mn[1], &sum[1]);
  return static_cast<float>(fma(cnat, mn[1] - mn[0], fp64::log_ratio<15, false>(sum[0], sum[1])));
}

// Called by every thread of blocks of kProdThreads.
__device__ __forceinline__ void rest_columns(const ProdArgs& G, const SymbolArgs& A, int masks, RestList& list) {
  if (!*A.any_left) return;                  // (looking the masks through takes 4 us at 2e6 symbols)
  ConstInt* head = reinterpret_cast<ConstInt*>(reinterpret_cast<uint64_t>(G.prod));
  ProdTables T;
  T.td = reinterpret_cast<ConstDouble*>(reinterpret_cast<uint64_t>(G.ptab));
  T.tf = nullptr;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t nmask = (A.N + 63) / 64;
  for (int64_t m0 = static_cast<int64_t>(blockIdx.x) * masks; m0 < nmask;
       m0 += static_cast<int64_t>(gridDim.x) * masks) {
    list_left(A.left, m0, nmask, masks, list);
    __syncthreads();
    const int count = __builtin_amdgcn_readfirstlane(list.count);
    const int runs = (count + 63) / 64;
    for (int job = wave; job < runs * A.m; job += kProdThreads / 64) {
      int b = job / runs;                        // the b-th bit of the factors in turn
      T.fd = head + kProdHead;
      while (b >= T.fd[0]) {
        b -= T.fd[0];
        T.fd += kProdFactor;
      }
      const int i = (job % runs) * 64 + lane;
      if (i >= count) continue;
      const int64_t n = 64 * m0 + list.item[i];
      const float* row = A.y + n * A.D;
      float L;
      switch (T.fd[0]) {
        case 1: L = column_llr<1>(T, row, b, A.c, A.cnat); break;
        case 2: L = column_llr<2>(T, row, b, A.c, A.cnat); break;
        case 3: L = column_llr<3>(T, row, b, A.c, A.cnat); break;
        default: L = column_llr<4>(T, row, b, A.c, A.cnat); break;
      }
      A.llr[n * A.m + T.fd[3 + b]] = L;
    }
    __syncthreads();
  }
}

inline ProdArgs prod_args(const Prepared& P) { return {P.prod, P.ptab, P.ptabf}; }
inline SymbolArgs symbol_args(const Prepared& P, int M, int D, const float* d_y, int64_t N, double sigma2,
                              float* d_llr) {
  SymbolArgs A;
  A.y = d_y;
  A.llr = d_llr;
  A.gmi_tx = P.gmi_tx;
  A.gmi_labels = P.gmi_labels;
  A.gmi_terms = P.gmi_terms;
  A.left = reinterpret_cast<uint64_t*>(P.fb_list);
  A.any_left = P.flags + 6;
  A.N = N;
  A.m = ilog2_pow2(M);
  A.D = D;
  A.cnat = 1.0 / (2.0 * sigma2);
  A.c = A.cnat * 1.4426950408889634;
  A.start = 0.0f;
  A.fp32_ok = true;
  return A;
}

}  // namespace prodk
}  // namespace md
