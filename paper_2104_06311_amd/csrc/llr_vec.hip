// Exact (and max-log) LLRs of small constellations (M = 32 or 64, D <= 8) with one thread
// per symbol.
//
// With 64 points per symbol the matrix-core kernel does two tiles per 32-symbol block, so
// its per-symbol prologue and epilogue (operand staging, subset combine) cost more than its
// tile work.  Here each thread takes a whole symbol: the score of point j (label order),
//   t_j = bias - c ||y - x_j||^2 = sum_d y_d (2c x_jd) + (-c ||x_j||^2) + (bias - c ||y||^2),
// from the two per-point terms prep writes (read at uniform addresses through the constant
// address space, so by scalar loads that the vector instructions take as operands), D + 1
// FP32 operations per point; e_j = 2^t_j with the fast kernel's fixed bias; the label-0
// and label-1 subset sums of every bit by one pass per bit over block sums; LLRs as
// ln 2 (log2 S0 - log2 S1).  A symbol whose sums leave the FP32 range is marked in a bitmap,
// and a second kernel finishes the marked ones in one pass.  Rounding: t_j carries about 2^-23 of c (|x_j| + |y|)^2,
// the same order as the split-FP16 contraction's dropped low-by-low product.
#include <type_traits>

#include "common.hpp"
#include "fp64_form.hpp"
#include "llr_fast.hpp"
#include "llr_kernels.hpp"
#include "llr_prod.hpp"

namespace md {
namespace {

constexpr int kVecThreads = prodk::kProdThreads;

// GMI: also the loss term T_n = sum_k log2((S0_k + S1_k) / S_sent,k) of every finished
// symbol (NaN for the symbols left to the later passes), as the fast kernel's fused
// epilogue writes it.
// MAXLOG: max-log LLRs instead, ln 2 (max_{bit 0} t_j - max_{bit 1} t_j), from the same
// per-point terms with maxima in place of the exponentials and sums (scores never leave
// the FP32 range, so no symbol is left).
template <int MB, int D, bool GMI, bool MAXLOG = false>
__global__ void __launch_bounds__(kVecThreads) llr_vec_kernel(const float* __restrict__ vx_g,
                                                              const float* __restrict__ y, int64_t N, float c,
                                                              float* __restrict__ llr, const int* __restrict__ flags,
                                                              uint64_t* __restrict__ left,
                                                              const uint32_t* __restrict__ gmi_tx,
                                                              const uint32_t* __restrict__ gmi_labels,
                                                              float* __restrict__ gmi_terms, prodk::ProdArgs G,
                                                              prodk::SymbolArgs A) {
  constexpr int M = 1 << MB;
  constexpr int m = MB;
  // a product constellation: by its factors (a launch less than a kernel of its own)
  if (flags[5]) {
    constexpr int mode = MAXLOG ? prodk::PROD_MAXLOG : prodk::PROD_FLOAT;
    return prodk::all_symbols<mode, GMI, (MB == 6 && (D == 2 || D == 4)) ? D : 0, MB>(G, flags, A);
  }
  typedef const __attribute__((address_space(4))) float ConstFloat;
  const bool invalid = flags[0] != 0;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kVecThreads;
  for (int64_t n = static_cast<int64_t>(blockIdx.x) * kVecThreads + threadIdx.x; n < N; n += stride) {
    // the table's address passes through an empty asm statement on every symbol, so that
    // the compiler loads the M (D + 1) terms inside the loop as they are used, instead of
    // hoisting them all into scalar registers that spill
    uint64_t vaddr = reinterpret_cast<uint64_t>(vx_g);
    asm volatile("" : "+s"(vaddr));
    ConstFloat* vx = reinterpret_cast<ConstFloat*>(vaddr);
    float yv[D];
    float ysq = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      yv[d] = y[n * D + d];
      ysq = fmaf(yv[d], yv[d], ysq);
    }
    const bool nan_y = ysq != ysq;
    // max-log takes differences of scores only: the terms common to all points (the bias
    // and -c ||y||^2) drop out, and leaving them out keeps the scores' magnitude small
    const float r = MAXLOG ? 0.0f : fmaf(-c, ysq, fastk::kExpBias);
    float v[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
      float t = vx[j * (D + 1) + D] + r;
#pragma unroll
      for (int d = 0; d < D; ++d) t = fmaf(yv[d], vx[j * (D + 1) + d], t);
      v[j] = MAXLOG ? t : __builtin_amdgcn_exp2f(t);
    }
    // level b: v[k] is the sum over the 2^b consecutive labels of block k, so bit b of a
    // label is the parity of its block index
    float S0[MB], S1[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const int cnt = M >> b;
      float a0 = v[0], a1 = v[1];
#pragma unroll
      for (int k = 2; k < cnt; k += 2) {
        a0 = MAXLOG ? fmaxf(a0, v[k]) : a0 + v[k];
        a1 = MAXLOG ? fmaxf(a1, v[k + 1]) : a1 + v[k + 1];
      }
      S0[b] = a0;
      S1[b] = a1;
#pragma unroll
      for (int k = 0; k < cnt / 2; ++k) v[k] = MAXLOG ? fmaxf(v[2 * k], v[2 * k + 1]) : v[2 * k] + v[2 * k + 1];
    }
    if constexpr (MAXLOG) {
#pragma unroll
      for (int k = 0; k < m; ++k) {
        const int b = m - 1 - k;
        llr[n * m + k] = invalid ? __builtin_nanf("") : fastk::kLn2 * (S0[b] - S1[b]);
      }
      continue;
    }
    // the wavefront's symbols left to the kernel below, one bit each (its 64 symbols are one
    // aligned run); an append to a common list, one atomic per wavefront that has any, took 190 us
    // at 1e6 symbols where a tenth of them is out of range
    // (a NaN sum of a received value that is none: an operand outside the FP32 range)
    const float all = S0[0] + S1[0];
    const bool out = !invalid && (!fastk::sums_in_range<MB>(S0, S1) || (all != all && !nan_y));
    const uint64_t mask = __ballot(out);
    if ((n & 63) == 0) left[n >> 6] = mask;
    if (invalid) {
#pragma unroll
      for (int k = 0; k < m; ++k) llr[n * m + k] = __builtin_nanf("");
      if constexpr (GMI) gmi_terms[n] = __builtin_nanf("");
    } else if (out) {
      if constexpr (GMI) gmi_terms[n] = __builtin_nanf("");   // taken from its final LLRs later
    } else {
      float l2s0[MB], l2s1[MB];
#pragma unroll
      for (int k = 0; k < m; ++k) {
        const int b = m - 1 - k;
        l2s0[b] = fastk::log2_normal(S0[b]);
        l2s1[b] = fastk::log2_normal(S1[b]);
        llr[n * m + k] = fastk::kLn2 * (l2s0[b] - l2s1[b]);
      }
      if constexpr (GMI) {
        const uint32_t u = gmi_tx[n];
        const uint32_t lab = u < static_cast<uint32_t>(M) ? gmi_labels[u] : 0xFFFFFFFFu;
        // S0 + S1 is the sum over all points for every bit: one logarithm serves all
        const float l2tot = fastk::log2_normal(S0[0] + S1[0]);
        float T = lab != 0xFFFFFFFFu ? 0.0f : __builtin_nanf("");
#pragma unroll
        for (int b = 0; b < MB; ++b) T += l2tot - (((lab >> b) & 1u) ? l2s1[b] : l2s0[b]);
        gmi_terms[n] = T;
      }
    }
  }
}

// The symbols the kernel above left (exact LLRs out of the FP32 range), four lanes each: lane q takes
// the M / 4 labels from q M / 4 on, so the two high label bits are the lane and the rest its position.
// A block takes chunks of up to 1024 symbols and lists the marked ones in LDS, where the points are
// too.  (Products: prodk::rest_columns.)  Distances, exponentials, sums and logarithms are FP64, as in the
// kernel for such symbols of larger constellations; every point's score relative to the best one is
// 2^k e (fp64_form.hpp), so a subset's sum is taken relative to its own largest term and no range is lost:
// M exponentials a symbol.  Scores saturate 2^30 below the best: a subset that far has its smallest
// distance alone (its sum moves the LLR by ln M at most, of 7e8).
// One launch in place of the matrix-core path's three later passes (two and three exponent windows,
// FP64).  What bounds it is the FP64 arithmetic of the listed symbols, and a call of a few thousand
// symbols waits for one symbol's chain: one lane a symbol (the distances formed twice to save
// registers) took 82 us where all of 2000 symbols are out of range and 260 us where all of 1e6 are, four
// 18.8 and 185, with FP32 exponentials.  FP64 ones are no slower at M = 64 since the points are read from
// LDS for every symbol (kept in registers they left one wavefront a SIMD): all of 2e6 symbols of 64 4D
// points 352 -> 310 us a call, 64 8D 418 -> 377; 32 2D points, whose registers sufficed, 141 -> 174.
// Whole calls at M = 64, 4D, by the three later passes -> now: 2000 symbols all out of range 66 -> 18 us, 2e6
// symbols 1.7 % out of range 264 -> 78, all 33100 -> 310.
template <int XOR>
__device__ __forceinline__ int quad_xor(int v) {
  return __builtin_amdgcn_update_dpp(0, v, XOR == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true);
}
template <int XOR>
__device__ __forceinline__ double quad_xor(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = static_cast<uint32_t>(quad_xor<XOR>(static_cast<int>(static_cast<uint32_t>(u))));
  const uint32_t hi = static_cast<uint32_t>(quad_xor<XOR>(static_cast<int>(static_cast<uint32_t>(u >> 32))));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ double quad_min(double v) {
  v = fmin(v, quad_xor<1>(v));
  return fmin(v, quad_xor<2>(v));
}
__device__ __forceinline__ int quad_max(int v) {
  v = max(v, quad_xor<1>(v));
  return max(v, quad_xor<2>(v));
}
__device__ __forceinline__ double quad_sum(double v) {
  v += quad_xor<1>(v);
  return v + quad_xor<2>(v);
}

// x: lane q's points.  All four lanes of a quad are here together.
template <int MB, int D>
__device__ __forceinline__ void rest_symbol(const float* x, int q, const float* __restrict__ y, int64_t n, double c,
                                            double cnat, float* __restrict__ llr) {
  constexpr int P = (1 << MB) / 4;
  double yv[D];
#pragma unroll
  for (int d = 0; d < D; ++d) yv[d] = static_cast<double>(y[n * D + d]);
  auto dist = [&](int i) {
    double d2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const double df = yv[d] - static_cast<double>(x[i * D + d]);
      d2 = fma(df, df, d2);
    }
    return d2;
  };
  double e[P];
  int k[P];
  {
    double d2[P];
    double dmin = INFINITY;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      d2[i] = dist(i);
      dmin = fmin(dmin, d2[i]);
    }
    dmin = quad_min(dmin);
#pragma unroll
    for (int i = 0; i < P; ++i) fp64::exp2_neg(c * (d2[i] - dmin), &k[i], &e[i]);
  }
  // lane q finishes the bits b = q mod 4
  constexpr int R = (MB + 3) / 4;
  double own0[R], own1[R];
  int shift[R];
  unsigned far = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    own0[r] = own1[r] = 1.0;
    shift[r] = 0;
  }
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const bool high = b >= MB - 2;
    const bool mine = high && ((q >> (b - (MB - 2))) & 1);    // the bit of all of this lane's labels
    int top[2] = {INT32_MIN, INT32_MIN};
    double sum[2] = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < P; ++i) top[high ? 0 : (i >> b) & 1] = max(top[high ? 0 : (i >> b) & 1], k[i]);
    if (high) {
      top[1] = mine ? top[0] : INT32_MIN;
      top[0] = mine ? INT32_MIN : top[0];
    }
    top[0] = quad_max(top[0]);
    top[1] = quad_max(top[1]);
    const int ref = mine ? top[1] : top[0];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int s = high ? 0 : (i >> b) & 1;
      sum[s] += ldexp(e[i], k[i] - (high ? ref : top[s]));
    }
    if (high) {
      sum[1] = mine ? sum[0] : 0.0;
      sum[0] = mine ? 0.0 : sum[0];
    }
    sum[0] = quad_sum(sum[0]);
    sum[1] = quad_sum(sum[1]);
    const bool keep = q == (b & 3);
    own0[b >> 2] = keep ? sum[0] : own0[b >> 2];
    own1[b >> 2] = keep ? sum[1] : own1[b >> 2];
    shift[b >> 2] = keep ? top[0] - top[1] : shift[b >> 2];
    far |= fp64::saturated(min(top[0], top[1])) ? 1u << b : 0u;
    __builtin_amdgcn_sched_barrier(0);         // one bit's temporaries at a time (registers)
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int b = 4 * r + q;
    const double L = fma(static_cast<double>(shift[r]), fp64::kLn2, fp64::log_ratio<15, false>(own0[r], own1[r]));
    if (b < MB) llr[n * MB + (MB - 1 - b)] = static_cast<float>(L);
  }
#pragma unroll 1
  for (; far; far &= far - 1) {
    const int b = __ffs(far) - 1;
    double m[2] = {INFINITY, INFINITY};
#pragma unroll 1
    for (int i = 0; i < P; ++i) {
      const bool one = ((q * P + i) >> b) & 1;
      const double d2 = dist(i);
      m[0] = one ? m[0] : fmin(m[0], d2);
      m[1] = one ? fmin(m[1], d2) : m[1];
    }
    m[0] = quad_min(m[0]);
    m[1] = quad_min(m[1]);
    // infinite points: no LLR
    const double L = (m[0] < INFINITY && m[1] < INFINITY) ? cnat * (m[1] - m[0]) : __builtin_nan("");
    if (q == (b & 3)) llr[n * MB + (MB - 1 - b)] = static_cast<float>(L);
  }
}

template <int MB, int D>
__global__ void __launch_bounds__(kVecThreads) llr_vec_rest_kernel(const float* __restrict__ xl_g,
                                                                   const float* __restrict__ y, int64_t N, double cnat,
                                                                   float* __restrict__ llr, int* __restrict__ flags,
                                                                   const uint64_t* __restrict__ left, int masks,
                                                                   prodk::ProdArgs G, prodk::SymbolArgs A) {
  constexpr int kRun = (1 << MB) / 4 * D, kStep = kRun + 4;   // the four runs of points in other LDS banks
  __shared__ float pts[4 * kStep];
  __shared__ prodk::RestList list;
  if (flags[5]) return prodk::rest_columns(G, A, masks, list);
  for (int i = threadIdx.x; i < 4 * kRun; i += kVecThreads) pts[i / kRun * kStep + i % kRun] = xl_g[i];
  const int64_t nmask = (N + 63) / 64;
  const double c = cnat * 1.4426950408889634;
  const int q = threadIdx.x & 3;
  for (int64_t m0 = static_cast<int64_t>(blockIdx.x) * masks; m0 < nmask;
       m0 += static_cast<int64_t>(gridDim.x) * masks) {
    prodk::list_left(left, m0, nmask, masks, list);
    __syncthreads();
    const int count = list.count;
    if (threadIdx.x == 0 && count) atomicAdd(&flags[1], count);
    for (int i = threadIdx.x / 4; i < count; i += kVecThreads / 4) {
      int at = q * kStep;                        // opaque: the points are read from LDS for every symbol (kept in
      asm volatile("" : "+v"(at));               // registers they leave one wavefront a SIMD)
      rest_symbol<MB, D>(pts + at, q, y, 64 * m0 + list.item[i], c, cnat, llr);
    }
    __syncthreads();
  }
}

template <int MB, int D, bool GMI, bool MAXLOG = false>
int launch_vec_g(const Prepared& P, const float* d_y, int64_t N, double sigma2, float* d_llr, hipStream_t stream) {
  auto kern = llr_vec_kernel<MB, D, GMI, MAXLOG>;
  int ncu = 0, occ = 0;
  MD_TRY(device_cus(&ncu));
  MD_TRY(blocks_per_cu(reinterpret_cast<const void*>(kern), kVecThreads, 0, &occ));
  int64_t grid = (N + kVecThreads - 1) / kVecThreads;
  const int64_t full = static_cast<int64_t>(ncu) * occ * 4;
  if (grid > full) grid = full;
  const float c = P.c_over_alpha * P.alpha;
  const int slot = timing_begin(stream);
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(kVecThreads), 0, stream, P.vx, d_y, N, c, d_llr,
                     P.flags, reinterpret_cast<uint64_t*>(P.fb_list), P.gmi_tx, P.gmi_labels, P.gmi_terms,
                     prodk::prod_args(P),
                     prodk::symbol_args(P, 1 << MB, D, d_y, N, sigma2, d_llr));
  timing_end(stream, slot);
  MD_LAUNCH_CHECK("llr_vec_kernel launch");
  if constexpr (MAXLOG) return MD_OK;         // scores never leave the range
  // four blocks per compute unit, then chunks of more than one mask
  const int64_t nmask = (N + 63) / 64;
  const int masks = prodk::rest_masks(nmask, 4 * ncu);
  int64_t rest = (nmask + masks - 1) / masks;
  if (rest > 4 * ncu) rest = 4 * ncu;
  hipLaunchKernelGGL((llr_vec_rest_kernel<MB, D>), dim3(static_cast<unsigned>(rest)), dim3(kVecThreads), 0, stream,
                     P.xl, d_y, N, 1.0 / (2.0 * sigma2), d_llr, P.flags, reinterpret_cast<const uint64_t*>(P.fb_list),
                     masks, prodk::prod_args(P), prodk::symbol_args(P, 1 << MB, D, d_y, N, sigma2, d_llr));
  MD_LAUNCH_CHECK("llr_vec_rest_kernel launch");
  return MD_OK;
}

template <int MB, int D>
int launch_vec_t(const Prepared& P, const float* d_y, int64_t N, double sigma2, bool maxlog, float* d_llr, hipStream_t stream) {
  if (maxlog) return launch_vec_g<MB, D, false, true>(P, d_y, N, sigma2, d_llr, stream);
  return P.gmi_terms ? launch_vec_g<MB, D, true>(P, d_y, N, sigma2, d_llr, stream)
                     : launch_vec_g<MB, D, false>(P, d_y, N, sigma2, d_llr, stream);
}

template <int MB>
int launch_vec_m(const Prepared& P, int D, const float* d_y, int64_t N, double sigma2, bool maxlog, float* d_llr,
                 hipStream_t stream) {
  switch (D) {
    case 1: return launch_vec_t<MB, 1>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    case 2: return launch_vec_t<MB, 2>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    case 3: return launch_vec_t<MB, 3>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    case 4: return launch_vec_t<MB, 4>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    case 5: return launch_vec_t<MB, 5>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    case 6: return launch_vec_t<MB, 6>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    case 7: return launch_vec_t<MB, 7>(P, d_y, N, sigma2, maxlog, d_llr, stream);
    default: return launch_vec_t<MB, 8>(P, d_y, N, sigma2, maxlog, d_llr, stream);
  }
}

}  // namespace

bool vec_exact_supported(int M, int D) { return (M == 32 || M == 64) && D >= 1 && D <= 8; }

int launch_vec_exact(const Prepared& P, int M, int D, const float* d_y, int64_t N, double sigma2, float* d_llr,
                     hipStream_t stream, bool maxlog) {
  if (!vec_exact_supported(M, D) || !P.vx) return fail(MD_EUNSUPPORTED, "vector demapper: M 32 or 64 and D <= 8");
  return M == 32 ? launch_vec_m<5>(P, D, d_y, N, sigma2, maxlog, d_llr, stream)
                 : launch_vec_m<6>(P, D, d_y, N, sigma2, maxlog, d_llr, stream);
}

}  // namespace md
