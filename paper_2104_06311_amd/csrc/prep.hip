// Per-call constellation preparation: label-order permutation, label validation and
// the MFMA A-operand fragments of the score contraction.
//
// Score contraction.  For a symbol y and a point x the demappers need
//   t = -c ||y - x||^2 + bias,  c = log2(e) / (2 sigma2)   (exponent in base 2),
// written as u.w + p a + a r with
//   u = a x,  w = (2c/a) y,  p = -(c/a) ||x||^2,  r = (bias - c ||y||^2)/a
// and a power of two a that balances the magnitudes of both operands.  Every factor is
// split into an FP16 high part and an FP16 low part, and the MFMA's K dimension
// carries the partial products as separate slots (3D + 4 of them):
//   point (A) side:  [ u_hi (D), u_lo (D), u_hi (D), p_hi, p_lo, a, a, 0 ... ]
//   symbol (B) side: [ w_hi (D), w_hi (D), w_lo (D), a,    a,    r_hi, r_lo, 0 ... ]
// so that one FP32-accumulating v_mfma_f32_32x32x16_f16 per 16 slots forms
// u_hi w_hi + u_lo w_hi + u_hi w_lo (the dropped u_lo w_lo is ~2^-22 |u||w|).
//
// Fragment layout.  Points are grouped in tiles of 32 consecutive labels.  Inside a
// tile, MFMA row i (0..31) holds the point whose label offset is
//   p(i) = 16 * ((i / 4) % 2) + 4 * (i / 8) + i % 4,
// chosen so that in the 32x32 MFMA result lane l, register r holds label offset
// 16 * (l / 32) + r: every lane owns 16 consecutive labels of one symbol.
// frag[(tile * KS + ks) * 64 + lane] is the 8-half A operand of that lane: row lane % 32,
// slots 16 ks + 8 (lane / 32) .. +7.
//
// One-pass layouts (the reduced-precision variants of llr_exact): each factor is rounded
// once, to FP16 or to BF16, and the K dimension holds D + 4 slots
//   point (A) side:  [ u (D), p_hi, p_lo, a, a, 0 ... ]
//   symbol (B) side: [ w (D), a,    a,    r_hi, r_lo, 0 ... ]
// (the biases keep a hi/lo split in the same format), so one MFMA per tile serves
// D <= 12 at a score error of about 2^-10 (FP16) or 2^-8 (BF16) of sum_k |u_k w_k|.
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "llr_kernels.hpp"

namespace md {
namespace {

__global__ void prep_init_kernel(uint32_t* __restrict__ inv, int M, int* __restrict__ flags) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < M) inv[s] = 0xFFFFFFFFu;
  if (s < 8) flags[s] = 0;
}

__global__ void prep_scatter_kernel(const uint32_t* __restrict__ labels, int M, uint32_t* __restrict__ inv,
                                    int* __restrict__ flags) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= M) return;
  const uint32_t l = labels[j];
  if (l >= static_cast<uint32_t>(M)) {
    flags[0] = 1;
    return;
  }
  inv[l] = static_cast<uint32_t>(j);
}

__device__ __forceinline__ void split_half(float v, _Float16* hi, _Float16* lo) {
  const _Float16 h = static_cast<_Float16>(v);
  *hi = h;
  *lo = static_cast<_Float16>(v - static_cast<float>(h));
}

// The BF16 bits of v (round to nearest even), carried in an FP16 slot of the row.
__device__ __forceinline__ _Float16 bf16_bits(float v) {
  return __builtin_bit_cast(_Float16, static_cast<__bf16>(v));
}
__device__ __forceinline__ void split_bf16(float v, _Float16* hi, _Float16* lo) {
  const __bf16 h = static_cast<__bf16>(v);
  *hi = __builtin_bit_cast(_Float16, h);
  *lo = bf16_bits(v - static_cast<float>(h));
}

// The slots 8 g .. 8 g + 7 of a fragment row (g = 0 .. 2 KS - 1) for the point xr (D values), in
// the layout sc names: the MFMA A operand of one lane for one K step.  `nrm` is ||x||^2 in
// FP64.
__device__ __forceinline__ uint4 row_group(const float* __restrict__ xr, int D, int sc, int g, float alpha,
                                           float c_over_alpha, double nrm) {
#pragma clang fp contract(off)
  const int nb = sc == 0 ? 3 * D : D;        // first bias slot
  const float p = -c_over_alpha * static_cast<float>(nrm);
  _Float16 slot[8];
  float x[8];                                // all loads first: their latency is paid once
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = 8 * g + e;
    x[e] = xr[k >= nb ? 0 : (k < D ? k : (k < 2 * D ? k - D : k - 2 * D))];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = 8 * g + e;
    _Float16 v = static_cast<_Float16>(0.0f);
    if (k < nb) {
      const float u = alpha * x[e];
      if (sc == 0) {
        _Float16 hi, lo;
        split_half(u, &hi, &lo);
        v = (k >= D && k < 2 * D) ? lo : hi;
      } else {
        v = sc == 1 ? static_cast<_Float16>(u) : bf16_bits(u);
      }
    } else if (k < nb + 2) {
      _Float16 hi, lo;
      if (sc == 2) split_bf16(p, &hi, &lo);
      else split_half(p, &hi, &lo);
      v = k == nb ? hi : lo;
    } else if (k < nb + 4) {
      v = sc == 2 ? bf16_bits(alpha) : static_cast<_Float16>(alpha);
    }
    slot[e] = v;
  }
  uint4 out;
  __builtin_memcpy(&out, slot, 16);
  return out;
}

// Whether row group g holds a slot of the point's bias p (and so needs ||x||^2).
__device__ __forceinline__ bool group_has_bias(int D, int sc, int g) {
  const int nb = sc == 0 ? 3 * D : D;
  return 8 * g + 7 >= nb && 8 * g < nb + 2;
}

// f(d, x_d) for the D coordinates of a point, eight loads in flight at a time (one load per
// iteration pays the memory latency D times over).
template <class F>
__device__ __forceinline__ void for_coords(const float* __restrict__ xr, int D, F f) {
  for (int d0 = 0; d0 < D; d0 += 8) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = d0 + e < D ? xr[d0 + e] : 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (d0 + e < D) f(d0 + e, v[e]);
  }
}

// Place of row group g of label slot s in the fragments.
__device__ __forceinline__ int64_t frag_index(int s, int KS, int g) {
  const int p = s & 31;
  const int h = p >> 4, r = p & 15;
  const int i = 8 * (r >> 2) + 4 * h + (r & 3);
  return (static_cast<int64_t>(s >> 5) * KS + (g >> 1)) * 64 + i + 32 * (g & 1);
}

// Looks for the factors of a product constellation: label bits and coordinates that fall into
// groups such that each coordinate depends on its group's bits alone, x_l = (x_A(l_A), x_B(l_B),
// ...).  The likelihood sums of such a constellation are products over the groups, so the LLRs
// of a group's bits need its own 2^bits points only (square QAM: two PAMs; the 4D products of
// QAM or PSK: their axes or planes).  Dependencies are read off the neighbours (one label bit
// flipped) of a few base labels; the groups they give are then verified on every point, with
// exact comparison (prep_one_kernel), so a wrong guess can only say "no product".  Up to 16
// points a group; with M <= kSmallM the whole constellation is one group if nothing else.
struct FactorGroups {
  uint32_t dep[32], comp[16];    // label bits a coordinate depends on; label bits of a group
  int of[32], rank[32];          // group of a coordinate (-1: equal for every point), its place there
  int size[32];                  // coordinates of its group
  int n, wide, odd;              // groups; flags, each written before one barrier only
};

// floor(e / q) for e < 2^18 by magic_of(q) (q = 1: 0)
inline uint32_t magic_of(int q) { return q > 1 ? static_cast<uint32_t>((uint64_t(1) << 32) / q + 1) : 0u; }
__device__ __forceinline__ int div_by(int e, uint32_t magic) {
  return magic ? static_cast<int>(__umulhi(static_cast<uint32_t>(e), magic)) : e;
}

// Coordinate d of the point with label l, from the points in LDS (row stride Dp, index order).
struct Points {
  const float* xs;
  const uint32_t* inv;
  int M, D, Dp;
  __device__ __forceinline__ float operator()(uint32_t l, int d) const {
    const uint32_t j = min(inv[l], static_cast<uint32_t>(M) - 1);
    return xs[j * Dp + d];
  }
};

// The groups, and tab[16 d + p]: coordinate d of its group's point p.  Called by every thread
// of one block; false: no product.
__device__ bool guess_groups(const Points& x, FactorGroups& G, float* __restrict__ tab, uint32_t magic_d, uint32_t magic_m,
                             bool one_group) {
  constexpr int kBases = 8;
  const int M = x.M, D = x.D;
  const int tid = threadIdx.x, nt = blockDim.x;
  const uint32_t all = static_cast<uint32_t>(M) - 1;
  const int m = 31 - __clz(M);
  const bool small = M <= kSmallM;
  if (tid < 32) G.dep[tid] = 0;
  if (tid == 0) G.wide = 0;
  __syncthreads();
  if (!one_group) {
    for (int e = tid; e < kBases * m * D; e += nt) {
      const int q = div_by(e, magic_d), d = e - q * D;
      const int r = div_by(q, magic_m), b = q - r * m;
      const uint32_t base = ((0x9E3779B9u * static_cast<uint32_t>(r)) >> 7) & all;
      if (x(base, d) != x(base ^ (1u << b), d)) atomicOr(&G.dep[d], 1u << b);
    }
    __syncthreads();
    if (!small && tid < D && __popc(G.dep[tid]) > kProdMaxBits) G.wide = 1;
    __syncthreads();
    if (G.wide) return false;                    // the usual end for unstructured constellations
  }
  if (tid < 64) {
    // one wavefront, lane d holds coordinate d's label bits: merge what overlaps until nothing
    // does, then number the distinct masks
    uint32_t mk = one_group ? (tid < D ? all : 0u) : (tid < D ? G.dep[tid] : 0u);
    uint32_t seen = 0;
    bool more = true;
    while (more) {
      const uint32_t old = mk;
      for (int j = 0; j < D; ++j) {
        const uint32_t o = __builtin_amdgcn_readlane(mk, j);
        if (mk & o) mk |= o;
      }
      more = __any(mk != old);
    }
    uint32_t same = 0;                           // coordinates with this one's bits
    for (int j = 0; j < D; ++j) {
      const uint32_t o = __builtin_amdgcn_readlane(mk, j);
      seen |= o;
      same |= static_cast<uint32_t>(o == mk) << j;
    }
    const bool ok = seen == all && !__any(__popc(mk) > kProdMaxBits);
    if (!ok && small) {                          // one group of everything
      mk = tid < D ? all : 0u;
      same = (1u << D) - 1;
    }
    const bool head = mk != 0 && (same & (0u - same)) == 1u << (tid & 31);
    const uint64_t heads = __ballot(head);
    const int f = __popcll(heads & ((1ull << (__ffs(same) - 1)) - 1));
    if (tid < D) {
      G.of[tid] = mk ? f : -1;
      G.rank[tid] = __popc(same & ((1u << tid) - 1));
      G.size[tid] = __popc(same);
    }
    if (head) G.comp[f] = mk;
    if (tid == 0) {
      G.n = __popcll(heads);
      G.odd = !ok && !small;
    }
  }
  __syncthreads();
  if (G.odd) return false;
  for (int e = tid; e < 16 * D; e += nt) {
    const int d = e >> 4, p = e & 15;
    const int f = G.of[d];
    uint32_t l = 0, mk = f >= 0 ? G.comp[f] : 0u;
    for (int i = 0; mk; ++i, mk &= mk - 1)
      if ((p >> i) & 1) l |= mk & (0u - mk);
    tab[e] = x(l, d);
  }
  __syncthreads();
  return true;
}

// Writes the factors (layout in common.hpp).
__device__ void write_groups(const FactorGroups& G, const float* __restrict__ tab, int M, int D, int* __restrict__ prod,
                             double* __restrict__ ptab, float* __restrict__ ptabf) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int m = 31 - __clz(M);
  for (int e = tid; e < 16 * D; e += nt) {
    ptab[e] = static_cast<double>(tab[e]);
    ptabf[e] = tab[e];
  }
  if (tid < D) {
    const int f = G.of[tid], rank = G.rank[tid];
    if (f < 0) {
      prod[2 + rank] = tid;
    } else {
      int* fd = prod + kProdHead + kProdFactor * f;
      fd[8 + rank] = tid;
      if (rank == 0) {
        int i = 0;
        const uint32_t all = G.comp[f], low = all & (0u - all);
        for (uint32_t mk = all; mk; mk &= mk - 1) fd[3 + i++] = m - __ffs(mk);   // column m - 1 - bit
        fd[0] = i;
        fd[1] = G.size[tid];
        fd[7] = all == low * ((1u << i) - 1);
      }
    }
  }
  if (tid == 64) prod[0] = G.n;
  const uint64_t constant = __ballot(tid < D && G.of[tid & 31] < 0);
  if (tid == 0) prod[1] = __popcll(constant);
}

// Everything of one call's preparation in one launch (see one_launch).
//
// What bounds it is latency: labels -> inverse permutation -> points -> rows is a chain of
// dependent loads, and as three launches (clear, scatter, build) each link also paid a kernel
// boundary: 16.2 -> 10.6 us of kernel time at 8D M = 2048 (under the tracer).  Here every block
// rebuilds the whole inverse permutation in its LDS (M loads, coalesced; 32 KiB at most) and so
// needs no other block.  Block 0 writes the counters, the label and range flags, the factors of
// a product constellation and the per-point terms, from X staged in its own order through LDS
// (one thread reading one point from memory took 8 us of scattered accesses at M = 2048); the
// others write the fragments, one 16-byte row group per thread, and the label-ordered points,
// one float per thread.
// The line is how long block 0 takes to read the constellation alone: 8.4 us for 4096 4D points
// and 10.5 for 2048 8D ones, about what the three launches cost, but 21 us in chunks for 8192 8D
// or 4096 16D points, which made whole calls 7 to 10 us slower.  So up to 24576 floats, in one
// piece (M <= 8192, where every block's own inverse permutation still fits beside it), and every
// M <= 1024, which need the factors.
constexpr int kOneMax = 8192;
constexpr int kOneThreads = 1024;
constexpr int kOneStage = 24576;
inline bool one_launch(int M, int D) {
  return M <= kProdMaxM || (M <= kOneMax && M * (D | 1) <= kOneStage);
}

__global__ void __launch_bounds__(kOneThreads) prep_one_kernel(const float* __restrict__ X,
                                                               const uint32_t* __restrict__ labels, int M, int Mpad,
                                                               int D, uint32_t magic, uint32_t magic_m, int KS,
                                                               int sc, float alpha, float c_over_alpha,
                                                               float* __restrict__ xl, uint4* __restrict__ frag,
                                                               int* __restrict__ flags, float* __restrict__ vx,
                                                               int* __restrict__ prod, double* __restrict__ ptab,
                                                               float* __restrict__ ptabf) {
  extern __shared__ uint32_t inv[];          // M entries; block 0: 16 D floats of factor points, the stage
  __shared__ int sh_bad, sh_range, sh_differs;
  __shared__ FactorGroups G;
  const int tid = threadIdx.x, nt = blockDim.x;
  float* tab = reinterpret_cast<float*>(inv + M);
  float* xs = tab + 16 * D;
  const int Dp = D | 1;                      // odd row stride: no LDS bank conflicts
  bool range = false;
  // up to 16 loads in flight per thread: the points come from HBM, 2 us away
  auto stage_batches = [&](int total, auto batch) {
    constexpr int U = decltype(batch)::value;
#pragma unroll 1
    for (int e0 = tid; e0 < total; e0 += U * nt) {
      float v[U];
#pragma unroll
      for (int i = 0; i < U; ++i) v[i] = e0 + i * nt < total ? X[e0 + i * nt] : 0.0f;
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int e = e0 + i * nt;
        if (e >= total) break;
        const int pt = div_by(e, magic), d = e - pt * D;
        range |= !(fabsf(alpha * v[i]) <= 30000.0f);
        xs[pt * Dp + d] = v[i];
      }
    }
  };
  for (int s = tid; s < M; s += nt) inv[s] = 0xFFFFFFFFu;
  if (tid == 0) sh_bad = sh_range = sh_differs = 0;
  if (blockIdx.x == 0) {                     // its loads are under way with the labels'
    if (M * D <= nt) stage_batches(M * D, std::integral_constant<int, 1>{});
    else stage_batches(M * D, std::integral_constant<int, 16>{});
  }
  __syncthreads();
#pragma unroll 4
  for (int j = tid; j < M; j += nt) {
    const uint32_t l = labels[j];
    if (l < static_cast<uint32_t>(M)) inv[l] = static_cast<uint32_t>(j);
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    // M labels that fill every slot are a permutation; a slot left empty means a label
    // outside [0, M) or one used twice
    bool bad = false;
    for (int s = tid; s < M; s += nt) bad |= inv[s] == 0xFFFFFFFFu;
    const Points pts{xs, inv, M, D, Dp};
    // (without fragments nobody asks for the range)
    for (int pt = tid; frag && pt < M; pt += nt) {
      double nrm = 0.0;
      for (int d = 0; d < D; ++d) nrm += static_cast<double>(xs[pt * Dp + d]) * static_cast<double>(xs[pt * Dp + d]);
      range |= !(fabsf(-c_over_alpha * static_cast<float>(nrm)) <= 30000.0f);
    }
    // factors: a guess, verified on every point (coordinate d is that of its group's point with
    // the same bits); a small constellation whose guess fails is one group
    bool product = false;
#pragma unroll 1
    for (int attempt = 0; prod && !product && attempt < 2; ++attempt) {
      if (!guess_groups(pts, G, tab, magic, magic_m, attempt == 1)) break;
      bool differs = false;
      // place of the bits mk of label l among themselves
      auto compact = [](uint32_t l, uint32_t mk) {
        uint32_t p = 0;
        for (int i = 0; mk; ++i, mk &= mk - 1) p |= ((l >> (__ffs(mk) - 1)) & 1u) << i;
        return p;
      };
      auto check = [&](int l, int d, uint32_t p) {
        const float v = pts(l, d);
        differs |= !(fabsf(v) < INFINITY) || v != tab[16 * d + p];
      };
      if (attempt == 0 && M < nt) {
        // a thread per point and coordinate (coordinate by coordinate, as below, 30 of them took 10 us)
#pragma unroll 1
        for (int e = tid; e < M * D; e += nt) {
          const int l = div_by(e, magic), d = e - l * D;
          const int f = G.of[d];
          check(l, d, compact(l, f >= 0 ? G.comp[f] : 0u));
        }
      } else {
#pragma unroll 1
        for (int d = 0; attempt == 0 && d < D; ++d) {
          const int f = __builtin_amdgcn_readfirstlane(G.of[d]);
          const uint32_t mk = f >= 0 ? __builtin_amdgcn_readfirstlane(G.comp[f]) : 0u;
          const uint32_t low = mk & (0u - mk);
          const int shift = mk ? __ffs(mk) - 1 : 0;
          const bool run = (mk & (mk + low)) == 0;       // consecutive bits: a shift and a mask
#pragma unroll 4
          for (int l = tid; l < M; l += nt) check(l, d, run ? (static_cast<uint32_t>(l) & mk) >> shift : compact(l, mk));
        }
      }
      if (differs) sh_differs = 1;
      __syncthreads();
      product = attempt == 1 || !sh_differs;
      if (M > kSmallM) break;
    }
    if (vx) {
      // the vector demapper's terms (M <= 64, resident): 2c x (D floats) and -c ||x||^2, FP32 as
      // it computes; NaN where that overflows, so that no sum misses the point unnoticed
      const float c = c_over_alpha * alpha;
      for (int s = tid; s < M; s += nt) {
        float n32 = 0.0f;
        for (int d = 0; d < D; ++d) {
          const float v = pts(s, d);
          vx[s * (D + 1) + d] = 2.0f * c * v;
          n32 = fmaf(v, v, n32);
        }
        vx[s * (D + 1) + D] = c * n32 < INFINITY ? -c * n32 : __builtin_nanf("");
      }
    }
    if (bad) sh_bad = 1;
    if (range) sh_range = 1;
    __syncthreads();
    // broken labels give NaN everywhere: M <= kSmallM by the product kernel, others by the
    // general one
    const bool take = product && (!sh_bad || M <= kSmallM);
    if (take) write_groups(G, tab, M, D, prod, ptab, ptabf);
    if (tid < 8) flags[tid] = tid == 0 ? sh_bad : (tid == 2 ? sh_range : (tid == 5 && take ? 1 : 0));
    return;
  }
  const int first = (blockIdx.x - 1) * nt + tid, step = (gridDim.x - 1) * nt;
  for (int e = first; e < M * D; e += step) {
    const int s = div_by(e, magic);
    const uint32_t j = inv[s];
    xl[e] = j < static_cast<uint32_t>(M) ? X[j * D + (e - s * D)] : 0.0f;
  }
  if (!frag) return;
  const int groups = 2 * KS;
  for (int t = first; t < Mpad * groups; t += step) {
    const int s = t / groups, g = t - s * groups;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);    // padded rows (M < 32) stay zero
    const uint32_t j = s < M ? inv[s] : 0xFFFFFFFFu;
    if (j < static_cast<uint32_t>(M)) {
      const float* xr = X + static_cast<int64_t>(j) * D;
      double nrm = 0.0;
      if (group_has_bias(D, sc, g))
        for_coords(xr, D, [&](int, float x) { nrm += static_cast<double>(x) * static_cast<double>(x); });
      v = row_group(xr, D, sc, g, alpha, c_over_alpha, nrm);
    }
    frag[frag_index(s, KS, g)] = v;
  }
}

// One thread per label slot (large constellations: no padding, no per-point terms).
__global__ void prep_build_kernel(const float* __restrict__ X, const uint32_t* __restrict__ labels,
                                  const uint32_t* __restrict__ inv, int M, int D, int KS, int sc, float alpha,
                                  float c_over_alpha, float* __restrict__ xl, uint4* __restrict__ frag,
                                  int* __restrict__ flags) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= M) return;
  const uint32_t j = inv[s];
  const bool ok = j < static_cast<uint32_t>(M) && labels[j] == static_cast<uint32_t>(s);
  if (!ok) flags[0] = 1;
  const float* xr = X + static_cast<int64_t>(ok ? j : 0) * D;
  double nrm = 0.0;
  bool range = false;
  for (int d = 0; d < D; ++d) {
    const float v = xr[d];
    xl[static_cast<int64_t>(s) * D + d] = v;
    nrm += static_cast<double>(v) * static_cast<double>(v);
    range |= !(fabsf(alpha * v) <= 30000.0f);
  }
  range |= !(fabsf(-c_over_alpha * static_cast<float>(nrm)) <= 30000.0f);
  if (range) flags[2] = 1;          // outside the FP16 split range (or NaN)
  for (int g = 0; g < 2 * KS; ++g) frag[frag_index(s, KS, g)] = row_group(xr, D, sc, g, alpha, c_over_alpha, nrm);
}

}  // namespace

int frag_ksteps(int D) { return (3 * D + 4 + 15) / 16; }
int frag_ksteps_single(int D) { return (D + 4 + 15) / 16; }

size_t prep_bytes(int M, int D, int64_t N) {
  const int Mpad = ((M + 31) / 32) * 32;
  const int KS = frag_ksteps(D);
  size_t b = 0;
  b += carve_size(sizeof(float) * static_cast<size_t>(M) * D);                 // xl
  b += carve_size(sizeof(uint4) * static_cast<size_t>(Mpad / 32) * KS * 64);      // frag
  b += carve_size(sizeof(uint32_t) * M);                                       // inv
  b += carve_size(sizeof(int) * 8);                                            // flags
  b += 2 * carve_size(sizeof(unsigned) * static_cast<size_t>(N > 0 ? N : 1)); // fallback lists
  if (vec_exact_supported(M, D)) b += carve_size(sizeof(float) * static_cast<size_t>(M) * (D + 1));   // vx
  if (M <= kProdMaxM)
    b += carve_size(sizeof(int) * kProdInts) + carve_size(sizeof(double) * 16 * D) + carve_size(sizeof(float) * 16 * D);
  return b;
}

int prepare(const float* d_X, const uint32_t* d_labels, int M, int D, int64_t N, float alpha,
            float c_over_alpha, char* ws, hipStream_t stream, Prepared* out, int* flags_given, int sc, bool product) {
  const int Mpad = ((M + 31) / 32) * 32;
  const int KS = sc == 0 ? frag_ksteps(D) : frag_ksteps_single(D);
  Carver cv{ws, 0};
  float* xl = cv.take<float>(static_cast<size_t>(M) * D);
  uint4* frag = cv.take<uint4>(static_cast<size_t>(Mpad / 32) * KS * 64);
  uint32_t* inv = cv.take<uint32_t>(M);
  int* flags_carved = cv.take<int>(8);
  int* flags = flags_given ? flags_given : flags_carved;
  unsigned* fb = cv.take<unsigned>(static_cast<size_t>(N > 0 ? N : 1));
  unsigned* fb2 = cv.take<unsigned>(static_cast<size_t>(N > 0 ? N : 1));
  float* vx = (sc == 0 && vec_exact_supported(M, D)) ? cv.take<float>(static_cast<size_t>(M) * (D + 1)) : nullptr;
  int* prod = nullptr;
  double* ptab = nullptr;
  float* ptabf = nullptr;
  if (product && M <= kProdMaxM) {
    prod = cv.take<int>(kProdInts);
    ptab = cv.take<double>(16 * static_cast<size_t>(D));
    ptabf = cv.take<float>(16 * static_cast<size_t>(D));
    if (M <= kSmallM) frag = nullptr;
  }
  if (one_launch(M, D)) {
    const int threads = M * D <= 1024 ? 256 : kOneThreads;    // fewer wavefronts to bring to each barrier
    const int rows = !frag ? 1 : (Mpad * 2 * KS + threads - 1) / threads;
    // at most 130 KiB: 1024 points of 30 coordinates, or kOneStage floats and 8192 labels
    const size_t lds = sizeof(uint32_t) * M + sizeof(float) * (16 * static_cast<size_t>(D) + static_cast<size_t>(M) * (D | 1));
    const int st = set_lds_limit(reinterpret_cast<const void*>(prep_one_kernel), 160 * 1024 - 1024);
    if (st != MD_OK) return st;
    hipLaunchKernelGGL(prep_one_kernel, dim3(1 + rows), dim3(threads), lds, stream, d_X, d_labels, M, Mpad, D,
                       magic_of(D), magic_of(ilog2_pow2(M)), KS, sc, alpha, c_over_alpha, xl, frag, flags, vx, prod, ptab, ptabf);
    MD_LAUNCH_CHECK("prep_one_kernel launch");
  } else {
    const int bs = 256;
    hipLaunchKernelGGL(prep_init_kernel, dim3((M + bs - 1) / bs), dim3(bs), 0, stream, inv, M, flags);
    MD_LAUNCH_CHECK("prep_init_kernel launch");
    hipLaunchKernelGGL(prep_scatter_kernel, dim3((M + bs - 1) / bs), dim3(bs), 0, stream, d_labels, M, inv, flags);
    MD_LAUNCH_CHECK("prep_scatter_kernel launch");
    hipLaunchKernelGGL(prep_build_kernel, dim3((M + bs - 1) / bs), dim3(bs), 0, stream, d_X, d_labels, inv, M, D, KS,
                       sc, alpha, c_over_alpha, xl, frag, flags);
    MD_LAUNCH_CHECK("prep_build_kernel launch");
  }
  out->xl = xl;
  out->frag = frag;
  out->flags = flags;
  out->fb_list = fb;
  out->fb_list2 = fb2;
  out->vx = vx;
  out->prod = prod;
  out->ptab = ptab;
  out->ptabf = ptabf;
  out->ks = KS;
  out->sc = sc;
  out->alpha = alpha;
  out->c_over_alpha = c_over_alpha;
  return MD_OK;
}

}  // namespace md
