// The product kernel (llr_prod.hpp) as a launch of its own: M <= 16, and constellations whose general
// path is the matrix-core kernel.  (M = 32 and 64 with D <= 8 call it from their own kernel.)
#include "llr_prod.hpp"
#include "llr_kernels.hpp"

namespace md {
namespace {

using namespace prodk;

template <int MODE, bool GMI, int DT>
__global__ void __launch_bounds__(kProdThreads) llr_prod_kernel(ProdArgs G, const int* __restrict__ flags, SymbolArgs A) {
  ConstInt* fl = reinterpret_cast<ConstInt*>(reinterpret_cast<uint64_t>(flags));
  if (!fl[5]) return;
  all_symbols<MODE, GMI, DT, 0>(G, flags, A);
}

template <int MODE, bool GMI, int DT>
int launch_prod_d(const Prepared& P, int M, int D, const float* d_y, int64_t N, double sigma2, float* d_llr,
                  hipStream_t stream) {
  auto kern = llr_prod_kernel<MODE, GMI, DT>;
  int ncu = 0, occ = 0;
  MD_TRY(device_cus(&ncu));
  MD_TRY(blocks_per_cu(reinterpret_cast<const void*>(kern), kProdThreads, 0, &occ));
  // one resident set of blocks, each taking the same number of passes: a second, part-filled set
  // would run as long as the first
  const int64_t need = (N + kProdThreads - 1) / kProdThreads;
  const int64_t passes = (need + static_cast<int64_t>(ncu) * occ - 1) / (static_cast<int64_t>(ncu) * occ);
  const int64_t grid = (need + passes - 1) / passes;
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(kProdThreads), 0, stream, prod_args(P), P.flags,
                     symbol_args(P, M, D, d_y, N, sigma2, d_llr));
  MD_LAUNCH_CHECK("llr_prod_kernel launch");
  return MD_OK;
}

template <int MODE, bool GMI>
int launch_prod_t(const Prepared& P, int M, int D, const float* d_y, int64_t N, double sigma2, float* d_llr,
                  hipStream_t stream) {
  if (D == 2) return launch_prod_d<MODE, GMI, 2>(P, M, D, d_y, N, sigma2, d_llr, stream);
  if (D == 4) return launch_prod_d<MODE, GMI, 4>(P, M, D, d_y, N, sigma2, d_llr, stream);
  return launch_prod_d<MODE, GMI, 0>(P, M, D, d_y, N, sigma2, d_llr, stream);
}

}  // namespace

int launch_prod(const Prepared& P, int M, int D, const float* d_y, int64_t N, double sigma2, bool maxlog,
                float* d_llr, hipStream_t stream) {
  if (!P.prod) return fail(MD_EUNSUPPORTED, "the call was prepared without the product analysis");
  if (maxlog) return launch_prod_t<PROD_MAXLOG, false>(P, M, D, d_y, N, sigma2, d_llr, stream);
  if (M <= kSmallM) return launch_prod_t<PROD_DOUBLE, false>(P, M, D, d_y, N, sigma2, d_llr, stream);
  return P.gmi_terms ? launch_prod_t<PROD_FLOAT, true>(P, M, D, d_y, N, sigma2, d_llr, stream)
                     : launch_prod_t<PROD_FLOAT, false>(P, M, D, d_y, N, sigma2, d_llr, stream);
}

}  // namespace md
