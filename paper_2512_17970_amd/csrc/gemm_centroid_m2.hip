// Centroid kernels for m = 2 codebooks (see gemm_centroid_impl.h and gemm_prompt_impl.h).
#include "gemm_prompt_impl.h"

namespace cg {
int launch_gemm_centroid_m2(const Geometry& g, const GemmParams& p, hipStream_t stream) { return launch_gemm_centroid_m<2>(g, p, stream); }
}  // namespace cg
