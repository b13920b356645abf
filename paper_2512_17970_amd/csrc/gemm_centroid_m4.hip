// Centroid kernels for m = 4 codebooks (see gemm_centroid_impl.h and gemm_prompt_impl.h).
#include "gemm_prompt_impl.h"

namespace cg {
int launch_gemm_centroid_m4(const Geometry& g, const GemmParams& p, hipStream_t stream) { return launch_gemm_centroid_m<4>(g, p, stream); }
}  // namespace cg
