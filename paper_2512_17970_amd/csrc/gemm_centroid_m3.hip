// Centroid kernels for m = 3 codebooks (see gemm_centroid_impl.h and gemm_prompt_impl.h).
#include "gemm_prompt_impl.h"

namespace cg {
int launch_gemm_centroid_m3(const Geometry& g, const GemmParams& p, hipStream_t stream) { return launch_gemm_centroid_m<3>(g, p, stream); }
}  // namespace cg
