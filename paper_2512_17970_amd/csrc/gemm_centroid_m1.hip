// Centroid kernels for m = 1 codebook (see gemm_centroid_impl.h and gemm_prompt_impl.h).
#include "gemm_prompt_impl.h"

namespace cg {
int launch_gemm_centroid_m1(const Geometry& g, const GemmParams& p, hipStream_t stream) { return launch_gemm_centroid_m<1>(g, p, stream); }
}  // namespace cg
