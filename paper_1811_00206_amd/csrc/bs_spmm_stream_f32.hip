// SpMM kernels that walk K in stages, fp32 values (see bs_spmm_stream_kernel.h).
#include "bs_spmm_stream_kernel.h"

namespace bs {
int spmm_stream_launch_f32(const SpmmStreamArgs& a, const SpmmLaunch& l) { return spmm_stream_launch_k<float, uint8_t>(a, l); }
}  // namespace bs
