// SpMM kernels that walk K in stages, 16-bit offsets (see bs_spmm_stream_kernel.h).
#include "bs_spmm_stream_kernel.h"

namespace bs {
namespace {
template <typename VT>
int launch_wide(const SpmmStreamArgs& a, const SpmmLaunch& l) {
    return a.k < 8 ? spmm_stream_launch_one<VT, uint16_t, -4>(a, l) : spmm_stream_launch_one<VT, uint16_t, -8>(a, l);
}
}  // namespace
int spmm_stream_launch_wide(int dtype, const SpmmStreamArgs& a, const SpmmLaunch& l) {
    return dtype == BS_F16 ? launch_wide<__half>(a, l) : launch_wide<float>(a, l);
}
}  // namespace bs
