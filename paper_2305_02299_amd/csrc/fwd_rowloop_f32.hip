// ROWLOOP forward kernels, fp32 storage.
#include "fwd_rowloop.inl"
namespace srigl {
srigl_status launch_rowloop_f32(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) { return launch_rowloop_x<float, int32_t>(a, p, st); }
}  // namespace srigl
