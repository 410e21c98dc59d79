// ROWLOOP forward kernels, bf16 storage.
#include "fwd_rowloop.inl"
namespace srigl {
srigl_status launch_rowloop_bf16(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) { return launch_rowloop_x<uint16_t, int32_t>(a, p, st); }
}  // namespace srigl
