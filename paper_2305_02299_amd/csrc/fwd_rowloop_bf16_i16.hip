// ROWLOOP forward kernels, bf16 storage, 16-bit indices.
#include "fwd_rowloop.inl"
namespace srigl {
srigl_status launch_rowloop_bf16_i16(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) { return launch_rowloop_x<uint16_t, uint16_t>(a, p, st); }
}  // namespace srigl
