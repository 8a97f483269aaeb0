// Stand-ins for the sweep kernels' launchers, linked into the sanitizer test's driver in
// place of the kernel sources: every call the driver makes fails its argument checks before
// any launch, so these are never called.
#include "../paper_2510_27351_amd/csrc/wf_path.h"
#include "../paper_2510_27351_amd/csrc/wf_soft.h"

namespace wf {
hipError_t launch_forward(int, int, const FwdArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_select(int, const SelArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_adjoint(int, int, const AdjArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_forward_soft(int, const FwdArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_soft_backward(int, const SoftArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_select_path(int, const SelArgs&, const PathLabels&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_zero(int, void*, int64_t, int64_t, int64_t, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_path(int, const PathArgs&, hipStream_t) { return hipErrorInvalidValue; }
}  // namespace wf
