// Line kernels with complex128 storage: storing launches, the general form
// (a file per type and kind, so that they compile in parallel).
#include "lines_kernel.h"

namespace helm {
namespace linek {
template hipError_t launch_lines_kernel<double2, false, false>(const LineDev& d, int P, int64_t blocks, hipStream_t s);
}  // namespace linek
}  // namespace helm
