// Line kernels with complex64 storage: reducing launches, real sigma
// (a file per type and kind, so that they compile in parallel).
#include "lines_kernel.h"

namespace helm {
namespace linek {
template hipError_t launch_lines_kernel<float2, true, true>(const LineDev& d, int P, int64_t blocks, hipStream_t s);
}  // namespace linek
}  // namespace helm
