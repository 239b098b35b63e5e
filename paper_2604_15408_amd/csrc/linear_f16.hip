// The linear kernel for F16 inputs.
#include "linear_kernel.h"

namespace ragged {

hipError_t launch_linear_f16(const TileShape& shape, int groups, const LinearArgs& args, hipStream_t stream) {
    return launch_linear_tile<F16>(shape, groups, args, stream);
}

}  // namespace ragged
