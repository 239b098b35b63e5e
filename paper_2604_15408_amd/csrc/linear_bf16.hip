// The linear kernel for BF16 inputs.
#include "linear_kernel.h"

namespace ragged {

hipError_t launch_linear_bf16(const TileShape& shape, int groups, const LinearArgs& args, hipStream_t stream) {
    return launch_linear_tile<BF16>(shape, groups, args, stream);
}

}  // namespace ragged
