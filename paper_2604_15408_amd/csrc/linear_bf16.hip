// The linear kernel for BF16 inputs.
#include "linear_kernel.h"

namespace ragged {

hipError_t launch_linear_bf16(int nj, int mt, int groups, const LinearArgs& args, hipStream_t stream) {
    return launch_linear_tile<BF16>(nj, mt, groups, args, stream);
}

}  // namespace ragged
