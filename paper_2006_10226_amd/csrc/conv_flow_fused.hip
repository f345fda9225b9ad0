// Instantiations of the short-loop conv kernel (conv_flow_kernel.h) whose
// epilogue applies a residual qnn.add, in a source of their own so that they
// compile beside the plain ones.
#include "conv_flow_kernel.h"

namespace qnn {

hipError_t launch_conv_flow_fused(const ConvArgs &a, int tile, hipStream_t st)
{
    if (!a.res || !a.staged)
        return hipErrorInvalidValue;
    return launch_flow_from<0, true>(a, tile, st);
}

}  // namespace qnn
