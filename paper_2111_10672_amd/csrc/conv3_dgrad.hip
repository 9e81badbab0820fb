// 3 x 3 convolutions over resident rows: input gradient (weights [channel][tap][n]).
#include "conv3_impl.h"

namespace spb {

hipError_t launch_conv3_dgrad(const GemmProblem& p, hipStream_t stream) { return gemm_dma_detail::launch_conv3<Layout::KRow>(p, stream); }

}  // namespace spb
