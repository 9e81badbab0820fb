// 3 x 3 convolutions over resident rows: forward (weights [n][tap][channel]).
#include "conv3_impl.h"

namespace spb {

hipError_t launch_conv3_fwd(const GemmProblem& p, hipStream_t stream) { return gemm_dma_detail::launch_conv3<Layout::RowK>(p, stream); }

}  // namespace spb
