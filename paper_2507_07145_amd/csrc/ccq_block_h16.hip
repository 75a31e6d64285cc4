// The prompt kernel (ccq_block.h) on hybrid-word weights.
#include "ccq_block.h"

namespace ccq {

template __global__ void ccq_block_kernel<4, 0, 4>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 0, 5>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 0, 6>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 0, 7>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 0, 8>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 1, 4>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 1, 5>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 1, 6>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 1, 7>(const BlockArgs);
template __global__ void ccq_block_kernel<4, 1, 8>(const BlockArgs);
template __global__ void ccq_block_grouped_kernel<4, 0>(const BlockArgs);
template __global__ void ccq_block_grouped_kernel<4, 1>(const BlockArgs);

BlockKernel block_kernel_h16(int scale_mode, int mt) { return scale_mode == 0 ? block_rows<4, 0>(mt) : block_rows<4, 1>(mt); }
BlockKernel block_grouped_h16(int scale_mode) { return scale_mode == 0 ? ccq_block_grouped_kernel<4, 0> : ccq_block_grouped_kernel<4, 1>; }

}  // namespace ccq
