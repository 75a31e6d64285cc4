// The prompt kernel (ccq_block.h) on per-group mixes.
#include "ccq_block.h"

namespace ccq {

template __global__ void ccq_block_kernel<3, 0, 4>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 0, 5>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 0, 6>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 0, 7>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 0, 8>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 1, 4>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 1, 5>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 1, 6>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 1, 7>(const BlockArgs);
template __global__ void ccq_block_kernel<3, 1, 8>(const BlockArgs);
template __global__ void ccq_block_grouped_kernel<3, 0>(const BlockArgs);
template __global__ void ccq_block_grouped_kernel<3, 1>(const BlockArgs);

BlockKernel block_kernel_mix(int scale_mode, int mt) { return scale_mode == 0 ? block_rows<3, 0>(mt) : block_rows<3, 1>(mt); }
BlockKernel block_grouped_mix(int scale_mode) { return scale_mode == 0 ? ccq_block_grouped_kernel<3, 0> : ccq_block_grouped_kernel<3, 1>; }

}  // namespace ccq
