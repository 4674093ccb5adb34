// Instantiation of the tree descent: 7 waves per SIMD, as many as its LDS leaves
// room for, since its waves are chains of dependent scalar and vector operations.
#include "launch.h"
#include "tree_kernel.h"

namespace wpm {

hipError_t launch_tree(dim3 grid, dim3 block, size_t lds, hipStream_t st, const uint32_t *tables,
                       const int64_t *offsets, const wpm_item *items, const KArgs &a) {
    hipLaunchKernelGGL(tree_kernel<7>, grid, block, lds, st, tables, offsets, items, a);
    return hipGetLastError();
}

hipError_t occupancy_tree(int *nb, int block, size_t lds) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, tree_kernel<7>, block, lds);
}

}  // namespace wpm
