// The counting pass's Alg. 2 (skip) walks over a VDB tree: hierarchical,
// voxel and sub-leaf steps, single- and multi-level, tree in LDS or not.
// In a source of their own only to compile beside the rest; sample.hip
// launches them.
#pragma clang fp contract(off)

#include "count.hpp"

namespace ogv {

#define OGV_COUNT_SKIP(V, L, L1)                                                                               \
    template __global__ void count_kernel<V, true, L, L1>(GridView, const float *, const float *, int64_t, Lattice, \
                                                          int32_t *, int32_t *, RunPool, int, RowMap, int64_t *,    \
                                                          int64_t *);
OGV_COUNT_SKIP_ALL
#undef OGV_COUNT_SKIP

}  // namespace ogv
