// 3- and 4-bit codes as two 2-bit ones each on the sparse matrix instruction, weight operands stationary in registers.
// (One translation unit per variant keeps build times even.)
#include "dg_sparse_ws_kernel.h"

namespace dgoh {
void unit_sparse_ws_nib(const DgProblem &p, const Pools &pools, int streams, hipStream_t stream)
{
    launch_sparse_ws<true>(p, pools, streams, false, stream);
}
}   // namespace dgoh
