// 2-bit table kernels on the sparse matrix instruction with staged operands, entries beyond int8 as two int8 planes.
#include "dg_sparse_staged_kernel.h"

namespace dgoh {
void unit_sparse_staged_two(const DgProblem &p, const Pools &pools, const Plan &q, int64_t wave_tiles, hipStream_t stream)
{
    launch_sparse_staged<false, true>(p, pools, 0, q, wave_tiles, stream);
}
}   // namespace dgoh
