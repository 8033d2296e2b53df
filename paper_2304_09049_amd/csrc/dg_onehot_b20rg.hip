// 2-bit table kernel on the sparse matrix instruction for filter taps that are no whole 32-position groups.
#include "dg_sparse_ragged_kernel.h"

namespace dgoh {
void unit_sparse_ragged(const DgProblem &p, const Pools &pools, const RaggedPlan &q, bool scale_rows, bool n_first, bool raw, hipStream_t stream)
{
    launch_ragged(p, pools, q, scale_rows, n_first, raw, stream);
}
}   // namespace dgoh
