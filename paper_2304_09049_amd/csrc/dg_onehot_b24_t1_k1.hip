// 3- and 4-bit codes as two 2-bit ones each on the sparse matrix instruction (activations on the MFMA rows: output stride-1 axis = m).
// (One translation unit per variant keeps build times even.)
#include "dg_onehot_kernel.h"

namespace dgoh {
void unit_main_b24_t1_k1(const DgProblem &p, const Pools &pools, const Plan &q, int64_t wave_tiles, hipStream_t stream)
{
    launch_main<24, true, false, 1>(p, pools, q, wave_tiles, stream);
}

void unit_split_b24_t1(const DgProblem &p, const Pools &pools, const Plan &q, int64_t blocks11, hipStream_t stream)
{
    launch_split<24, true, false>(p, pools, q, blocks11, stream);
}
}   // namespace dgoh
