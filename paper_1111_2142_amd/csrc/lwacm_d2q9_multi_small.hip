// lwacm_d2q9_multi_small.hip -- the multi-step D2Q9 kernels on tiles of 8 and 16
// nodes (small grids, link-wall distances, link velocities).
#include "lwacm_d2q9_multi.hpp"

namespace lwacm {

template <>
void launch_fwd_multi_tile<8>(const ProblemArgs &p, unsigned nb, const MultiFwd &f,
                               const ReduceArgs &r, hipStream_t s)
{
    fwd_multi_tile<8>(p, nb, f, r, s);
}

template <>
void launch_adj_multi_tile<8>(const ProblemArgs &p, unsigned nb, const MultiAdj &a, hipStream_t s)
{
    adj_multi_tile<8>(p, nb, a, s);
}

template <>
void launch_fwd_multi_tile<16>(const ProblemArgs &p, unsigned nb, const MultiFwd &f,
                               const ReduceArgs &r, hipStream_t s)
{
    fwd_multi_tile<16>(p, nb, f, r, s);
}

template <>
void launch_adj_multi_tile<16>(const ProblemArgs &p, unsigned nb, const MultiAdj &a, hipStream_t s)
{
    adj_multi_tile<16>(p, nb, a, s);
}

}  // namespace lwacm
