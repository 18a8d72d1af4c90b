// lwacm_d2q9_multi.hip -- several D2Q9 steps per launch: tiles of 32 nodes, the
// choice of the tile and the launchers.
#include "lwacm_d2q9_multi.hpp"

namespace lwacm {

template <>
void launch_fwd_multi_tile<32>(const ProblemArgs &p, unsigned nb, const MultiFwd &f,
                               const ReduceArgs &r, hipStream_t s)
{
    fwd_multi_tile<32>(p, nb, f, r, s);
}

template <>
void launch_adj_multi_tile<32>(const ProblemArgs &p, unsigned nb, const MultiAdj &a, hipStream_t s)
{
    adj_multi_tile<32>(p, nb, a, s);
}

static long long tiles_of(const ProblemArgs &p, int mt)
{
    return ((long long)(p.nx + mt - 1) / mt) * ((p.ny + mt - 1) / mt);
}

// The smallest tile whose workgroups the device takes about one per CU: a small
// tile's launch is the shorter one (fewer nodes per workgroup and step), but
// recomputes more of the halo.  Eight steps on tiles of 8 / 16 / 32 nodes: 9.6 /
// 11.2 / 16.1 us at 128^2 (256 / 64 / 16 workgroups), 12.1 / 11.5 / 16.2 at
// 164^2, 19.1 / 11.5 / 16.3 at 256^2, 15.2 (16) against 16.5 (32) at 324^2, 22 /
// 16.8 at 512^2, 93 / 63 at 1501 x 1003.
void d2q9_multi_choose_tile(ProblemArgs &p, int ncu)
{
    p.multi_tile = tiles_of(p, 8) <= ncu ? 8 : (4 * tiles_of(p, 16) <= 7 * ncu ? 16 : 32);
    p.multi_many = tiles_of(p, 32) > ncu;
}

// the tile of a launch: link data fit the small tiles' LDS only
static int multi_tile(const ProblemArgs &p)
{
    return p.multi_tile > 16 && (p.qd || p.uwl) ? 16 : p.multi_tile;
}

bool d2q9_multi_supported(const ProblemArgs &p)
{
    return p.Q == 9 && p.nz == 1 && p.nx >= 1 && p.ny >= 1 && p.multi_tile > 0 &&
           (p.mask || (!p.qd && !p.uwl));
}

unsigned d2q9_multi_num_blocks(const ProblemArgs &p)
{
    return (unsigned)tiles_of(p, multi_tile(p));
}

hipError_t launch_adj_d2q9_multi(const ProblemArgs &p, const float *states, size_t slot_floats,
                                 int slot_hi, int ksteps, int final_last, const float *mu_in,
                                 float *mu_out, double *partials, size_t stride, unsigned slice0,
                                 hipStream_t s)
{
    if (!d2q9_multi_supported(p) || ksteps < 1 || ksteps > kMultiSteps || slot_hi < ksteps - 1)
        return hipErrorInvalidValue;
    const unsigned nb = d2q9_multi_num_blocks(p);
    const MultiAdj a{states, slot_floats, slot_hi, ksteps,  final_last,
                     mu_in,  mu_out,      partials, stride, slice0};
    switch (multi_tile(p)) {
    case 8: launch_adj_multi_tile<8>(p, nb, a, s); break;
    case 16: launch_adj_multi_tile<16>(p, nb, a, s); break;
    default: launch_adj_multi_tile<32>(p, nb, a, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_fwd_d2q9_multi(const ProblemArgs &p, const float *src, float *dst, int ksteps,
                                 const ReduceArgs &r, hipStream_t s, float *slots,
                                 size_t slot_floats)
{
    if (!d2q9_multi_supported(p) || ksteps < 1 || ksteps > kMultiSteps) return hipErrorInvalidValue;
    const unsigned nb = d2q9_multi_num_blocks(p);
    const MultiFwd f{src, dst, ksteps, slots, slot_floats};
    switch (multi_tile(p)) {
    case 8: launch_fwd_multi_tile<8>(p, nb, f, r, s); break;
    case 16: launch_fwd_multi_tile<16>(p, nb, f, r, s); break;
    default: launch_fwd_multi_tile<32>(p, nb, f, r, s); break;
    }
    return hipGetLastError();
}

}  // namespace lwacm
