// lwacm_d2q9_strip.hip -- eight D2Q9 steps per launch on large grids without
// walls or force: each wave marches a strip of columns in y.
//
// A wave's 64 lanes are 64 neighbouring columns, of which the middle 48 are its
// output; it loads row after row, and eight levels (steps) follow each other one
// row apart, so that the row a step makes is the next step's newest row.  The
// link terms are formed once, by the node they start from (the tile kernels of
// lwacm_d2q9_multi.hpp form them at each of the nodes they reach), go to the
// neighbouring columns by DPP wave shifts and wait in registers for the rows
// above: no LDS and no barriers.  Terms, sums and normalisation are the
// operations of link_update (lwacm_generic_update.hpp) in its order, so the
// fields are bitwise those of single steps.
//
// Bound by VALU issue: about 75 instructions a node and step against about 90 and
// seven 16-byte LDS reads in the tile kernels.  The halo costs 64 / 48 in x (8
// columns a side, one a step) and, with the levels started as their first rows
// arrive, (rows + 7) / rows in y.  d2q9_strip_choose_rows has the times.
#include <type_traits>

#include "lwacm_device.hpp"
#include "lwacm_generic_update.hpp"
#include "lwacm_internal.hpp"

namespace lwacm {

namespace {

constexpr int K = kMultiSteps;       // steps per launch
constexpr int SW = kWave - 2 * K;    // output columns of a wave
constexpr int WPB = 4;               // waves per workgroup
constexpr int NT = WPB * kWave;

// the value of the lane to the left or right (the wave's end lanes get 0: they
// are halo columns whose nodes are no longer needed)
__device__ __forceinline__ float from_left(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, v), 0x138 /* wave_shr:1 */, 0xf, 0xf, true));
}

__device__ __forceinline__ float from_right(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, v), 0x130 /* wave_shl:1 */, 0xf, 0xf, true));
}

// The terms s_i of one row's nodes as they arrive in a column (already shifted
// in x), by relaxation A; s0 with s[0].
__device__ __forceinline__ void row_terms(float dr, float rx, const float (&u)[3], float B, float A,
                                          float (&s)[9])
{
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if (i == 0) {
            s[0] = fmaf(rx, B, dr);
        } else {
            const float t = link_term_unweighted(dr, rx, vdot<9>(i, u), B, A);
            s[i] = link_cx(i) > 0 ? from_left(t) : (link_cx(i) < 0 ? from_right(t) : t);
        }
    }
}

// What one level keeps between rows: of its two last source rows the links
// going up (3, 5, 8; slot = the row's parity), and of the last row the own
// state and the sums over its links 0 to 2.
template <bool SPLIT>
struct Level {
    float s3[2], s5[2], s8[2];
    float p3[SPLIT ? 2 : 1], p5[SPLIT ? 2 : 1], p8[SPLIT ? 2 : 1];  // the density's terms
    float D, J0, rx, ux, uy;
};

// Row (dr, u), of parity PAR, arrives at a level, whose node of the row below is
// complete with it: its new state replaces (dr, u).
template <bool SPLIT, int PAR>
__device__ __forceinline__ void arrive(const ProblemArgs &p, Level<SPLIT> &l, float &dr, float &ux,
                                       float &uy)
{
    constexpr int Q = SPLIT ? PAR : 0;
    const float u[3] = {ux, uy, 0.0f};
    const float rx = 1.0f + dr, B = node_B(u);
    float s[9], sp[9];
    row_terms(dr, rx, u, B, p.A, s);
    if (SPLIT) row_terms(dr, rx, u, B, p.Ap, sp);
    const float(&d)[9] = SPLIT ? sp : s;  // the density's terms
    // 36 w s is exact, so each fma rounds like adding it
    const float a3 = l.s3[PAR], a5 = l.s5[PAR], a8 = l.s8[PAR];
    const float d3 = SPLIT ? l.p3[Q] : a3, d5 = SPLIT ? l.p5[Q] : a5, d8 = SPLIT ? l.p8[Q] : a8;
    float D = fmaf(4.0f, d3, l.D);
    D = fmaf(4.0f, d[4], D);
    D += d5;
    D += d[6];
    D += d[7];
    D += d8;
    const float J0 = l.J0 + a5 - s[6] + s[7] - a8;
    const float J1 = fmaf(-4.0f, s[4], 4.0f * a3) + a5 - s[6] - s[7] + a8;
    const float J[2] = {J0, J1}, uo[3] = {l.ux, l.uy, 0.0f};
    float out[3], e;
    finish_node<2>(p, l.rx, uo, D, J, out, e);
    l.s3[PAR] = s[3];
    l.s5[PAR] = s[5];
    l.s8[PAR] = s[8];
    if (SPLIT) {
        l.p3[Q] = sp[3];
        l.p5[Q] = sp[5];
        l.p8[Q] = sp[8];
    }
    l.D = fmaf(4.0f, d[2], fmaf(4.0f, d[1], 16.0f * d[0]));
    l.J0 = fmaf(-4.0f, s[2], 4.0f * s[1]);
    l.rx = rx;
    l.ux = ux;
    l.uy = uy;
    dr = out[0];
    ux = out[1];
    uy = out[2];
}

template <bool SPLIT>
__global__ __launch_bounds__(NT) void k_fwd_d2q9_strip(ProblemArgs p, const float *__restrict__ src,
                                                       float *__restrict__ dst, int rows,
                                                       ReduceArgs r)
{
    const int lane = threadIdx.x % kWave;
    const unsigned w = (unsigned)__builtin_amdgcn_readfirstlane(blockIdx.x * WPB + threadIdx.x / kWave);
    const unsigned strips = (unsigned)(p.nx + SW - 1) / SW;
    const int x0 = (int)(w % strips) * SW;
    const int y0 = (int)min((long long)(w / strips) * rows, (long long)p.ny);
    const int nout = min(rows, p.ny - y0);  // 0: past the last strip
    double acc[2] = {0.0, 0.0};
    if (nout > 0) {
        const int x = x0 - K + lane;
        const bool put = lane >= K && lane < K + SW && x < p.nx;
        int gx = x % p.nx;
        gx = gx < 0 ? gx + p.nx : gx;
        int yl = (y0 - K) % p.ny;  // the row to load next, wrapped
        yl = yl < 0 ? yl + p.ny : yl;
        float in[2][3];
        auto load = [&](float (&v)[3]) {
            const float *a = src + 3 * (size_t)yl * p.nx + 3 * (size_t)gx;
            v[0] = a[0];
            v[1] = a[1];
            v[2] = a[2];
            yl = yl + 1 == p.ny ? 0 : yl + 1;
        };
        load(in[0]);
        load(in[1]);
        Level<SPLIT> lv[K] = {};
        // source row j (from y0 - K) arrives at level 1; level s + 1 gets row
        // j - s of level s, which is right from j = 2 s on
        auto row = [&](auto par, int j, int last) {  // levels 1 .. last + 1 run
            constexpr int PAR = decltype(par)::value;
            float dr = in[PAR][0], ux = in[PAR][1], uy = in[PAR][2];
            load(in[PAR]);  // row j + 2 (wrapped: also past the strip's last row a row of src)
#pragma unroll
            for (int s = 0; s < K; ++s) {
                if (s > last) return;
                arrive<SPLIT, PAR>(p, lv[s], dr, ux, uy);
            }
            if (last == K) {
                const int y = y0 + j - 2 * K;
                if (put && y < y0 + nout) {
                    float *o = dst + 3 * (size_t)y * p.nx + 3 * (size_t)x;
                    o[0] = dr;
                    o[1] = ux;
                    o[2] = uy;
                    float e = 0.0f;
                    e = fmaf(ux, ux, e);
                    e = fmaf(uy, uy, e);
                    acc[0] += (double)dr;
                    acc[1] += 0.5 * (double)e;
                }
            }
        };
        using Even = std::integral_constant<int, 0>;
        using Odd = std::integral_constant<int, 1>;
#pragma unroll 1
        for (int m = 0; m < K; ++m) {
            row(Even{}, 2 * m, m);
            row(Odd{}, 2 * m + 1, m);
        }
#pragma unroll 1
        for (int j = 2 * K; j < 2 * K + nout; j += 2) {
            row(Even{}, j, K);
            row(Odd{}, j + 1, K);
        }
    }
    store_block_partials<2>(acc, r.partials, blockIdx.x);
    if (blockIdx.x == 0 && r.prev_nblocks)
        finish_previous_sums(r.prev_partials, r.prev_nblocks, r.prev_out, r.prev_out2);
}

long long strip_waves(const ProblemArgs &p, int rows)
{
    return ((long long)(p.nx + SW - 1) / SW) * ((p.ny + rows - 1) / rows);
}

}  // namespace

bool d2q9_strip_supported(const ProblemArgs &p)
{
    return p.Q == 9 && p.nz == 1 && !p.mask && !p.has_force && p.strip_rows[p.split] > 0;
}

// Rows per wave: a SIMD's waves run one after the other, each (rows + 8) rows long
// (the levels' start costs about eight), so the least ceil(waves / SIMDs) *
// (rows + 8).  Eight steps take 10.6 + 1.085 us times that (with omega_p 11 +
// 1.63); on tiles of 32, which run a round of one per CU at a time, 6 + 10 us
// times the rounds (with omega_p 5 + 12), so strips are taken where
// cost + 5 < 9 rounds, with omega_p where 1.63 cost + 6 < 12 rounds.  Tiles / strips:
// 512^2 17.5 / 24.9, 600^2 26.3 / 27.7, 1024 x 512 25.2 / 32.3, 724^2 36.6 / 32.3,
// 1024^2 44.3 / 44.5, 1501 x 1003 63.0 / 54.0, 2000^2 156 / 114, 4096^2 608 / 392;
// with omega_p 724^2 43.4 / 43.6, 961 x 1009 55.4 / 59.6, 1501 x 1003 80.3 / 76.8,
// 2000^2 188 / 161.
void d2q9_strip_choose_rows(ProblemArgs &p, int ncu)
{
    if (ncu < 1) ncu = 1;
    int best = 0;
    long long best_cost = 0;
    for (int m = 1; m <= p.ny; ++m) {
        const int rows = (p.ny + m - 1) / m;
        if (m > 1 && (rows < 4 || strip_waves(p, rows) > 16LL * ncu)) break;
        const long long cost = ((strip_waves(p, rows) + 4LL * ncu - 1) / (4LL * ncu)) * (rows + 8LL);
        if (!best || cost < best_cost) {
            best = rows;
            best_cost = cost;
        }
    }
    const long long tiles = ((p.nx + 31LL) / 32) * ((p.ny + 31LL) / 32);
    const long long rounds = (tiles + ncu - 1) / ncu;
    p.strip_rows[0] = best_cost + 5 < 9 * rounds ? best : 0;
    p.strip_rows[1] = 163 * best_cost + 600 < 1200 * rounds ? best : 0;
}

unsigned d2q9_strip_num_blocks(const ProblemArgs &p)
{
    return (unsigned)((strip_waves(p, p.strip_rows[p.split]) + WPB - 1) / WPB);
}

hipError_t launch_fwd_d2q9_strip(const ProblemArgs &p, const float *src, float *dst,
                                 const ReduceArgs &r, hipStream_t s)
{
    if (!d2q9_strip_supported(p)) return hipErrorInvalidValue;
    const unsigned nb = d2q9_strip_num_blocks(p);
    if (p.split) k_fwd_d2q9_strip<true><<<nb, NT, 0, s>>>(p, src, dst, p.strip_rows[p.split], r);
    else k_fwd_d2q9_strip<false><<<nb, NT, 0, s>>>(p, src, dst, p.strip_rows[p.split], r);
    return hipGetLastError();
}

}  // namespace lwacm
