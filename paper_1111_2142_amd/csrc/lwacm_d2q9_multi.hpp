// lwacm_d2q9_multi.hpp -- several D2Q9 steps per launch (temporal blocking): the
// kernels (instantiated by lwacm_d2q9_multi.hip and lwacm_d2q9_multi_small.hip).
//
// The 2D workloads are small (64^2 to 512^2 nodes: under a microsecond of
// HBM time per step), so one launch per step is bound by the interval between
// dependent launches (about 4 us on this device), not by the step.  Here a
// workgroup owns an MT x MT tile of output nodes, loads the tile and a halo of
// K = 8 nodes on every side (periodic wrap) into LDS once, and advances the
// region K steps in LDS: step s is computed on the region less s nodes on
// each side, which is exactly what the next step needs, so after K steps the
// tile is exact.  Each node is updated by the same function as the one-step
// kernel (link_update in lwacm_generic_update.hpp), so the fields are bitwise
// those of K single steps.  The mass and energy of the last step are summed
// per workgroup in FP64 (a different order than the one-step kernel's, so
// equal to FP64 rounding only).
//
// A launch is bound by one workgroup's own steps: VALU issue and LDS reads of
// the region on its compute unit.  Tiles of 32 nodes waste the least on the
// halo (1.5 node updates per output node and step) and serve grids that fill
// the chip with them; smaller grids take tiles of 16 (2.1) or 8 (3.8), which
// spread the same nodes over more compute units (d2q9_multi_choose_tile).
//
// Large grids without walls or force take eight steps at a time as strips in
// registers instead (lwacm_d2q9_strip.hip).
//
// FP32 storage, one to eight steps per launch.  What the steps need beyond the
// states is put into LDS with them: a force field (two floats a node), the
// wall-motion terms of the per-id table (one float per id and link), and for
// link-wall distances or velocities given link by link the distance and the
// term of the nodes next to a wall (sixteen floats a node: tiles of at most
// 16).  Problems with the semi-implicit update, a temperature, FP16 storage
// or a diagnostics history run one step per launch.
#pragma once

#include "lwacm_device.hpp"
#include "lwacm_generic_update.hpp"
#include "lwacm_internal.hpp"

namespace lwacm {

namespace {

constexpr int MK = kMultiSteps;      // halo width = most steps per launch

// Rows per thread: a strip of MR nodes of one column shares its neighbours'
// loads.  Two rows cost less LDS time, one row gives every SIMD two waves to
// hide latency with: tiles of 8 nodes, and the longer node updates (walls, the
// reverse step), gain by one row (eight steps at 256 x 64, two rows / one:
// tiles of 8 9.9 / 9.6 us, with walls and force 17.3 / 13.5, reverse 18.2 /
// 13.9, tiles of 16 with walls 18.0 / 16.3), the plain update on larger tiles by
// two (tiles of 16 11.3 / 13.2, of 32 16.1 / 21.4).
constexpr int fwd_rows(int MT, bool MASK) { return MT == 8 || (MT == 16 && MASK) ? 1 : 2; }
constexpr int kAdjRows = 1;

// Threads of a workgroup: one per strip of the first step, as far as 1024 go.
constexpr int multi_threads(int MT, int rows)
{
    return (MT == 8 ? 512 : (MT == 16 ? 1024 : 2048)) / rows < 1024
               ? (MT == 8 ? 512 : 1024) / rows
               : 1024;
}

// With walls or a separate omega_p a workgroup of 1024 threads takes more than
// half of a CU's registers, and one runs at a time.  Where tiles of 32 come in
// more than one round, workgroups of 512 run in pairs, and one's arithmetic
// fills the other's barriers and LDS reads (eight steps with walls at 520^2 38.2
// -> 31.3 us, at 1501 x 1003 107 -> 82; omega_p at 1024^2 62.8 -> 50.7; a single
// round is as fast with 1024, and the plain update fits twice as it is).  Not with
// a force field (92 KB of LDS: one workgroup a CU either way) nor with walls, a
// force and omega_p together (136 VGPRs, three waves a SIMD): in pairs of which
// only one runs, eight steps at 520^2 with walls and a field took 57 us, now 49;
// with omega_p beside them 75, now 63; walls, a force and omega_p 74, now 62.
constexpr bool fwd_pair(int MT, bool MASK, int FORCE, bool SPLIT)
{
    return MT == 32 && (MASK || SPLIT) && FORCE < 2 && !(MASK && FORCE && SPLIT);
}
constexpr unsigned kLdsPerCu = 160 * 1024;

// v in [-MK, n + MT + MK) wrapped into [0, n)
template <int MT>
__device__ __forceinline__ int wrap_region(int v, int n)
{
    if (n >= MT + 2 * MK) return v < 0 ? v + n : (v >= n ? v - n : v);
    const int m = v % n;
    return m < 0 ? m + n : m;
}

// The site of a region node without walls around it (see GlobalSite).
template <int FORCE>
struct MultiSite {
    const ProblemArgs &p;
    const float2 *gf;  // force field (FORCE 2)
    int l;
    __device__ __forceinline__ float g(int k) const
    {
        if (FORCE == 2) return k == 0 ? gf[l].x : gf[l].y;
        return p.g[k];
    }
    __device__ __forceinline__ float wall(int, int, uint8_t) const { return 0.0f; }
    __device__ __forceinline__ float wall_p(int, uint8_t) const { return 0.0f; }
    __device__ __forceinline__ bool has_q() const { return false; }
    __device__ __forceinline__ float q(int) const { return 0.5f; }
};

// Walls around a region node, in LDS: the wall-motion terms v_i . uw by wall id
// and link (wtab, wtab_p), or by link and node (wv, QW) with the weight ca of
// the node's own term in the interpolated bounce-back of link ib = opp(i): 2 q
// (bit ib of modes: the second node's term takes the rest) or 1 / (2 q) (bit
// 16 + ib: the node's term of link i takes it).
template <bool QW, int NREG>
struct MultiWalls {
    bool moving;  // some wall-motion term of the table is not zero
    const float *wtab, *wtab_p;
    const float (*ca)[NREG], (*wv)[NREG];
    const unsigned *modes;
};

// link_update (lwacm_generic_update.hpp) for a strip with walls around it:
// every link's term is formed both ways and selected, with the same operations
// in the same order for the one selected, so the results are bitwise
// link_update's.  A branch per link, as there, ran the eight wall links one
// after the other, each waiting for its own LDS reads (eight steps at 256 x 64
// with walls and force 20.5 us, now 13.5; between cylinders at 164^2 42, now 21).
template <bool FORCE, bool SPLIT, bool QW, int NREG, class FSite, class FState>
__device__ __forceinline__ void wall_update(const ProblemArgs &p, const FSite &site,
                                            const MultiWalls<QW, NREG> &walls, float drx,
                                            const float (&ux)[3], float Bx, const FState &fnode,
                                            float (&out)[3])
{
    using L = Lattice<9>;
    const float rx = 1.0f + drx;
    float g3[3] = {0.0f, 0.0f, 0.0f};
    if (FORCE)
#pragma unroll
        for (int k = 0; k < 2; ++k) g3[k] = 3.0f * rx * site.g(k);
    const unsigned modes = QW ? walls.modes[site.l] : 0u;
    float D36 = 0.0f, J36[2] = {0.0f, 0.0f};
    bool dset = false, jset[2] = {false, false};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const float fg = FORCE ? vdot<9>(i, g3) : 0.0f;
        auto addf = [&](float d) { return FORCE ? d + fg : d; };
        float s, sp = 0.0f;
        if (i == 0) {
            s = fmaf(rx, Bx, addf(drx));
            if (SPLIT) sp = s;
        } else {
            const int ib = link_opp(i);
            const float4 y = fnode(-link_cx(i), -link_cy(i));  // upstream node
            const float uy[3] = {y.y, y.z, 0.0f};
            const float cy = vdot<9>(i, uy);
            const bool solid = y.w > 0.0f;
            const int m = solid ? (int)y.w : 0;
            s = link_term_unweighted(addf(y.x), 1.0f + y.x, cy, y.w, p.A);
            if (SPLIT) sp = link_term_unweighted(addf(y.x), 1.0f + y.x, cy, y.w, p.Ap);
            // the term returned by a wall
            const float cb = vdot<9>(ib, ux);
            float sb = link_term_unweighted(addf(drx), rx, cb, Bx, p.A);
            float wsc = 1.0f, wm = 0.0f;
            if (QW) {
                const float ca = walls.ca[QW ? ib - 1 : 0][site.l];
                const bool near = (modes >> ib) & 1u, far = (modes >> (16 + ib)) & 1u;
                const float4 z = fnode(link_cx(i), link_cy(i));  // second node
                const float uz[3] = {z.y, z.z, 0.0f};
                const float so = link_term_unweighted(
                    addf(near ? z.x : drx), near ? 1.0f + z.x : rx,
                    near ? vdot<9>(ib, uz) : vdot<9>(i, ux), near ? z.w : Bx, p.A);
                const float mix = fmaf(ca, sb, (1.0f - ca) * so);
                sb = (near || far) ? mix : sb;
                wsc = far ? ca : 1.0f;
                wm = walls.wv[QW ? i - 1 : 0][site.l];
            } else if (walls.moving) {
                wm = walls.wtab[m * 9 + i];
            }
            const float sw = fmaf(wsc, wm, sb);
            s = solid ? sw : s;
            if (SPLIT) {
                const float wp = walls.moving ? walls.wtab_p[m * 9 + i] : 0.0f;
                const float spw = link_term_unweighted(addf(drx), rx, cb, Bx, p.Ap) + wp;
                sp = solid ? spw : sp;
            }
        }
        s *= L::w36(i);
        accum(D36, dset, SPLIT ? sp * L::w36(i) : s);
        if (link_cx(i) != 0) accum(J36[0], jset[0], link_cx(i) > 0 ? s : -s);
        if (link_cy(i) != 0) accum(J36[1], jset[1], link_cy(i) > 0 ? s : -s);
    }
    float e;
    finish_node<2>(p, rx, ux, D36, J36, out, e);
}

// FORCE: 0 none, 1 uniform, 2 field; SPLIT: a separate omega_p; QW: link-wall
// distances or wall velocities given link by link (with MASK); PAIR: half the
// threads, so that two workgroups share a CU (fwd_pair).
template <int MT, bool MASK, int FORCE, bool SPLIT, bool QW, bool PAIR>
__global__ __launch_bounds__((multi_threads(MT, fwd_rows(MT, MASK)) >> PAIR)) void k_fwd_d2q9_multi(
    ProblemArgs p, const float *__restrict__ src, float *__restrict__ dst, int ksteps, ReduceArgs r,
    float *__restrict__ slots, size_t slot_floats)
{
    static_assert(!QW || (MASK && !SPLIT && MT <= 16), "link data: walls, one omega, small tiles");
    constexpr int MR = fwd_rows(MT, MASK);
    constexpr int NT = multi_threads(MT, MR) >> PAIR;
    constexpr int MW = MT + 2 * MK;      // region side
    constexpr int NREG = MW * MW;
    // per node of the region, two steps' buffers: (rho - 1, u_x, u_y, w) with
    // w = node_B(u) <= -0 at a fluid node (computed once where the node is
    // written, not at each of its eight readers) and w = mask id >= 1 at a
    // solid node
    __shared__ float4 buf[2][NREG];
    __shared__ float2 gf[FORCE == 2 ? NREG : 1];
    __shared__ float wtab[MASK ? 9 * kMaxWallIds : 1], wtab_p[MASK && SPLIT ? 9 * kMaxWallIds : 1];
    constexpr int NQ = QW ? NREG : 1;
    __shared__ float ca[QW ? 8 : 1][NQ], wv[QW ? 8 : 1][NQ];
    __shared__ unsigned modes[NQ];
    static_assert(!PAIR || 2 * (sizeof(buf) + sizeof(gf) + sizeof(wtab) + sizeof(wtab_p) +
                                sizeof(ca) + sizeof(wv) + sizeof(modes)) <= kLdsPerCu,
                  "two workgroups share a CU");
    const int ntx = (p.nx + MT - 1) / MT;
    const int tile_x0 = (int)(blockIdx.x % ntx) * MT;
    const int tile_y0 = (int)(blockIdx.x / ntx) * MT;
    const int tid = threadIdx.x;

    // region load: node (lx, ly) of the region is global node
    // (tile_x0 - MK + lx, tile_y0 - MK + ly) wrapped; every thread issues all
    // of its loads before the first LDS store, so their latencies overlap
    constexpr int NL = (NREG + NT - 1) / NT;
    auto node_of = [&](int j) {
        const int ly = j / MW, lx = j - (j / MW) * MW;
        return (long long)wrap_region<MT>(tile_y0 - MK + ly, p.ny) * p.nx +
               wrap_region<MT>(tile_x0 - MK + lx, p.nx);
    };
    float4 v[NL];
    float2 fv[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int j = tid + k * NT;
        if (j < NREG) {
            const long long g = node_of(j);
            v[k] = make_float4(src[3 * g], src[3 * g + 1], src[3 * g + 2],
                               MASK ? (float)p.mask[g] : 0.0f);
            if (FORCE == 2) fv[k] = make_float2(p.g_field[g], p.g_field[p.n + g]);
        }
    }
    bool moving = false;
    if (MASK && !QW)
#pragma unroll
        for (int m = 1; m < kMaxWallIds; ++m)
            moving = moving || p.wall_u[m][0] != 0.0f || p.wall_u[m][1] != 0.0f;
    if (MASK && !QW && tid < 9 * kMaxWallIds) {
        const int m = tid / 9;
#pragma unroll
        for (int i = 1; i < 9; ++i)
            if (tid == m * 9 + i) {
                const float uw[3] = {p.wall_term[m][0], p.wall_term[m][1], p.wall_term[m][2]};
                wtab[tid] = vdot<9>(i, uw);
                if (SPLIT) {
                    const float uwp[3] = {p.wall_term_p[m][0], p.wall_term_p[m][1],
                                          p.wall_term_p[m][2]};
                    wtab_p[SPLIT ? tid : 0] = vdot<9>(i, uwp);
                }
            }
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int j = tid + k * NT;
        if (j < NREG) {
            const float u[3] = {v[k].y, v[k].z, 0.0f};
            buf[0][j] = make_float4(v[k].x, u[0], u[1], v[k].w > 0.0f ? v[k].w : node_B(u));
            if (FORCE == 2) gf[FORCE == 2 ? j : 0] = fv[k];
        }
    }
    __syncthreads();
    if constexpr (QW) {
        // distance and wall-motion term of every link of the fluid nodes next
        // to a wall, all of a node's loads in flight together
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int j = tid + k * NT;
            const int ly = j / MW, lx = j - (j / MW) * MW;
            if (j >= NREG || lx < 1 || ly < 1 || lx >= MW - 1 || ly >= MW - 1 || v[k].w > 0.0f)
                continue;
            float m[9];
            bool next = false;
#pragma unroll
            for (int i = 1; i < 9; ++i) {  // the node at x - v_i
                m[i] = buf[0][j - link_cy(i) * MW - link_cx(i)].w;
                next = next || m[i] > 0.0f;
            }
            if (!next) continue;
            const long long g = node_of(j);
            float q[9], u0[9], u1[9];
#pragma unroll
            for (int ib = 1; ib < 9; ++ib) {
                q[ib] = p.qd ? p.qd[(long long)ib * p.n + g] : 0.5f;
                u0[ib] = p.uwl ? p.uwl[((long long)ib * 2) * p.n + g] : 0.0f;
                u1[ib] = p.uwl ? p.uwl[((long long)ib * 2 + 1) * p.n + g] : 0.0f;
            }
            unsigned md = 0u;
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int ib = link_opp(i);
                const float qv = q[ib];
                if (p.qd) {
                    if (!(qv < 0.5f)) md |= 1u << (16 + ib);
                    else if (!(m[ib] > 0.0f)) md |= 1u << ib;  // x + v_i = x - v_ib is fluid
                }
                ca[QW ? ib - 1 : 0][j] = qv < 0.5f ? 2.0f * qv : 0.5f / qv;
                const int id = m[i] > 0.0f ? (int)m[i] : 0;
                float uw[3] = {p.wall_scale * u0[ib], p.wall_scale * u1[ib], 0.0f};
                if (!p.uwl) {
                    uw[0] = p.wall_term[id][0];
                    uw[1] = p.wall_term[id][1];
                }
                wv[QW ? i - 1 : 0][j] = vdot<9>(i, uw);
            }
            modes[j] = md;
        }
        __syncthreads();
    }

    // step s computes the region's rows and columns [s, MW - s), an even
    // number m of them, as m / MR x m work items of MR nodes of one
    // column (a strip), numbered row of strips by row of strips so that a
    // wave's lanes take neighbouring columns; the strip's
    // neighbourhood is read from LDS once and kept in registers
    static_assert(MW % 2 == 0 && MR <= 2, "strips tile every step's square");
    for (int s = 1; s <= ksteps; ++s) {
        const int b0 = (s - 1) & 1, b1 = s & 1;
        const int m = MW - 2 * s;
        const int items = (m / MR) * m;
        // item / m in FP32: (item + 1/2) / m lies at least 1/(2m) from an
        // integer and m <= 46, far above the rounding of the product
        const float inv_m = 1.0f / (float)m;
        for (int it = tid; it < items; it += NT) {
            const int strip = (int)(((float)it + 0.5f) * inv_m);
            const int lx = s + (it - strip * m);
            const int ly0 = s + strip * MR;
            float4 w[MR + 2][3];
#pragma unroll
            for (int rr = 0; rr < MR + 2; ++rr)
#pragma unroll
                for (int cc = 0; cc < 3; ++cc)
                    w[rr][cc] = buf[b0][(ly0 - 1 + rr) * MW + lx - 1 + cc];
            // a strip with no solid node around it takes the update without walls
            bool walls = false;
            if (MASK)
#pragma unroll
                for (int rr = 0; rr < MR + 2; ++rr)
#pragma unroll
                    for (int cc = 0; cc < 3; ++cc) walls = walls || w[rr][cc].w > 0.0f;
            // (a wave with one strip next to a wall takes that update for all:
            // the same results, and only one of the two run)
            if (MASK) walls = __builtin_amdgcn_ballot_w64(walls) != 0ull;
#pragma unroll
            for (int rr = 0; rr < MR; ++rr) {
                const int ly = ly0 + rr;
                const int l = ly * MW + lx;
                const float4 own = w[rr + 1][1];
                // slots: every step's state goes out, tile node by tile node
                const int sgx = tile_x0 - MK + lx, sgy = tile_y0 - MK + ly;
                const bool put = slots && lx >= MK && lx < MK + MT && ly >= MK && ly < MK + MT &&
                                 sgx < p.nx && sgy < p.ny;
                float *const so = put ? slots + (size_t)(s - 1) * slot_floats +
                                            3 * ((size_t)sgy * p.nx + sgx)
                                      : nullptr;
                if (MASK && own.w > 0.0f) {  // solid: unchanged
                    buf[b1][l] = own;
                    if (put) {
                        so[0] = own.x;
                        so[1] = own.y;
                        so[2] = own.z;
                    }
                    continue;
                }
                const float ux[3] = {own.y, own.z, 0.0f};
                auto fnode = [&](int dx, int dy) { return w[rr + 1 + dy][1 + dx]; };
                const MultiSite<FORCE> site{p, gf, l};
                float out[3], e;
                if (MASK && walls) {
                    const MultiWalls<QW, NQ> wl{moving, wtab, wtab_p, ca, wv, modes};
                    wall_update<FORCE != 0, SPLIT, QW, NQ>(p, site, wl, own.x, ux, own.w, fnode,
                                                           out);
                } else {
                    auto fmask = [&](int, int, int) -> uint8_t { return 0; };
                    auto fstate = [&](int dx, int dy, int, float &dr, float (&u)[3], float &B) {
                        const float4 v = fnode(dx, dy);
                        dr = v.x;
                        u[0] = v.y;
                        u[1] = v.z;
                        u[2] = 0.0f;
                        B = v.w;
                    };
                    link_update<9, false, FORCE != 0, SPLIT>(p, site, own.x, ux, own.w, fmask,
                                                             fstate, out, e);
                }
                const float un[3] = {out[1], out[2], 0.0f};
                buf[b1][l] = make_float4(out[0], out[1], out[2], node_B(un));
                if (put) {
                    so[0] = out[0];
                    so[1] = out[1];
                    so[2] = out[2];
                }
            }
        }
        __syncthreads();
    }

    // the tile's nodes after ksteps steps, and their mass and energy
    const int bf = ksteps & 1;
    double acc[2] = {0.0, 0.0};
    for (int j = tid; j < MT * MT; j += NT) {
        const int oy = j / MT, ox = j - (j / MT) * MT;
        const int gx = tile_x0 + ox, gy = tile_y0 + oy;
        if (gx >= p.nx || gy >= p.ny) continue;
        const float4 v = buf[bf][(oy + MK) * MW + (ox + MK)];
        const long long g = (long long)gy * p.nx + gx;
        if (!slots) {  // with slots the last step's state is already out
            dst[3 * g] = v.x;
            dst[3 * g + 1] = v.y;
            dst[3 * g + 2] = v.z;
        }
        if (MASK && v.w > 0.0f) continue;
        float e = 0.0f;
        e = fmaf(v.y, v.y, e);
        e = fmaf(v.z, v.z, e);
        acc[0] += (double)v.x;
        acc[1] += 0.5 * (double)e;
    }
    store_block_partials<2>(acc, r.partials, blockIdx.x);
    if (blockIdx.x == 0 && r.prev_nblocks)
        finish_previous_sums(r.prev_partials, r.prev_nblocks, r.prev_out, r.prev_out2);
}

// Several D2Q9 reverse steps per launch, the same temporal blocking: the
// region's mu (with the mask id) is loaded into LDS once; reverse step s (the
// forward step of slot slot_hi - s + 1 of the caller's state slots) is
// computed on the region less s nodes on each side from the node's own state,
// read from its slot, and the mu of its neighbours y + v_k in LDS.  Each node
// goes through adj_node_update, as in the one-step reverse kernel, so mu is
// bitwise that of ksteps single reverse steps.  Each step's dL/da of the
// tile's nodes is summed per workgroup into slice slice0 + s - 1 of the
// partials (a different order of addition than the one-step kernel's blocks):
// per wave during the step, over the waves after the last step, so a step
// ends with a single barrier.
// final_last: the last step is step 0, its lambda goes out field-major.
template <int MT, bool MASK>
__global__ __launch_bounds__(multi_threads(MT, kAdjRows)) void k_adj_d2q9_multi(
    ProblemArgs p, const float *__restrict__ states, size_t slot_floats, int slot_hi, int ksteps,
    int final_last, const float *__restrict__ mu_in, float *__restrict__ mu_out,
    double *__restrict__ partials, size_t stride, unsigned slice0)
{
    constexpr int MR = kAdjRows;
    constexpr int NT = multi_threads(MT, MR);
    constexpr int MW = MT + 2 * MK;  // region side
    // per node of the region, two steps' buffers: (mu_R, mu_Jx, mu_Jy, mask id)
    __shared__ float4 buf[2][MW * MW];
    // each step's dL/da per wave, added up after the last step
    constexpr int NWAVES = NT / kWave;
    __shared__ double stepsum[MK][NWAVES];
    const int ntx = (p.nx + MT - 1) / MT;
    const int tile_x0 = (int)(blockIdx.x % ntx) * MT;
    const int tile_y0 = (int)(blockIdx.x / ntx) * MT;
    const int tid = threadIdx.x;

    constexpr int NL = (MW * MW + NT - 1) / NT;
    float4 v[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int j = tid + k * NT;
        if (j < MW * MW) {
            const int ly = j / MW, lx = j - (j / MW) * MW;
            const long long g = (long long)wrap_region<MT>(tile_y0 - MK + ly, p.ny) * p.nx +
                                wrap_region<MT>(tile_x0 - MK + lx, p.nx);
            v[k] = make_float4(mu_in[3 * g], mu_in[3 * g + 1], mu_in[3 * g + 2],
                               MASK ? (float)p.mask[g] : 0.0f);
        }
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int j = tid + k * NT;
        if (j < MW * MW) buf[0][j] = v[k];
    }
    __syncthreads();

    static_assert(MW % 2 == 0 && MR <= 2, "strips tile every step's square");
    // the thread's first strip of step s: its states, loaded a step ahead so
    // that they arrive while the step before is computed
    float pre[MR][3];
    auto strip_of = [&](int it, int s, int &lx, int &ly0) {
        const int m = MW - 2 * s;
        const int strip = (int)(((float)it + 0.5f) * (1.0f / (float)m));
        lx = s + (it - strip * m);
        ly0 = s + strip * MR;
    };
    auto load_states = [&](int s, int lx, int ly0, float (&o)[MR][3]) {
        const float *st = states + (size_t)(slot_hi - s + 1) * slot_floats;
#pragma unroll
        for (int rr = 0; rr < MR; ++rr) {
            const long long g =
                (long long)wrap_region<MT>(tile_y0 - MK + ly0 + rr, p.ny) * p.nx +
                wrap_region<MT>(tile_x0 - MK + lx, p.nx);
            o[rr][0] = st[3 * g];
            o[rr][1] = st[3 * g + 1];
            o[rr][2] = st[3 * g + 2];
        }
    };
    auto prefetch = [&](int s) {
        const int m = MW - 2 * s;
        if (s > ksteps || tid >= (m / MR) * m) return;
        int lx, ly0;
        strip_of(tid, s, lx, ly0);
        load_states(s, lx, ly0, pre);
    };
    prefetch(1);
    for (int s = 1; s <= ksteps; ++s) {
        const int b0 = (s - 1) & 1, b1 = s & 1;
        const bool fin = final_last && s == ksteps;
        const int m = MW - 2 * s;
        const int items = (m / MR) * m;
        double da_sum = 0.0;
        for (int it = tid; it < items; it += NT) {
            int lx, ly0;
            strip_of(it, s, lx, ly0);
            float sv[MR][3];
#pragma unroll
            for (int rr = 0; rr < MR; ++rr)
#pragma unroll
                for (int c = 0; c < 3; ++c) sv[rr][c] = pre[rr][c];
            if (it == tid) prefetch(s + 1);
            else load_states(s, lx, ly0, sv);
            float4 w[MR + 2][3];
#pragma unroll
            for (int rr = 0; rr < MR + 2; ++rr)
#pragma unroll
                for (int cc = 0; cc < 3; ++cc)
                    w[rr][cc] = buf[b0][(ly0 - 1 + rr) * MW + lx - 1 + cc];
#pragma unroll
            for (int rr = 0; rr < MR; ++rr) {
                const int ly = ly0 + rr;
                const int l = ly * MW + lx;
                const float4 own = w[rr + 1][1];
                const int gx = tile_x0 - MK + lx, gy = tile_y0 - MK + ly;
                const bool tile = lx >= MK && lx < MK + MT && ly >= MK && ly < MK + MT &&
                                  gx < p.nx && gy < p.ny;
                const long long g = (long long)wrap_region<MT>(gy, p.ny) * p.nx + wrap_region<MT>(gx, p.nx);
                if (MASK && own.w != 0.0f) {  // solid: mu (or lambda) zero
                    if (fin) {
                        if (tile) mu_out[g] = mu_out[p.n + g] = mu_out[2 * p.n + g] = 0.0f;
                    } else {
                        buf[b1][l] = make_float4(0.0f, 0.0f, 0.0f, own.w);
                    }
                    continue;
                }
                const float uy[3] = {sv[rr][1], sv[rr][2], 0.0f};
                const float dry = sv[rr][0];
                const float muJ[3] = {own.y, own.z, 0.0f};
                auto fmask = [&](int dx, int dy, int) -> uint8_t {
                    return MASK ? (uint8_t)w[rr + 1 + dy][1 + dx].w : (uint8_t)0;
                };
                auto fm = [&](int k) {
                    const float4 q = w[rr + 1 + link_cy(k)][1 + link_cx(k)];
                    const float mt[3] = {q.y, q.z, 0.0f};
                    return q.x + vdot<9>(k, mt);
                };
                float lr, lu[3], da;
                adj_node_update<9, MASK>(p, dry, uy, own.x, muJ, fmask, fm, lr, lu, da);
                if (tile) da_sum += (double)da;
                if (fin) {
                    if (tile) {
                        mu_out[g] = lr;
                        mu_out[p.n + g] = lu[0];
                        mu_out[2 * p.n + g] = lu[1];
                    }
                } else {
                    float mR, mJ[3];
                    adj_fold<2>(dry, uy, lr, lu, mR, mJ);
                    buf[b1][l] = make_float4(mR, mJ[0], mJ[1], own.w);
                }
            }
        }
        // the wave's sum now; the sum over the waves, in wave order (the
        // order of block_sum), after the last step, one thread per step
        const double wsum = wave_sum(da_sum);
        if ((tid & (kWave - 1)) == 0) stepsum[s - 1][tid / kWave] = wsum;
        __syncthreads();  // ends the step
    }
    if (tid < ksteps) {
        double sum = 0.0;
        for (int w = 0; w < NWAVES; ++w) sum += stepsum[tid][w];
        partials[(size_t)(slice0 + tid) * stride + blockIdx.x] = sum;
    }

    if (!final_last) {
        const int bf = ksteps & 1;
        for (int j = tid; j < MT * MT; j += NT) {
            const int oy = j / MT, ox = j - (j / MT) * MT;
            const int gx = tile_x0 + ox, gy = tile_y0 + oy;
            if (gx >= p.nx || gy >= p.ny) continue;
            const float4 q = buf[bf][(oy + MK) * MW + (ox + MK)];
            const long long g = (long long)gy * p.nx + gx;
            mu_out[3 * g] = q.x;
            mu_out[3 * g + 1] = q.y;
            mu_out[3 * g + 2] = q.z;
        }
    }
}

}  // namespace

// What a launch of either kernel takes; one pair of launchers per tile size.
struct MultiFwd {
    const float *src;
    float *dst;
    int ksteps;
    float *slots;
    size_t slot_floats;
};
struct MultiAdj {
    const float *states;
    size_t slot_floats;
    int slot_hi, ksteps, final_last;
    const float *mu_in;
    float *mu_out;
    double *partials;
    size_t stride;
    unsigned slice0;
};
template <int MT>
void launch_fwd_multi_tile(const ProblemArgs &p, unsigned nb, const MultiFwd &f,
                           const ReduceArgs &r, hipStream_t s);
template <int MT>
void launch_adj_multi_tile(const ProblemArgs &p, unsigned nb, const MultiAdj &a, hipStream_t s);

namespace {

template <int MT, bool MASK, int FORCE, bool SPLIT, bool QW>
void fwd_multi(const ProblemArgs &p, unsigned nb, const MultiFwd &f, const ReduceArgs &r,
               hipStream_t s)
{
    constexpr int nt = multi_threads(MT, fwd_rows(MT, MASK));
    if constexpr (fwd_pair(MT, MASK, FORCE, SPLIT))
        if (p.multi_many) {
            k_fwd_d2q9_multi<MT, MASK, FORCE, SPLIT, QW, true><<<nb, nt / 2, 0, s>>>(
                p, f.src, f.dst, f.ksteps, r, f.slots, f.slot_floats);
            return;
        }
    k_fwd_d2q9_multi<MT, MASK, FORCE, SPLIT, QW, false><<<nb, nt, 0, s>>>(
        p, f.src, f.dst, f.ksteps, r, f.slots, f.slot_floats);
}

template <int MT, bool MASK, int FORCE>
void fwd_multi_force(const ProblemArgs &p, unsigned nb, const MultiFwd &f, const ReduceArgs &r,
                     hipStream_t s)
{
    if constexpr (MASK && MT <= 16) {
        if (p.qd || p.uwl) {
            fwd_multi<MT, MASK, FORCE, false, true>(p, nb, f, r, s);
            return;
        }
    }
    if (p.split) fwd_multi<MT, MASK, FORCE, true, false>(p, nb, f, r, s);
    else fwd_multi<MT, MASK, FORCE, false, false>(p, nb, f, r, s);
}

template <int MT, bool MASK>
void fwd_multi_mask(const ProblemArgs &p, unsigned nb, const MultiFwd &f, const ReduceArgs &r,
                    hipStream_t s)
{
    if (p.g_field) fwd_multi_force<MT, MASK, 2>(p, nb, f, r, s);
    else if (p.has_force) fwd_multi_force<MT, MASK, 1>(p, nb, f, r, s);
    else fwd_multi_force<MT, MASK, 0>(p, nb, f, r, s);
}

// instantiated once per tile size
template <int MT>
void fwd_multi_tile(const ProblemArgs &p, unsigned nb, const MultiFwd &f, const ReduceArgs &r,
                    hipStream_t s)
{
    if (p.mask) fwd_multi_mask<MT, true>(p, nb, f, r, s);
    else fwd_multi_mask<MT, false>(p, nb, f, r, s);
}

template <int MT>
void adj_multi_tile(const ProblemArgs &p, unsigned nb, const MultiAdj &a, hipStream_t s)
{
    constexpr int nt = multi_threads(MT, kAdjRows);
    if (p.mask)
        k_adj_d2q9_multi<MT, true><<<nb, nt, 0, s>>>(p, a.states, a.slot_floats, a.slot_hi,
                                                     a.ksteps, a.final_last, a.mu_in, a.mu_out,
                                                     a.partials, a.stride, a.slice0);
    else
        k_adj_d2q9_multi<MT, false><<<nb, nt, 0, s>>>(p, a.states, a.slot_floats, a.slot_hi,
                                                      a.ksteps, a.final_last, a.mu_in, a.mu_out,
                                                      a.partials, a.stride, a.slice0);
}

}  // namespace

}  // namespace lwacm
