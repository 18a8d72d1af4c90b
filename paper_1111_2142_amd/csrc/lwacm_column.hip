// lwacm_column.hip -- D3Q19 steps on grids the tile kernels do not take, as
// column-marching gathers.
//
// Every thread owns one (x, y) column and walks up a chunk of planes.  For
// each plane it loads the nodes of its own and the eight columns around it (nine
// 16-byte or 8-byte loads, one plane ahead), forms the link terms they send to
// its own column (five columns send to three planes each, the four diagonal ones
// to one) and keeps them in registers until their target plane is complete.  A
// node's state is thus read nine times through the vector caches instead of
// nineteen, with one address per column for the whole chunk, no LDS and no
// barriers, on grids of any sides: the consecutive threads of a wave take
// consecutive columns across row ends.
//
// The terms and their sums are the operations of link_update and
// adj_node_update (lwacm_generic_update.hpp) in the same order, so fields,
// stored FP16 bits and mu are bitwise those of the one-thread-per-node kernels.
//
// Walls: the column part leaves out the fluid nodes next to a wall (class 1 of
// launch_classify) and writes solid nodes through.  The nodes next to a wall
// run link_update itself, one thread per node of the wall list, in the first
// workgroups of the same launch: all of a node's neighbours, masks and link
// distances are loaded before the first is used, so a node costs one memory
// latency instead of one per link.
//
// The classes and the list are those of lwacm_init, but the mask is the
// caller's, who may edit it between calls: launch_mask_check compares the two at
// the start of a call, and once they differ every node goes through link_update
// with the mask as it is.
#include "lwacm_device.hpp"
#include "lwacm_generic_update.hpp"
#include "lwacm_internal.hpp"
#include "lwacm_march_common.hpp"

namespace lwacm {

namespace {

constexpr int NT = 256;  // threads per workgroup

// Column offsets (dx, dy) in load order: own, the four axis neighbours, the
// four diagonal ones.
constexpr int kDx[9] = {0, 1, -1, 0, 0, 1, -1, 1, -1};
constexpr int kDy[9] = {0, 0, 0, 1, -1, 1, -1, -1, 1};

// Block b of nb in an order that gives each XCD (blocks go to the eight of them
// in turn) one run of neighbouring blocks.
__device__ __forceinline__ unsigned xcd_order(unsigned b, unsigned nb)
{
    const unsigned k = b % 8u, q = nb / 8u, rem = nb % 8u;
    return k * q + min(k, rem) + b / 8u;
}

struct ColumnIdx {
    unsigned col[9];  // element offset in a plane of the nine columns
    bool active;      // false: past the last column (clamped)
    int z0, z1;       // planes of the chunk
};

__device__ __forceinline__ ColumnIdx column_of(const ProblemArgs &p, int nzc, unsigned block,
                                               unsigned nblocks)
{
    const unsigned plane = (unsigned)(p.nx * p.ny);
    const unsigned ncg = (plane + NT - 1) / NT;
    const unsigned lb = xcd_order(block, nblocks);
    const unsigned zc = lb / ncg;
    unsigned c = (lb - zc * ncg) * NT + threadIdx.x;
    ColumnIdx ci;
    ci.active = c < plane;
    c = min(c, plane - 1);
    const int y = (int)(c / (unsigned)p.nx), x = (int)(c - (unsigned)y * (unsigned)p.nx);
#pragma unroll
    for (int k = 0; k < 9; ++k)
        ci.col[k] = (unsigned)(wrap_index(y + kDy[k], p.ny) * p.nx + wrap_index(x + kDx[k], p.nx));
    ci.z0 = (int)zc * nzc;
    ci.z1 = min(ci.z0 + nzc, p.nz);
    return ci;
}

// The link whose upstream node lies in column k, dz planes up (dz = -1, 0, 1):
// v = (-dx, -dy, -dz).
constexpr int link_from(int k, int dz) { return link_index(-kDx[k], -kDy[k], -dz); }
// the link towards column k, dz planes up
constexpr int link_to(int k, int dz) { return link_index(kDx[k], kDy[k], dz); }

// One upstream node's part of a link term (Eq. ACM2.0b): without a force the
// whole term; with one, its factor c (A + 9/2 c) + B, whose product with rho
// meets the target's forcing in the addend.
template <int FORCE>
__device__ __forceinline__ float upstream_term(float dr, float rho, float c, float B, float A)
{
    if (!FORCE) return link_term_unweighted(dr, rho, c, B, A);
    float t = fmaf(4.5f, c, A);
    return fmaf(c, t, B);
}

// Sums over the complete link terms of a node (s in link order), as
// link_update forms them.
__device__ __forceinline__ void sum_links(const float (&term)[19], float &D36, float (&J36)[3])
{
    using L = Lattice<19>;
    bool dset = false, jset[3] = {false, false, false};
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        float s = term[i];
        s *= L::w36(i);
        accum(D36, dset, s);
        if (link_cx(i) != 0) accum(J36[0], jset[0], link_cx(i) > 0 ? s : -s);
        if (link_cy(i) != 0) accum(J36[1], jset[1], link_cy(i) > 0 ? s : -s);
        if (link_cz(i) != 0) accum(J36[2], jset[2], link_cz(i) > 0 ? s : -s);
    }
}

// ------------------------------------------------------ nodes next to walls
struct WallList {
    const unsigned *list;  // fluid nodes next to a wall
    unsigned n, blocks;    // entries, and workgroups that take them
    const unsigned *edited;  // not zero: the mask is no longer the list's
};

// Solid or fluid in the mask where the classes say otherwise?  Bound by the
// launch: 3.5 us a call (not a step) at 33x17x8 and at 150x84x75.  A step asks the
// flag: 8.2 -> 8.4 us at 33x17x8; at 150x84x75 15.2 -> 15.5, with a force 16.2 as
// before, with a field 19.5 -> 20.1 (two registers more are spilled).
__global__ __launch_bounds__(NT) void k_mask_check(const uint8_t *__restrict__ mask,
                                                   const uint8_t *__restrict__ cls, unsigned n,
                                                   unsigned *edited)
{
    const unsigned first = blockIdx.x * NT + threadIdx.x, threads = gridDim.x * NT;
    unsigned diff = 0u;
    const unsigned body = ((uintptr_t)mask & 15u) ? 0u : n / 16u;  // 16 bytes at a time
    const uint4 *m4 = reinterpret_cast<const uint4 *>(mask);
    const uint4 *c4 = reinterpret_cast<const uint4 *>(cls);
    for (unsigned i = first; i < body; i += threads) {
        const uint4 m = m4[i], c = c4[i];
        const unsigned mw[4] = {m.x, m.y, m.z, m.w}, cw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // bit 7 of each byte: mask not zero, class 2 (the classes are 0 to 2)
            const unsigned solid = ((mw[k] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | mw[k];
            diff |= (solid ^ (cw[k] << 6)) & 0x80808080u;
        }
    }
    for (unsigned i = 16u * body + first; i < n; i += threads)
        diff |= (mask[i] != 0) != (cls[i] == 2) ? 1u : 0u;
    if (diff) *edited = 1u;
}

// Site of a listed node: distances loaded ahead, the wall table in LDS.
struct ListSite {
    GlobalSite<19> g_;
    const float (*table)[3];  // wall_term by id, or null: every wall at rest
    const float (&qv)[19];
    __device__ __forceinline__ float g(int k) const { return g_.g(k); }
    __device__ __forceinline__ float wall(int i, int ib, uint8_t m) const
    {
        if (g_.p.uwl) return g_.wall(i, ib, m);
        if (!table) return 0.0f;
        const float uw[3] = {table[m][0], table[m][1], table[m][2]};
        return vdot<19>(i, uw);
    }
    __device__ __forceinline__ float wall_p(int, uint8_t) const { return 0.0f; }
    __device__ __forceinline__ bool has_q() const { return g_.p.qd != nullptr; }
    __device__ __forceinline__ float q(int ib) const { return qv[ib]; }
};

// The wall-motion terms by mask id into LDS; false: every wall at rest.
__device__ __forceinline__ bool load_wall_table(const ProblemArgs &p, float (&table)[kMaxWallIds][3])
{
    bool moving = false;
#pragma unroll
    for (int m = 1; m < kMaxWallIds; ++m)
        moving = moving || p.wall_u[m][0] != 0.0f || p.wall_u[m][1] != 0.0f ||
                 p.wall_u[m][2] != 0.0f;
    if (threadIdx.x < 3 * kMaxWallIds)
        table[threadIdx.x / 3][threadIdx.x % 3] = p.wall_term[threadIdx.x / 3][threadIdx.x % 3];
    __syncthreads();
    return moving;
}

// Fluid node idx by link_update; out: its new state, e: |u|^2.  SOLID: the node
// may be solid (then false, nothing done).
template <class T, bool FORCE, bool SOLID>
__device__ __forceinline__ bool gather_node(const ProblemArgs &p, const float (*table)[3],
                                            const T *src, unsigned idx, float (&out)[4], float &e)
{
    const unsigned t = idx / (unsigned)p.nx;
    const int x = (int)(idx - t * (unsigned)p.nx);
    const int z = (int)(t / (unsigned)p.ny), y = (int)(t - (unsigned)z * (unsigned)p.ny);
    float st[19][4];
    uint8_t mk[19];
    float q[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) {  // the node at x + v_i
        const unsigned at =
            ((unsigned)wrap_index(z + link_cz(i), p.nz) * (unsigned)p.ny +
             (unsigned)wrap_index(y + link_cy(i), p.ny)) * (unsigned)p.nx +
            (unsigned)wrap_index(x + link_cx(i), p.nx);
        NodeState<T, 4>::load(src, at, p.ld_scale, st[i]);
        mk[i] = i || SOLID ? p.mask[at] : (uint8_t)0;
    }
    if (SOLID && mk[0]) return false;
#pragma unroll
    for (int i = 0; i < 19; ++i)
        q[i] = (p.qd && mk[i]) ? p.qd[(long long)i * p.n + idx] : 0.5f;
    const float ux[3] = {st[0][1], st[0][2], st[0][3]};
    auto fmask = [&](int dx, int dy, int dz) -> uint8_t { return mk[link_index(dx, dy, dz)]; };
    auto fstate = [&](int dx, int dy, int dz, float &dr, float (&u)[3], float &B) {
        const float(&v)[4] = st[link_index(dx, dy, dz)];
        dr = v[0];
        u[0] = v[1];
        u[1] = v[2];
        u[2] = v[3];
        B = node_B(u);
    };
    const ListSite site{{p, (long long)idx}, table, q};
    link_update<19, true, FORCE, false>(p, site, st[0][0], ux, node_B(ux), fmask, fstate, out, e);
    return true;
}

template <class T, bool SR>
__device__ __forceinline__ void store_gathered(const ProblemArgs &p, T *dst, unsigned idx,
                                               const float (&out)[4], float e, double (&acc)[2])
{
    if (SR)
        NodeState<T, 4>::store_sr(dst, idx, out, p.st_scale, sr_words(idx, p.sr_word));
    else
        NodeState<T, 4>::store(dst, idx, out, p.st_scale);
    acc[0] += (double)out[0];
    acc[1] += 0.5 * (double)e;
}

// ------------------------------------------------------------ forward step
// FORCE: 0 none, 1 uniform, 2 field (loaded with the planes); SR: FP16 storage
// with stochastic rounding.  Both are template parameters so that the plane
// loop has no branches: with one around the rounding the loads no longer
// overlapped the planes' arithmetic and a step took twice as long.
// Three waves a SIMD (168 VGPRs): with walls and a force it took 170 and ran two
// (150x84x75, sphere in a duct with distances and a uniform force 18.7 us a
// step, then 15.8; force field 19.8, then 18.7; 16.1 and 19.0 with the branch for
// an edited mask, whose instances spill 2 to 9 VGPRs).  Not for the force field
// without walls, which would spill eight VGPRs in the plane loop (14.5, held to
// 168 16.7; 250^3 176, 209), nor the reverse step (19.7, held 22.1).
constexpr int fwd_waves(bool MASK, int FORCE) { return MASK || FORCE < 2 ? 3 : 2; }
template <class T, bool SR, bool MASK, int FORCE>
__global__ __launch_bounds__((NT), (fwd_waves(MASK, FORCE))) void k_fwd_column(ProblemArgs p, int nzc, WallList wl,
                                                   const uint8_t *__restrict__ cls,
                                                   const T *__restrict__ src, T *__restrict__ dst,
                                                   ReduceArgs r)
{
    double acc[2] = {0.0, 0.0};
    const unsigned first = MASK ? wl.blocks : 0u;
    const unsigned plane = (unsigned)(p.nx * p.ny);
    const unsigned edited = MASK ? *wl.edited : 0u;
    if (MASK && blockIdx.x < first) {
        // the listed nodes, unless the mask is no longer the list's (asked last:
        // the answer arrives beside the nodes' own loads)
        __shared__ float table[kMaxWallIds][3];
        const bool moving = load_wall_table(p, table);
        const unsigned k = blockIdx.x * NT + threadIdx.x;
        if (k < wl.n) {
            const unsigned idx = wl.list[k];
            float out[4], e;
            gather_node<T, FORCE != 0, false>(p, moving ? table : nullptr, src, idx, out, e);
            if (!edited) store_gathered<T, SR>(p, dst, idx, out, e, acc);
        }
    } else {
        const ColumnIdx ci = column_of(p, nzc, blockIdx.x - first, gridDim.x - first);
        constexpr unsigned NB = BufIO<T>::kNodeBytes;
        const Rsrc rs = make_rsrc(src, (unsigned long long)p.n * NB);
        const Rsrc rd = make_rsrc(dst, (unsigned long long)p.n * NB);
        const Rsrc rc = make_rsrc(MASK ? cls : nullptr, MASK ? (unsigned long long)p.n : 0ull);
        struct Plane {
            typename BufIO<T>::Raw v[9];
            unsigned cls;
            float g[3];
        };
        // node-by-node acceleration: three FP32 fields, one resource each
        const unsigned long long gbytes = FORCE == 2 ? (unsigned long long)p.n * 4u : 0ull;
        const Rsrc rg[3] = {make_rsrc(FORCE == 2 ? p.g_field : nullptr, gbytes),
                            make_rsrc(FORCE == 2 ? p.g_field + p.n : nullptr, gbytes),
                            make_rsrc(FORCE == 2 ? p.g_field + 2 * p.n : nullptr, gbytes)};
        auto load = [&](Plane &b, int pz) {
            const unsigned pw = (unsigned)wrap_index(min(pz, ci.z1), p.nz);
#pragma unroll
            for (int k = 0; k < 9; ++k) b.v[k] = BufIO<T>::load(rs, ci.col[k] * NB, pw * plane * NB);
            if (MASK) b.cls = __builtin_amdgcn_raw_buffer_load_b8(rc, ci.col[0], pw * plane, 0);
            if (FORCE == 2)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    b.g[c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                           rg[c], ci.col[0] * 4u, pw * plane * 4u, 0));
        };
        // terms in flight, by link: from the plane below the target (two
        // generations), and of the target's own plane; with a force, the
        // upstream rho - 1 beside them
        float below0[5], below1[5], same[9], dbelow0[5], dbelow1[5], dsame[9];
#pragma unroll
        for (int k = 0; k < 5; ++k) below0[k] = below1[k] = dbelow0[k] = dbelow1[k] = 0.0f;
#pragma unroll
        for (int k = 0; k < 9; ++k) same[k] = dsame[k] = 0.0f;
        typename BufIO<T>::Raw own_raw = {};
        float own[4] = {0.0f, 0.0f, 0.0f, 0.0f}, ownB = 0.0f;  // of the target plane
        float own_g[3] = {0.0f, 0.0f, 0.0f};
        unsigned own_cls = 0u;
        auto process = [&](const Plane &b, int pz) {
            float dr[9], u[9][3], B[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                dr[k] = BufIO<T>::value(b.v[k], 0, p.ld_scale[0]);
#pragma unroll
                for (int c = 0; c < 3; ++c) u[k][c] = BufIO<T>::value(b.v[k], c + 1, p.ld_scale[1]);
                B[k] = node_B(u[k]);
            }
            // the target plane tz = pz - 1 is complete with the terms from above
            const int tz = pz - 1;
            const unsigned node = (unsigned)tz * plane + ci.col[0];
            const float rx = 1.0f + own[0];
            const float ux[3] = {own[1], own[2], own[3]};
            float g3[3] = {0.0f, 0.0f, 0.0f};
            const bool in = tz >= ci.z0 && tz < ci.z1 && ci.active;
            if (FORCE)
#pragma unroll
                for (int k = 0; k < 3; ++k) g3[k] = 3.0f * rx * (FORCE == 2 ? own_g[k] : p.g[k]);
            float s[19];
            auto put = [&](int i, float t, float d) {
                s[i] = FORCE ? fmaf(1.0f + d, t, d + vdot<19>(i, g3)) : t;
            };
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                put(link_from(k, 1), upstream_term<FORCE>(dr[k], 1.0f + dr[k],
                                                          vdot<19>(link_from(k, 1), u[k]), B[k], p.A),
                    dr[k]);
                put(link_from(k, -1), below0[k], dbelow0[k]);
            }
#pragma unroll
            for (int k = 1; k < 9; ++k) put(link_from(k, 0), same[k], dsame[k]);
            // the rest link
            s[0] = fmaf(rx, ownB, FORCE ? own[0] + vdot<19>(0, g3) : own[0]);
            float D36 = 0.0f, J36[3] = {0.0f, 0.0f, 0.0f}, out[4], e;
            sum_links(s, D36, J36);
            finish_node<3>(p, rx, ux, D36, J36, out, e);
            const bool solid = MASK && own_cls == 2u;
            typename BufIO<T>::Raw o;
            if (SR)
                o = BufIO<T>::pack_sr(out[0], out[1], out[2], out[3], p.st_scale,
                                      sr_words(node, p.sr_word));
            else
                o = BufIO<T>::pack(out[0], out[1], out[2], out[3], p.st_scale);
            if (solid) o = own_raw;
            // planes outside the chunk and nodes next to a wall: past the end of
            // the buffer, where the hardware drops the store
            BufIO<T>::store_raw(rd, in && !(MASK && own_cls == 1u) ? node * NB : 0xfffffff0u, 0u, o);
            const bool count = in && (!MASK || own_cls == 0u);
            acc[0] += count ? (double)out[0] : 0.0;
            acc[1] += count ? 0.5 * (double)e : 0.0;
            // this plane's terms for its own plane and the one above
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                below0[k] = below1[k];
                below1[k] = upstream_term<FORCE>(dr[k], 1.0f + dr[k],
                                                 vdot<19>(link_from(k, -1), u[k]), B[k], p.A);
                if (FORCE) {
                    dbelow0[k] = dbelow1[k];
                    dbelow1[k] = dr[k];
                }
            }
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                same[k] = upstream_term<FORCE>(dr[k], 1.0f + dr[k],
                                               vdot<19>(link_from(k, 0), u[k]), B[k], p.A);
                if (FORCE) dsame[k] = dr[k];
            }
            own[0] = dr[0];
#pragma unroll
            for (int c = 0; c < 3; ++c) own[c + 1] = u[0][c];
            ownB = B[0];
            if (MASK) {
                own_raw = b.v[0];
                own_cls = b.cls;
            }
            if (FORCE == 2)
#pragma unroll
                for (int c = 0; c < 3; ++c) own_g[c] = b.g[c];
        };
        Plane a, b;
        load(a, ci.z0 - 1);
        const int n = ci.z1 - ci.z0 + 2;  // planes z0 - 1 .. z1
        // two planes per iteration, each loaded while the other is computed (an
        // odd last one repeats plane z1 and stores nothing)
#pragma unroll 1
        for (int k = 0; k < n; k += 2) {
            load(b, ci.z0 + k);
            __builtin_amdgcn_sched_barrier(0);
            process(a, ci.z0 - 1 + k);
            load(a, ci.z0 + k + 1);
            __builtin_amdgcn_sched_barrier(0);
            process(b, ci.z0 + k);
        }
        if (MASK && __builtin_amdgcn_readfirstlane(edited) != 0u) {
            // every node of the columns again, by the mask as it is and by the
            // thread that stored it above (asked for last: before the planes the
            // flag's latency cost a step 0.3 us)
            __shared__ float table[kMaxWallIds][3];
            const bool moving = load_wall_table(p, table);
            acc[0] = acc[1] = 0.0;
#pragma unroll 1
            for (int z = ci.z0; z < ci.z1 && ci.active; ++z) {
                const unsigned idx = (unsigned)z * plane + ci.col[0];
                float out[4], e;
                if (gather_node<T, FORCE != 0, true>(p, moving ? table : nullptr, src, idx, out,
                                                     e)) {
                    store_gathered<T, SR>(p, dst, idx, out, e, acc);
                } else {  // solid: written through
                    using Raw = typename BufIO<T>::Raw;
                    reinterpret_cast<Raw *>(dst)[idx] = reinterpret_cast<const Raw *>(src)[idx];
                }
            }
        }
    }
    store_block_partials<2>(acc, r.partials, blockIdx.x);
    if (blockIdx.x == 0 && r.prev_nblocks)
        finish_previous_sums(r.prev_partials, r.prev_nblocks, r.prev_out, r.prev_out2);
}

// ------------------------------------------------------------ reverse step
template <class T, bool FINAL>
__global__ __launch_bounds__(NT) void k_adj_column(ProblemArgs p, int nzc,
                                                   const T *__restrict__ state,
                                                   const float *__restrict__ mu_in,
                                                   float *__restrict__ mu_out, ReduceArgs r)
{
    double acc[1] = {0.0};
    const ColumnIdx ci = column_of(p, nzc, blockIdx.x, gridDim.x);
    const unsigned plane = (unsigned)(p.nx * p.ny);
    constexpr unsigned NB = BufIO<T>::kNodeBytes;
    const Rsrc rm = make_rsrc(mu_in, (unsigned long long)p.n * 16u);
    const Rsrc rst = make_rsrc(state, (unsigned long long)p.n * NB);
    const Rsrc rout = make_rsrc(mu_out, (unsigned long long)p.n * 16u);
    struct Plane {
        f32x4 v[9];
        typename BufIO<T>::Raw st;
    };
    auto load = [&](Plane &b, int pz) {
        const unsigned pw = (unsigned)wrap_index(min(pz, ci.z1), p.nz);
#pragma unroll
        for (int k = 0; k < 9; ++k) b.v[k] = BufIO<float>::load(rm, ci.col[k] * 16u, pw * plane * 16u);
        b.st = BufIO<T>::load(rst, ci.col[0] * NB, pw * plane * NB);
    };
    // link cotangents m_k of planes not yet complete: towards the plane below
    // the node that holds them (two generations) and its own
    float below0[5], below1[5], same[9];
#pragma unroll
    for (int k = 0; k < 5; ++k) below0[k] = below1[k] = 0.0f;
#pragma unroll
    for (int k = 0; k < 9; ++k) same[k] = 0.0f;
    float own[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // mu and state of the target plane
    typename BufIO<T>::Raw own_st = {};
    auto process = [&](const Plane &b, int pz) {
        float mr[9], mt[9][3];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            mr[k] = b.v[k].x;
            mt[k][0] = b.v[k].y;
            mt[k][1] = b.v[k].z;
            mt[k][2] = b.v[k].w;
        }
        auto cot = [&](int k, int dz) {  // m of the link towards column k, dz planes up
            return mr[k] + vdot<19>(link_to(k, dz), mt[k]);
        };
        const int tz = pz - 1;
        const unsigned node = (unsigned)tz * plane + ci.col[0];
        float m[19];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            m[link_to(k, 1)] = cot(k, 1);
            m[link_to(k, -1)] = below0[k];
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) m[link_to(k, 0)] = same[k];
        const float dry = BufIO<T>::value(own_st, 0, p.ld_scale[0]);
        const float uy[3] = {BufIO<T>::value(own_st, 1, p.ld_scale[1]),
                             BufIO<T>::value(own_st, 2, p.ld_scale[1]),
                             BufIO<T>::value(own_st, 3, p.ld_scale[1])};
        const float muJ[3] = {own[1], own[2], own[3]};
        float lr, lu[3], da;
        adj_node_update<19, false>(
            p, dry, uy, own[0], muJ, [](int, int, int) -> uint8_t { return 0; },
            [&](int k) { return m[k]; }, lr, lu, da);
        const bool in = tz >= ci.z0 && tz < ci.z1 && ci.active;
        if (FINAL) {
            const unsigned off = node * 4u, fs = (unsigned)(p.n * 4);
            const f32x4 l = {lr, lu[0], lu[1], lu[2]};
            const u32x4 lb = __builtin_bit_cast(u32x4, l);
            __builtin_amdgcn_raw_buffer_store_b32(lb.x, rout, in ? off : 0xfffffff0u, 0, 0);
            store_data_guard();
            __builtin_amdgcn_raw_buffer_store_b32(lb.y, rout, in ? off + fs : 0xfffffff0u, 0, 0);
            store_data_guard();
            __builtin_amdgcn_raw_buffer_store_b32(lb.z, rout, in ? off + 2 * fs : 0xfffffff0u, 0, 0);
            store_data_guard();
            __builtin_amdgcn_raw_buffer_store_b32(lb.w, rout, in ? off + 3 * fs : 0xfffffff0u, 0, 0);
            store_data_guard();
        } else {
            float mR, mJ[3];
            adj_fold<3>(dry, uy, lr, lu, mR, mJ);
            BufIO<float>::store_raw(rout, in ? node * 16u : 0xfffffff0u, 0u,
                                    f32x4{mR, mJ[0], mJ[1], mJ[2]});
        }
        acc[0] += in ? (double)da : 0.0;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            below0[k] = below1[k];
            below1[k] = cot(k, -1);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) same[k] = cot(k, 0);
        own[0] = mr[0];
#pragma unroll
        for (int c = 0; c < 3; ++c) own[c + 1] = mt[0][c];
        own_st = b.st;
    };
    Plane a, b;
    load(a, ci.z0 - 1);
    const int n = ci.z1 - ci.z0 + 2;  // planes z0 - 1 .. z1
#pragma unroll 1
    for (int k = 0; k < n; k += 2) {
        load(b, ci.z0 + k);
        __builtin_amdgcn_sched_barrier(0);
        process(a, ci.z0 - 1 + k);
        load(a, ci.z0 + k + 1);
        __builtin_amdgcn_sched_barrier(0);
        process(b, ci.z0 + k);
    }
    store_block_partials<1>(acc, r.partials, blockIdx.x);
}

unsigned wall_blocks(unsigned nlist) { return (nlist + NT - 1) / NT; }

unsigned column_blocks(const ProblemArgs &p, int nzc)
{
    const unsigned ncg = ((unsigned)(p.nx * p.ny) + NT - 1) / NT;
    return ncg * (unsigned)((p.nz + nzc - 1) / nzc);
}

template <class T, bool SR, bool MASK>
void fwd_force(const ProblemArgs &p, const T *src, T *dst, const uint8_t *cls, const WallList &wl,
               const ReduceArgs &r, hipStream_t s)
{
    const int c = p.col_nzc;
    const unsigned nb = column_blocks(p, c) + wl.blocks;
    if (p.g_field) k_fwd_column<T, SR, MASK, 2><<<nb, NT, 0, s>>>(p, c, wl, cls, src, dst, r);
    else if (p.has_force) k_fwd_column<T, SR, MASK, 1><<<nb, NT, 0, s>>>(p, c, wl, cls, src, dst, r);
    else k_fwd_column<T, SR, MASK, 0><<<nb, NT, 0, s>>>(p, c, wl, cls, src, dst, r);
}

template <class T, bool SR>
hipError_t fwd(const ProblemArgs &p, const void *src, void *dst, const uint8_t *cls,
               const WallList &wl, const ReduceArgs &r, hipStream_t s)
{
    const T *a = static_cast<const T *>(src);
    T *b = static_cast<T *>(dst);
    if (p.mask) fwd_force<T, SR, true>(p, a, b, cls, wl, r, s);
    else fwd_force<T, SR, false>(p, a, b, cls, wl, r, s);
    return hipGetLastError();
}

template <class T>
hipError_t adj(const ProblemArgs &p, const void *state, const float *mu_in, float *mu_out,
               int final_t0, const ReduceArgs &r, hipStream_t s)
{
    const T *st = static_cast<const T *>(state);
    const int c = p.col_nzc;
    const unsigned nb = column_blocks(p, c);
    if (final_t0) k_adj_column<T, true><<<nb, NT, 0, s>>>(p, c, st, mu_in, mu_out, r);
    else k_adj_column<T, false><<<nb, NT, 0, s>>>(p, c, st, mu_in, mu_out, r);
    return hipGetLastError();
}

}  // namespace

bool column_supported(const ProblemArgs &p)
{
    // 32-bit byte offsets inside a state buffer: n * 16 bytes < 4 GiB
    return p.Q == 19 && !p.split && p.n < (1LL << 28) && p.col_nzc > 0;
}

// Planes per chunk: as many chunks as give every CU two workgroups (the
// kernels' 120 to 175 VGPRs leave room for two or three), of equal depth, from 2
// to 32 planes: a chunk loads two planes more than it finishes, and fewer waves
// leave the SIMDs waiting.  A step at 75^3 9.0 us with 4 planes (8: 9.7, 2: 11.4), at
// 150x84x75 12.6 with 8 (4: 14.8, 16: 13.7), at 150^3 27.1 with 32 (8: 29.2), at
// 250^3 158 with 32 (8: 174).
int column_choose_depth(const ProblemArgs &p, int ncu)
{
    const int groups = (int)(((long long)p.nx * p.ny + NT - 1) / NT);
    int m = 2 * ncu / (groups > 0 ? groups : 1);
    const int most = (p.nz + 1) / 2, least = (p.nz + 31) / 32;
    m = m > most ? most : (m < least ? least : m);
    // no more workgroups than lwacm_step_static has room for, where that can be
    // had (67 million nodes and more: 34 planes at 407^3)
    const long long room = groups > 0 ? (long long)kStaticMaxBlocks / groups : 0;
    if (room >= 1 && m > room) m = (int)room;
    return (p.nz + m - 1) / m;
}

// Where the columns beat one thread per node.  What they load beyond the nodes'
// own planes is the lanes past a small plane's end and two planes a chunk: over =
// loaded / own.  Generic / columns, us a step:
//   without walls, FP32   41^3 (over 2.2) 6.75 / 6.72, 49^3 7.3 / 6.4, 57^3 8.8 / 7.0,
//     76^3 11.2 / 8.7; 2 x 800 x 801 (2.0) 27.6 / 20.7, 3 x 250 x 251 (2.3) 9.6 / 7.9,
//     1 x 800 x 801 (3.0) 14.3 / 20.0, 4000 x 8 x 9 (5.3) 8.6 / 10.6, 20000 x 3 x 3 6.7 / 35
//   FP16   57^3 7.2 / 8.0, 65^3 9.0 / 10.1, 76^3 12.5 / 10.2, 4 x 300 x 301 (1.5) 11.5 /
//     10.1, 3000 x 17 x 17 (2.1) 18.0 / 18.8, 1500 x 23 x 23 (1.8) 16.8 / 16.6
//   reverse, FP32   49^3 8.07 / 8.14, 57^3 10.5 / 9.8, 76^3 15.3 / 12.3, 3 x 250 x 251
//     9.6 / 10.6, 1 x 800 x 801 19.7 / 34, 2 x 800 x 801 35.9 / 39.1; FP16   65^3 12.9 /
//     13.3, 76^3 14.9 / 13.9
//   walls and a force, FP32 (FP16 alike)   9^3 12.9 / 10.0, 33^3 13.8 / 9.8, 100^3 58.5 /
//     18.1, 1 x 400 x 401 17.4 / 10.5, 1000 x 9 x 9 (6.3) 15.2 / 11.0, 20000 x 5 x 5
//     (10.7) 30 / 51, 9001 x 3 x 3 12 / 22
// Below some nodes a CU (at 256 CUs 10^5 for the FP32 step, 1.3 10^5 for its
// reverse, 3.6 10^5 in FP16) both take a launch's latency and the simple kernel
// starts sooner.
bool column_pays(const ProblemArgs &p, int storage, bool reverse)
{
    const double plane = (double)p.nx * p.ny;
    const double groups = (double)(((long long)p.nx * p.ny + NT - 1) / NT);
    const double chunks = (double)((p.nz + p.col_nzc - 1) / p.col_nzc);
    const double over = groups * NT / plane * (p.nz + 2.0 * chunks) / p.nz;
    if (p.mask) return over <= 8.0;
    const long long per_cu = p.n / (p.ncu > 0 ? p.ncu : 1);
    if (storage) return per_cu >= 1400 && over <= 1.8;
    return reverse ? per_cu >= 500 && over <= 2.3 && p.nz >= 4 : per_cu >= 390 && over <= 2.4;
}

unsigned column_num_blocks(const ProblemArgs &p, unsigned nlist)
{
    return column_blocks(p, p.col_nzc) + (p.mask ? wall_blocks(nlist) : 0u);
}

hipError_t launch_fwd_column(const ProblemArgs &p, int storage, const void *src, void *dst,
                             const uint8_t *cls, const unsigned *list, unsigned nlist,
                             const unsigned *edited, const ReduceArgs &r, hipStream_t stream)
{
    if (!column_supported(p) || (p.mask && (!cls || !list || !edited))) return hipErrorNotSupported;
    const WallList wl{list, nlist, p.mask ? wall_blocks(nlist) : 0u, edited};
    if (!storage) return fwd<float, false>(p, src, dst, cls, wl, r, stream);
    return p.fp16_sr ? fwd<__half, true>(p, src, dst, cls, wl, r, stream)
                     : fwd<__half, false>(p, src, dst, cls, wl, r, stream);
}

hipError_t launch_mask_check(const ProblemArgs &p, const uint8_t *cls, unsigned *edited,
                             hipStream_t stream)
{
    if (!p.mask || !cls || !edited || p.n >= (1LL << 28)) return hipErrorInvalidValue;
    const unsigned nb = (unsigned)((p.n + 16 * NT - 1) / (16 * NT));
    k_mask_check<<<nb < 1024u ? nb : 1024u, NT, 0, stream>>>(p.mask, cls, (unsigned)p.n, edited);
    return hipGetLastError();
}

hipError_t launch_adj_column(const ProblemArgs &p, int storage, const void *state,
                             const float *mu_in, float *mu_out, int final_t0, const ReduceArgs &r,
                             hipStream_t stream)
{
    if (!column_supported(p) || p.mask) return hipErrorNotSupported;
    const hipError_t e = storage ? adj<__half>(p, state, mu_in, mu_out, final_t0, r, stream)
                                 : adj<float>(p, state, mu_in, mu_out, final_t0, r, stream);
    // r.out null: the caller adds the block partials itself (lwacm_adjoint_sweep)
    if (e != hipSuccess || !r.out) return e;
    return launch_reduce(r, 1, column_num_blocks(p, 0), stream);
}

}  // namespace lwacm
