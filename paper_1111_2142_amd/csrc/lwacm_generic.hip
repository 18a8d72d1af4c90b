// lwacm_generic.hip -- one-thread-per-node LW-ACM kernels for D2Q9 and D3Q19.
//
// Forward step (Eq. ACM2.0 in pull form, Eqs. ACM2.0b): every fluid node x
// gathers, for each link i, the pre-combined term of its upstream node
// x - v_i; a solid upstream node is replaced by the node's own term for the
// opposite link plus the moving-wall correction (halfway bounce-back,
// Eqs. ACM2.0cbb-ACM2.0ccccbb).  The post-combine term sums to a rho_x u_x in
// the momentum, and the forcing of Eq. force adds rho_x g.  Neighbours come
// straight from global memory (L2 hits); this path serves every lattice,
// size and mask and is the baseline the tile kernels are checked against.
//
// Reverse step: every source node y collects, for each of its links k, the
// cotangent weight of the node that consumes its term (y + v_k, or y itself
// through bounce-back) and applies the transposed derivative of the link term.
#include <type_traits>

#include "lwacm_device.hpp"
#include "lwacm_generic_update.hpp"
#include "lwacm_internal.hpp"

namespace lwacm {

namespace {

struct Coord {
    int x, y, z;
};

__device__ __forceinline__ Coord decompose(long long idx, int nx, int ny)
{
    long long t = idx / nx;
    Coord c;
    c.x = (int)(idx - t * nx);
    c.z = (int)(t / ny);
    c.y = (int)(t - (long long)c.z * ny);
    return c;
}

__device__ __forceinline__ int wrap_add(int a, int d, int n)
{
    int r = a + d;
    return r < 0 ? r + n : (r >= n ? r - n : r);
}

__device__ __forceinline__ long long node_at(const ProblemArgs &p, int x, int y, int z)
{
    return ((long long)z * p.ny + y) * p.nx + x;
}

// State of node idx (node-interleaved storage): rho - 1 and u (u[2] = 0 in 2D).
template <int D, class T>
__device__ __forceinline__ void load_state(const T *s, long long idx, const ProblemArgs &p,
                                           float &drho, float (&u)[3])
{
    float v[D + 1];
    NodeState<T, D + 1>::load(s, idx, p.ld_scale, v);
    drho = v[0];
    u[0] = v[1];
    u[1] = v[2];
    u[2] = (D == 3) ? v[D] : 0.0f;
}

// The reverse sweep's mu (dL/dD, dL/dJ) between steps: node-interleaved
// FP32, D+1 values per node (one 16-byte access in 3D).
template <int D>
__device__ __forceinline__ void load_mu(const float *mu, long long idx, float &r, float (&j)[3])
{
    if constexpr (D == 3) {
        const float4 q = reinterpret_cast<const float4 *>(mu)[idx];
        r = q.x;
        j[0] = q.y;
        j[1] = q.z;
        j[2] = q.w;
    } else {
        r = mu[3 * idx];
        j[0] = mu[3 * idx + 1];
        j[1] = mu[3 * idx + 2];
        j[2] = 0.0f;
    }
}

template <int D>
__device__ __forceinline__ void store_mu(float *mu, long long idx, float r, const float (&j)[3])
{
    if constexpr (D == 3) {
        reinterpret_cast<float4 *>(mu)[idx] = make_float4(r, j[0], j[1], j[2]);
    } else {
        mu[3 * idx] = r;
        mu[3 * idx + 1] = j[0];
        mu[3 * idx + 2] = j[1];
    }
}

template <int Q, class T, bool MASK, bool FORCE, bool SPLIT>
__global__ __launch_bounds__(kGenericBlock) void k_fwd_generic(ProblemArgs p, const T *__restrict__ src,
                                                               T *__restrict__ dst, ReduceArgs r)
{
    using L = Lattice<Q>;
    constexpr int D = L::D;
    const long long n = p.n;
    double acc[2] = {0.0, 0.0};  // mass deviation sum(rho - 1), energy
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (long long)gridDim.x * blockDim.x) {
        float drx, ux[3];
        load_state<D, T>(src, idx, p, drx, ux);
        if (MASK && p.mask[idx] != 0) {
            // solid node: never updated, copied through to the other buffer
            // (a stored value converts back to itself exactly)
            float v[D + 1];
            v[0] = drx;
#pragma unroll
            for (int k = 0; k < D; ++k) v[k + 1] = ux[k];
            NodeState<T, D + 1>::store(dst, idx, v, p.st_scale);
            continue;
        }
        const Coord c = decompose(idx, p.nx, p.ny);
        auto at = [&](int dx, int dy, int dz) {
            return node_at(p, wrap_add(c.x, dx, p.nx), wrap_add(c.y, dy, p.ny),
                           wrap_add(c.z, dz, p.nz));
        };
        auto fmask = [&](int dx, int dy, int dz) -> uint8_t { return p.mask[at(dx, dy, dz)]; };
        auto fstate = [&](int dx, int dy, int dz, float &dr, float (&u)[3], float &B) {
            load_state<D, T>(src, at(dx, dy, dz), p, dr, u);
            B = node_B(u);
        };
        float out[D + 1], e;
        link_update<Q, MASK, FORCE, SPLIT>(p, GlobalSite<Q>{p, idx}, drx, ux, node_B(ux), fmask, fstate, out, e);
        if (std::is_same<T, __half>::value && p.fp16_sr) {
            NodeState<T, D + 1>::store_sr(dst, idx, out, p.st_scale,
                                          sr_words((uint32_t)idx, p.sr_word));
        } else {
            NodeState<T, D + 1>::store(dst, idx, out, p.st_scale);
        }
        acc[0] += (double)out[0];
        acc[1] += 0.5 * (double)e;
    }
    store_block_partials<2>(acc, r.partials, blockIdx.x);
    if (blockIdx.x == 0 && r.prev_nblocks)
        finish_previous_sums(r.prev_partials, r.prev_nblocks, r.prev_out, r.prev_out2);
}

// Semi-implicit pressure update (Section "The main algorithm: Finite
// difference formulation", item 2, Eq. FDcompact_si), second pass of a step:
// the density of the step is the zeroth moment of the Eq. ACM2.0 populations
// evaluated with the old density (src) and the velocity the explicit pass
// has just written (dst); it replaces that pass's density in dst.  Other
// threads read only the velocity of dst, so writing the density field in
// place is safe (a node's density value loaded with its velocity goes
// unused).  Forcing adds nothing to the density.  FP32 storage.
template <int Q, bool MASK>
__global__ __launch_bounds__(kGenericBlock) void k_density_si(ProblemArgs p,
                                                              const float *__restrict__ src,
                                                              float *dst, ReduceArgs r)
{
    using L = Lattice<Q>;
    constexpr int D = L::D;
    const long long n = p.n;
    double acc[2] = {0.0, 0.0};
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (long long)gridDim.x * blockDim.x) {
        if (MASK && p.mask[idx] != 0) continue;
        const Coord c = decompose(idx, p.nx, p.ny);
        float drx, ux[3], dnew, unew[3];
        load_state<D, float>(src, idx, p, drx, ux);
        load_state<D, float>(dst, idx, p, dnew, unew);
        (void)dnew;
        (void)ux;
        const float rx = 1.0f + drx;
        const float Bx = -1.5f * (unew[0] * unew[0] + unew[1] * unew[1] + unew[2] * unew[2]);
        float D36 = 0.0f;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const long long up = node_at(p, wrap_add(c.x, -link_cx(i), p.nx),
                                         wrap_add(c.y, -link_cy(i), p.ny),
                                         wrap_add(c.z, -link_cz(i), p.nz));
            float s;
            uint8_t m = 0;
            if (MASK) m = p.mask[up];
            if (MASK && m != 0) {
                // halfway bounce-back and the wall motion's share of the density
                const int ib = link_opp(i);
                const float uw[3] = {p.wall_term[m][0], p.wall_term[m][1], p.wall_term[m][2]};
                s = link_term_unweighted(drx, rx, vdot<Q>(ib, unew), Bx, p.A) + vdot<Q>(i, uw);
            } else {
                float dry, uy_old[3];
                load_state<D, float>(src, up, p, dry, uy_old);
                (void)uy_old;
                float dyn, uy[3];
                load_state<D, float>(dst, up, p, dyn, uy);
                (void)dyn;
                const float By = -1.5f * (uy[0] * uy[0] + uy[1] * uy[1] + uy[2] * uy[2]);
                s = link_term_unweighted(dry, 1.0f + dry, vdot<Q>(i, uy), By, p.A);
            }
            D36 = fmaf(L::w36(i), s, D36);
        }
        const float Dsum = div36(D36);
        dst[(long long)(D + 1) * idx] = Dsum;
        float e = 0.0f;
#pragma unroll
        for (int k = 0; k < D; ++k) e = fmaf(unew[k], unew[k], e);
        acc[0] += (double)Dsum;
        acc[1] += 0.5 * (double)e;
    }
    store_block_partials<2>(acc, r.partials, blockIdx.x);
}

template <int Q, class T, bool MASK>
__global__ __launch_bounds__(kGenericBlock) void k_adj_generic(ProblemArgs p, const T *__restrict__ state,
                                                               const float *__restrict__ mu_in,
                                                               float *__restrict__ mu_out,
                                                               int final_t0, ReduceArgs r)
{
    using L = Lattice<Q>;
    constexpr int D = L::D;
    const long long n = p.n;
    double acc[1] = {0.0};  // dL/da
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (long long)gridDim.x * blockDim.x) {
        if (MASK && p.mask[idx] != 0) {
            if (final_t0) {
                for (int k = 0; k <= D; ++k) mu_out[k * n + idx] = 0.0f;
            } else {
                const float z[3] = {0.0f, 0.0f, 0.0f};
                store_mu<D>(mu_out, idx, 0.0f, z);
            }
            continue;
        }
        float dry, uy[3];
        load_state<D, T>(state, idx, p, dry, uy);
        const Coord c = decompose(idx, p.nx, p.ny);
        float muR_y, muJ_y[3];
        load_mu<D>(mu_in, idx, muR_y, muJ_y);
        auto at = [&](int dx, int dy, int dz) {
            return node_at(p, wrap_add(c.x, dx, p.nx), wrap_add(c.y, dy, p.ny),
                           wrap_add(c.z, dz, p.nz));
        };
        auto fmask = [&](int dx, int dy, int dz) -> uint8_t { return p.mask[at(dx, dy, dz)]; };
        auto fm = [&](int k) {
            float mr, mt[3];
            load_mu<D>(mu_in, at(link_cx(k), link_cy(k), link_cz(k)), mr, mt);
            return mr + vdot<Q>(k, mt);
        };
        float lr, lu[3], da;
        adj_node_update<Q, MASK>(p, dry, uy, muR_y, muJ_y, fmask, fm, lr, lu, da);
        if (final_t0) {
            // the gradient with respect to the initial state, field-major
            mu_out[idx] = lr;
#pragma unroll
            for (int j = 0; j < D; ++j) mu_out[(j + 1) * n + idx] = lu[j];
        } else {
            float mR, mJ[3];
            adj_fold<D>(dry, uy, lr, lu, mR, mJ);
            store_mu<D>(mu_out, idx, mR, mJ);
        }
        acc[0] += (double)da;
    }
    store_block_partials<1>(acc, r.partials, blockIdx.x);
}

template <int D, class T>
__global__ __launch_bounds__(kGenericBlock) void k_adj_seed(ProblemArgs p, const T *__restrict__ state,
                                                            const float *__restrict__ lam,
                                                            float *__restrict__ mu)
{
    const long long n = p.n;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (long long)gridDim.x * blockDim.x) {
        float mj[3] = {0.0f, 0.0f, 0.0f};
        if (p.mask && p.mask[idx] != 0) {
            store_mu<D>(mu, idx, 0.0f, mj);
            continue;
        }
        float dr, u[3];
        load_state<D, T>(state, idx, p, dr, u);
        const float inv = 1.0f / (1.0f + dr);
        float lu_u = 0.0f;
        for (int j = 0; j < D; ++j) lu_u = fmaf(lam[(j + 1) * n + idx], u[j], lu_u);
        for (int j = 0; j < D; ++j) mj[j] = lam[(j + 1) * n + idx] * inv;
        store_mu<D>(mu, idx, lam[idx] - lu_u * inv, mj);
    }
}

// The state from field-major FP32 fields, with the (mass deviation, energy)
// sums of the stored values over the fluid nodes (as k_moments sums them).
// other: the second state buffer of a masked problem, which holds the solid
// nodes' values too (a step may leave them unwritten).  One pass, bound by HBM:
// at 256^3 FP32 the fields read and the state written once, where a copy of the
// state and a pass for the sums took as long again each (270 us, now 105).
template <int D, class T>
__global__ __launch_bounds__(kGenericBlock) void k_set_state(ProblemArgs p, const float *__restrict__ drho,
                                                             const float *__restrict__ u,
                                                             T *__restrict__ dst,
                                                             T *__restrict__ other, ReduceArgs r)
{
    const long long n = p.n;
    double acc[2] = {0.0, 0.0};
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (long long)gridDim.x * blockDim.x) {
        float v[D + 1];
        v[0] = drho[idx];
        for (int k = 0; k < D; ++k) v[k + 1] = u[k * n + idx];
        NodeState<T, D + 1>::store(dst, idx, v, p.st_scale);
        if (p.mask && p.mask[idx] != 0) {
            NodeState<T, D + 1>::store(other, idx, v, p.st_scale);
            continue;
        }
        if constexpr (std::is_same<T, __half>::value)  // the values as stored
#pragma unroll
            for (int f = 0; f <= D; ++f)
                v[f] = __half2float(__float2half_rn(v[f] * p.st_scale[f > 0])) * p.ld_scale[f > 0];
        float e = 0.0f;
        for (int k = 0; k < D; ++k) e = fmaf(v[k + 1], v[k + 1], e);
        acc[0] += (double)v[0];
        acc[1] += 0.5 * (double)e;
    }
    store_block_partials<2>(acc, r.partials, blockIdx.x);
}

// SUMS: the (mass deviation, energy) sums too.
template <int D, class T, bool SUMS>
__global__ __launch_bounds__(kGenericBlock) void k_moments(ProblemArgs p, const T *__restrict__ src,
                                                           float *__restrict__ drho,
                                                           float *__restrict__ u, ReduceArgs r)
{
    const long long n = p.n;
    double acc[2] = {0.0, 0.0};
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (long long)gridDim.x * blockDim.x) {
        float dr, uu[3];
        load_state<D, T>(src, idx, p, dr, uu);
        if (drho) drho[idx] = dr;
        if (u)
            for (int k = 0; k < D; ++k) u[k * n + idx] = uu[k];
        if (!SUMS || (p.mask && p.mask[idx] != 0)) continue;
        float e = 0.0f;
        for (int k = 0; k < D; ++k) e = fmaf(uu[k], uu[k], e);
        acc[0] += (double)dr;
        acc[1] += 0.5 * (double)e;
    }
    if (SUMS) store_block_partials<2>(acc, r.partials, blockIdx.x);
}

// Largest mask value and number of fluid nodes (integer atomics: exact).  The
// two words take every block's atomics one after the other, so few blocks with
// 16-byte loads: 192^3 104 us with 4096 blocks and a byte a thread, 11 us now.
__global__ __launch_bounds__(kGenericBlock) void k_mask_scan(ProblemArgs p, unsigned *out)
{
    __shared__ unsigned s_max, s_fluid;
    if (threadIdx.x == 0) s_max = s_fluid = 0;
    __syncthreads();
    unsigned mx = 0, fluid = 0;
    auto node = [&](unsigned m) {
        mx = m > mx ? m : mx;
        fluid += (m == 0);
    };
    const long long first = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long threads = (long long)gridDim.x * blockDim.x;
    // bytes up to the first 16-byte boundary, whole uint4, the rest
    const long long to16 = (long long)((16u - (unsigned)((uintptr_t)p.mask & 15u)) & 15u);
    const long long head = to16 < p.n ? to16 : p.n;
    const long long body = (p.n - head) / 16;
    const long long tail = head + 16 * body;  // n - tail < 16
    if (first < head) node(p.mask[first]);
    const uint4 *v = reinterpret_cast<const uint4 *>(p.mask + head);
#pragma unroll 4
    for (long long i = first; i < body; i += threads) {
        const uint4 q = v[i];
        const unsigned w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            for (int b = 0; b < 32; b += 8) node((w[k] >> b) & 255u);
    }
    if (first < p.n - tail) node(p.mask[tail + first]);
#pragma unroll
    for (int o = kWave / 2; o > 0; o /= 2) {
        const unsigned m = __shfl_xor(mx, o);
        mx = m > mx ? m : mx;
        fluid += __shfl_xor(fluid, o);
    }
    if (threadIdx.x % kWave == 0) {
        atomicMax(&s_max, mx);
        atomicAdd(&s_fluid, fluid);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicMax(&out[0], s_max);
        atomicAdd(&out[1], s_fluid);
    }
}

unsigned grid_for(long long n)
{
    long long b = (n + kGenericBlock - 1) / kGenericBlock;
    if (b < 1) b = 1;
    return (unsigned)(b > (long long)kGenericMaxBlocks ? kGenericMaxBlocks : b);
}

template <int Q, class T, bool SPLIT>
hipError_t fwd_dispatch_split(const ProblemArgs &p, bool force, const T *a, T *b,
                              const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    if (p.mask) {
        if (force)
            k_fwd_generic<Q, T, true, true, SPLIT><<<nb, kGenericBlock, 0, s>>>(p, a, b, r);
        else
            k_fwd_generic<Q, T, true, false, SPLIT><<<nb, kGenericBlock, 0, s>>>(p, a, b, r);
    } else {
        if (force)
            k_fwd_generic<Q, T, false, true, SPLIT><<<nb, kGenericBlock, 0, s>>>(p, a, b, r);
        else
            k_fwd_generic<Q, T, false, false, SPLIT><<<nb, kGenericBlock, 0, s>>>(p, a, b, r);
    }
    return hipGetLastError();
}

template <int Q, class T>
hipError_t fwd_dispatch(const ProblemArgs &p, bool force, const void *src, void *dst,
                        const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    const T *a = static_cast<const T *>(src);
    T *b = static_cast<T *>(dst);
    if (p.split)
        return fwd_dispatch_split<Q, T, true>(p, force, a, b, r, nb, s);
    return fwd_dispatch_split<Q, T, false>(p, force, a, b, r, nb, s);
}

template <int Q, class T>
hipError_t adj_dispatch(const ProblemArgs &p, const void *state, const float *mu_in,
                        float *mu_out, int final_t0, const ReduceArgs &r, unsigned nb,
                        hipStream_t s)
{
    const T *st = static_cast<const T *>(state);
    if (p.mask)
        k_adj_generic<Q, T, true><<<nb, kGenericBlock, 0, s>>>(p, st, mu_in, mu_out, final_t0, r);
    else
        k_adj_generic<Q, T, false><<<nb, kGenericBlock, 0, s>>>(p, st, mu_in, mu_out, final_t0, r);
    return hipGetLastError();
}

// Second pass of the grid reductions: one block adds the NV partial sums of
// nblocks blocks in a fixed order (strided per thread, then a fixed tree).
template <int NV>
__global__ __launch_bounds__(kGenericBlock) void k_reduce_partials(ReduceArgs r, unsigned nblocks)
{
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    for (unsigned b = threadIdx.x; b < nblocks; b += kReduceThreads)
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] += r.partials[(size_t)NV * b + k];
    block_sum<NV>(acc);
    if (threadIdx.x == 0) {
        if (r.accumulate) {
            r.out[0] += acc[0] * r.out_scale;
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) acc[k] *= r.out_scale;
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                r.out[k] = acc[k];
                if (r.out2) r.out2[k] = acc[k];
            }
        }
    }
}

// The per-step block partials of a reverse sweep (one reduction per slice of
// `stride` doubles, nb_first or nb_rest of them filled): block s adds slice s
// in the order of k_reduce_partials.
__global__ __launch_bounds__(kGenericBlock) void k_reduce_slices(const double *partials,
                                                                 size_t stride, unsigned nb_first,
                                                                 unsigned nfirst, unsigned nb_rest,
                                                                 double *totals)
{
    const double *slice = partials + (size_t)blockIdx.x * stride;
    const unsigned nblocks = blockIdx.x < nfirst ? nb_first : nb_rest;
    double acc[1] = {0.0};
    for (unsigned b = threadIdx.x; b < nblocks; b += kReduceThreads) acc[0] += slice[b];
    block_sum<1>(acc);
    if (threadIdx.x == 0) totals[blockIdx.x] = acc[0];
}

// out += total_s * scale for s = 0, 1, ... in turn: what the reductions of
// separate reverse-step calls add, in the same order.  One wave, so that the
// totals arrive together and only the additions run one after the other.
__global__ __launch_bounds__(kWave) void k_accumulate_totals(const double *totals, unsigned n,
                                                             double scale, double *out)
{
    __shared__ double t[kWave];
    double v = out[0];
    for (unsigned s0 = 0; s0 < n; s0 += kWave) {
        if (s0 + threadIdx.x < n) t[threadIdx.x] = totals[s0 + threadIdx.x] * scale;
        __syncthreads();
        if (threadIdx.x == 0)
            for (unsigned s = 0; s < n - s0 && s < kWave; ++s) v += t[s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = v;
}

}  // namespace

hipError_t launch_reduce_slices(const double *partials, size_t stride, unsigned nb_first,
                                unsigned nfirst, unsigned nb_rest, unsigned nslices,
                                double *totals, double scale, double *out, hipStream_t s)
{
    if (nslices == 0) return hipSuccess;
    // the thread count and tree of k_reduce_partials
    k_reduce_slices<<<nslices, kReduceThreads, 0, s>>>(partials, stride, nb_first, nfirst, nb_rest,
                                                       totals);
    k_accumulate_totals<<<1, kWave, 0, s>>>(totals, nslices, scale, out);
    return hipGetLastError();
}

hipError_t launch_reduce(const ReduceArgs &r, int nv, unsigned nblocks, hipStream_t s)
{
    if (nv == 1)
        k_reduce_partials<1><<<1, kReduceThreads, 0, s>>>(r, nblocks);
    else
        k_reduce_partials<2><<<1, kReduceThreads, 0, s>>>(r, nblocks);
    return hipGetLastError();
}

hipError_t launch_density_si(const ProblemArgs &p, const float *src, float *dst,
                             const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    if (p.Q == 9) {
        if (p.mask)
            k_density_si<9, true><<<nb, kGenericBlock, 0, s>>>(p, src, dst, r);
        else
            k_density_si<9, false><<<nb, kGenericBlock, 0, s>>>(p, src, dst, r);
    } else {
        if (p.mask)
            k_density_si<19, true><<<nb, kGenericBlock, 0, s>>>(p, src, dst, r);
        else
            k_density_si<19, false><<<nb, kGenericBlock, 0, s>>>(p, src, dst, r);
    }
    return hipGetLastError();
}

hipError_t launch_fwd_generic(const ProblemArgs &p, int storage, bool force, const void *src,
                              void *dst, const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    if (p.Q == 9)
        return storage ? fwd_dispatch<9, __half>(p, force, src, dst, r, nb, s)
                       : fwd_dispatch<9, float>(p, force, src, dst, r, nb, s);
    return storage ? fwd_dispatch<19, __half>(p, force, src, dst, r, nb, s)
                   : fwd_dispatch<19, float>(p, force, src, dst, r, nb, s);
}

hipError_t launch_adj_generic(const ProblemArgs &p, int storage, const void *state,
                              const float *mu_in, float *mu_out, int final_t0,
                              const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    hipError_t e;
    if (p.Q == 9)
        e = storage ? adj_dispatch<9, __half>(p, state, mu_in, mu_out, final_t0, r, nb, s)
                    : adj_dispatch<9, float>(p, state, mu_in, mu_out, final_t0, r, nb, s);
    else
        e = storage ? adj_dispatch<19, __half>(p, state, mu_in, mu_out, final_t0, r, nb, s)
                    : adj_dispatch<19, float>(p, state, mu_in, mu_out, final_t0, r, nb, s);
    // r.out null: the caller adds the block partials itself (lwacm_adjoint_sweep)
    if (e != hipSuccess || !r.out) return e;
    return launch_reduce(r, 1, nb, s);
}

hipError_t launch_adj_seed(const ProblemArgs &p, int storage, const void *state,
                           const float *lambda, float *mu, hipStream_t s)
{
    const unsigned nb = grid_for(p.n);
    if (p.D == 2) {
        if (storage)
            k_adj_seed<2, __half><<<nb, kGenericBlock, 0, s>>>(p, (const __half *)state, lambda, mu);
        else
            k_adj_seed<2, float><<<nb, kGenericBlock, 0, s>>>(p, (const float *)state, lambda, mu);
    } else {
        if (storage)
            k_adj_seed<3, __half><<<nb, kGenericBlock, 0, s>>>(p, (const __half *)state, lambda, mu);
        else
            k_adj_seed<3, float><<<nb, kGenericBlock, 0, s>>>(p, (const float *)state, lambda, mu);
    }
    return hipGetLastError();
}

hipError_t launch_set_state(const ProblemArgs &p, int storage, const float *drho,
                            const float *u, void *dst, void *other, const ReduceArgs &r,
                            hipStream_t s)
{
    const unsigned nb = grid_for(p.n);
    __half *dh = (__half *)dst, *oh = (__half *)other;
    float *df = (float *)dst, *of = (float *)other;
    if (p.D == 2) {
        if (storage) k_set_state<2, __half><<<nb, kGenericBlock, 0, s>>>(p, drho, u, dh, oh, r);
        else k_set_state<2, float><<<nb, kGenericBlock, 0, s>>>(p, drho, u, df, of, r);
    } else {
        if (storage) k_set_state<3, __half><<<nb, kGenericBlock, 0, s>>>(p, drho, u, dh, oh, r);
        else k_set_state<3, float><<<nb, kGenericBlock, 0, s>>>(p, drho, u, df, of, r);
    }
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_reduce(r, 2, nb, s);
}

template <int D, class T>
static void moments_t(const ProblemArgs &p, const void *src, float *drho, float *u,
                      const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    if (r.out)
        k_moments<D, T, true><<<nb, kGenericBlock, 0, s>>>(p, (const T *)src, drho, u, r);
    else
        k_moments<D, T, false><<<nb, kGenericBlock, 0, s>>>(p, (const T *)src, drho, u, r);
}

hipError_t launch_moments(const ProblemArgs &p, int storage, const void *src, float *drho,
                          float *u, const ReduceArgs &r, unsigned nb, hipStream_t s)
{
    if (p.D == 2) {
        if (storage) moments_t<2, __half>(p, src, drho, u, r, nb, s);
        else moments_t<2, float>(p, src, drho, u, r, nb, s);
    } else {
        if (storage) moments_t<3, __half>(p, src, drho, u, r, nb, s);
        else moments_t<3, float>(p, src, drho, u, r, nb, s);
    }
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || !r.out ? e : launch_reduce(r, 2, nb, s);
}

hipError_t launch_mask_scan(const ProblemArgs &p, unsigned *d_out2, hipStream_t s)
{
    const unsigned nb = grid_for((p.n + 63) / 64);  // four uint4 a thread
    k_mask_scan<<<nb < 256u ? nb : 256u, kGenericBlock, 0, s>>>(p, d_out2);
    return hipGetLastError();
}

unsigned generic_grid(long long n) { return grid_for(n); }

}  // namespace lwacm
