// lwacm_adjoint_march.hip -- reverse (adjoint) step of the D3Q19 LW-ACM
// update as a z-marching tile kernel.
//
// The per-node arithmetic (moments of the link cotangents, Eqs. ACM2.0b
// differentiated) is in lwacm_adjoint_common.hpp.
//
// Design (gfx950).  A workgroup owns a 32 x 16 tile of columns and a chunk of
// planes, as the forward march kernel.  Every plane of mu (tile plus a
// one-column halo ring) passes once through a rolling window of four LDS
// planes, its four components in separate arrays; each interior thread then reads its 18
// neighbours' mu from the three planes around its own, accumulates the ten
// moments with integer weights 36 w_k (pairs of opposite links share one
// expansion), and finishes the node from its own state, which it loads
// itself (16 B FP32 / 8 B FP16 per node).  Halo waves only load mu into LDS.
// One barrier per plane; four window planes mean a plane is overwritten only
// after every thread has passed the next barrier.  HBM traffic per node:
// state + mu_in + mu_out = 48 B (FP32 state).
//
// The plane loop is rolled (plane_loop), the chunk depth a run-time value, and a
// ragged last chunk is moved down to end at nz, as in the other
// tile kernels: its planes below zs are written twice with the same bits and
// counted once.  Every load and store is unconditional and a ring slot is
// refilled after its last use, so the loads stay in flight across the back
// edge.
#include "lwacm_adjoint_common.hpp"

namespace lwacm {

namespace {

constexpr int TX = 32;
constexpr int TY = 16;
constexpr int RING = 3;                     // planes of loads in flight per thread
constexpr int NWIN = 4;                     // LDS window planes
constexpr int NINT = TX * TY;
constexpr int NTHREADS = NINT + 2 * kWave;  // + Y-halo wave + X-halo wave
constexpr int SX = TX + 2;
constexpr int NSLOT = SX * (TY + 2);

static_assert(2 * TX <= kWave && 2 * (TY + 2) <= kWave, "halo rows must fit one wave each");

enum Role { INTERIOR = 0, HALO_Y = 1, HALO_X = 2 };

// The plane loop; TAIL 0: grids of fewer than eight planes (n <= 9), too short for
// plane_loop, unrolled.
template <int TAIL, class F>
__device__ __forceinline__ void adj_loop(int n, F &&body)
{
    if constexpr (TAIL != 0) {
        plane_loop<TAIL>(n, body);
    } else {
        static_for<9>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (k < n) body(k, PlaneIter<k % 3, (k < 5 ? k : 5), true>{});
        });
    }
}

// XOUT (no walls): the factors (rho, x) of the nodes' dL/da = rho x go to xout
// (n pairs) instead of into block partials; chunks of any depth then give the same sums
// (k_adj_dadomega adds them).
//
// PAIR: held to 80 VGPRs (six waves a SIMD; 7 to 23 spilled).  The 88 to 93 it
// takes otherwise allow five, 20 waves a CU, which two workgroups of ten fill
// exactly, and not on every CU do the second one's waves find their SIMDs: where
// the grid is one full round of two workgroups a CU, the ones left over make a
// round of their own (256^3, 512 workgroups: 189 us, held 170).  On other grids the
// spills cost more (224^3, 392 workgroups: 121, held 133; 288 x 256 x 256, 576:
// 208, held 221; 192^3, one a CU: 67, held 82).
template <class T, int TAIL, bool MASK, bool FINAL, bool XOUT, bool PAIR>
__global__ __launch_bounds__((NTHREADS), (PAIR ? 6 : 1)) void k_adj_march(ProblemArgs p, int nzc,
                                                        const T *__restrict__ state,
                                                        const float *__restrict__ mu_in,
                                                        float *__restrict__ mu_out,
                                                        const unsigned *__restrict__ bb_bits,
                                                        const float4 *__restrict__ wallg,
                                                        float2 *__restrict__ xout, ReduceArgs r)
{
    static_assert(!(XOUT && MASK), "x is written for problems without walls");
    // one spare slot: idle halo lanes write there instead of branching
    __shared__ float win[NWIN][4][NSLOT + 1];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int nx = p.nx, ny = p.ny, nz = p.nz;
    const long long n = p.n;
    const long long plane = (long long)nx * ny;

    const TileIdx ti = tile_of_block(nx, ny, TX, TY);
    const int zs = ti.zc * nzc;
    const int z0 = min(zs, nz - nzc);

    // column in tile coordinates [-1, TX] x [-1, TY]
    const int role = tid < NINT ? INTERIOR : (tid < NINT + kWave ? HALO_Y : HALO_X);
    int lx, ly;
    bool active = true;
    if (role == INTERIOR) {
        lx = tid % TX;
        ly = tid / TX;
    } else if (role == HALO_Y) {
        const bool top = lane >= TX;
        lx = top ? lane - TX : lane;
        ly = top ? TY : -1;
        active = lane < 2 * TX;
        if (!active) lx = 0;
    } else {
        const bool right = lane >= TY + 2;
        const int l = right ? lane - (TY + 2) : lane;
        lx = right ? TX : -1;
        ly = l - 1;
        active = lane < 2 * (TY + 2);
        if (!active) ly = 0;
    }
    const int gx = wrap_index(ti.x0 + lx, nx);
    const int gy = wrap_index(ti.y0 + ly, ny);
    const unsigned col = (unsigned)(gy * nx + gx);
    const int slot = (ly + 1) * SX + (lx + 1);
    const int wslot = active ? slot : NSLOT;

    // (fewer than eight planes: loads past the chunk stay at its upper end)
    auto wrapz = [&](int pz) { return wrap_index(TAIL ? pz : min(pz, z0 + nzc), nz); };
    constexpr unsigned NB = StateIO<T>::kNodeBytes;
    const Rsrc rmu = make_rsrc(mu_in, (unsigned long long)n * 16u);
    const Rsrc rst = make_rsrc(state, (unsigned long long)n * NB);
    const Rsrc rout = make_rsrc(mu_out, (unsigned long long)n * 16u);
    const Rsrc rbits = make_rsrc(bb_bits, MASK ? (unsigned long long)n * 4u : 0ull);
    const Rsrc rx = make_rsrc(XOUT ? xout : nullptr, XOUT ? (unsigned long long)n * 8u : 0ull);
    const unsigned mu_plane = (unsigned)(plane * 16);
    const unsigned st_plane = (unsigned)(plane * NB);
    const unsigned voff_mu = col * 16u;
    const unsigned voff_st = col * NB;

    // Load rings, indexed by k % 3 at compile time: mu of plane pz = z0 - 1 + k
    // is in mr[k % 3] at iteration k, the state (and, with MASK, the link set)
    // of the plane finalised there, pz - 1, in sr[(k + 2) % 3].
    f32x4 mr[RING];
    typename StateIO<T>::Raw sr[RING];
    unsigned bw[RING] = {0u, 0u, 0u};
    auto load_state = [&](int j, int pz) {
        const unsigned pw = (unsigned)wrapz(pz);
        sr[j] = StateIO<T>::load(rst, voff_st, pw * st_plane);
        if (MASK)
            bw[j] = __builtin_amdgcn_raw_buffer_load_b32(rbits, col * 4u, pw * (unsigned)(plane * 4),
                                                         0);
    };
#pragma unroll
    for (int j = 0; j < RING; ++j) mr[j] = load_f4(rmu, voff_mu, (unsigned)wrapz(z0 - 1 + j) * mu_plane);
    if (role == INTERIOR) {
        load_state(1, z0);
        load_state(2, z0 + 1);
        load_state(0, z0 + 2);
    }

    float da = 0.0f;
    const int N = nzc + 2;  // planes z0 - 1 .. z1 of mu

    // mu of plane pz into window slot k % NWIN (every thread)
    auto enter = [&](int k, auto It) {
        using I = decltype(It);
        __builtin_amdgcn_sched_barrier(0);
        float(*W)[NSLOT + 1] = win[k % NWIN];
        const f32x4 q = mr[I::j];
        W[0][wslot] = q.x;
        W[1][wslot] = q.y;
        W[2][wslot] = q.z;
        W[3][wslot] = q.w;
        __builtin_amdgcn_sched_barrier(0);
        if (I::refill) mr[I::j] = load_f4(rmu, voff_mu, (unsigned)wrapz(z0 + 2 + k) * mu_plane);
    };

    if (role == INTERIOR) {
        adj_loop<TAIL>(N, [&](int k, auto kc) {
            using I = decltype(kc);
            constexpr int jm = (I::j + 2) % 3;
            enter(k, I{});
            __syncthreads();
            if (I::phase < 2) return;
            const int tz = z0 - 2 + k;  // plane finalised now (z0 .. z1 - 1)
            float d, ux, uy, uz;
            StateIO<T>::unpack(sr[jm], p.ld_scale, d, ux, uy, uz);
            const unsigned bits = bw[jm];
            const bool solid = MASK && (bits & 1u);  // bit 0: a solid node
            float dan = da;
            f32x4 lam = adj_point<MASK, NSLOT + 1, SX, XOUT>(
                win[(k + NWIN - 2) % NWIN], win[(k + NWIN - 1) % NWIN], win[k % NWIN], slot, d, ux,
                uy, uz, bits, wallg, (long long)tz * plane + col, p, dan);
            if (XOUT) {
                store_factors(rx, col * 8u, (unsigned)tz * (unsigned)(plane * 8), d, dan);
            } else {
                da = (tz >= zs && !solid) ? dan : da;
            }
            if (FINAL) {
                // the gradient with respect to the initial state, field-major
                if (solid) lam = f32x4{0.0f, 0.0f, 0.0f, 0.0f};  // solid nodes carry no cotangent
                const unsigned so = (unsigned)tz * (unsigned)(plane * 4);
                const unsigned fs = (unsigned)(n * 4);
                const u32x4 lb = __builtin_bit_cast(u32x4, lam);
                __builtin_amdgcn_raw_buffer_store_b32(lb.x, rout, col * 4u, so, 0);
                store_data_guard();
                __builtin_amdgcn_raw_buffer_store_b32(lb.y, rout, col * 4u, so + fs, 0);
                store_data_guard();
                __builtin_amdgcn_raw_buffer_store_b32(lb.z, rout, col * 4u, so + 2 * fs, 0);
                store_data_guard();
                __builtin_amdgcn_raw_buffer_store_b32(lb.w, rout, col * 4u, so + 3 * fs, 0);
                store_data_guard();
            } else {
                f32x4 mu = fold_normalisation(lam, d, ux, uy, uz);
                if (solid) mu = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, mu), rout, voff_mu,
                                                       (unsigned)tz * mu_plane, 0);
                store_data_guard();
            }
            __builtin_amdgcn_sched_barrier(0);  // the state's last use is above
            if (I::refill) load_state(jm, z0 + 1 + k);
        });
    } else {
        adj_loop<TAIL>(N, [&](int k, auto kc) {
            enter(k, kc);
            __syncthreads();
        });
    }

    if (XOUT) return;
    double v[1] = {(double)da};
    store_block_partials<1>(v, r.partials, blockIdx.x);
}

// dL/da of reverse steps whose nodes' factors (rho, x) were written by the tile
// kernels (XOUT).  The reverse kernels without XOUT sum a thread's planes in
// FP32 (da = fma(rho, x, da) up its chunk of nzc planes), then over the block
// and the grid in FP64; this kernel does the same sums on the same tiles,
// chunks and threads, so each step's dL/domega is bitwise theirs while the
// reverse kernel itself runs shallower chunks that fill the chip.  Step s =
// blockIdx.y has its factors at x + s * n and its partials at partials + s *
// stride.  8 bytes read per node and step; few threads walk far, so each has 32
// loads in flight.
__global__ __launch_bounds__(NINT) void k_adj_dadomega(ProblemArgs p, int nzc,
                                                       const float2 *__restrict__ x,
                                                       double *__restrict__ partials, size_t stride)
{
    const TileIdx ti = tile_of_block(p.nx, p.ny, TX, TY);
    const size_t plane = (size_t)p.nx * p.ny;
    const size_t col = (size_t)(ti.y0 + (int)threadIdx.x / TX) * p.nx + ti.x0 + threadIdx.x % TX;
    const float2 *xs = x + (size_t)blockIdx.y * p.n;
    const int z0 = ti.zc * nzc, z1 = min(z0 + nzc, p.nz);
    constexpr int U = 32;
    float da = 0.0f;
    for (int z = z0; z < z1; z += U) {
        float2 v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = xs[(size_t)min(z + j, z1 - 1) * plane + col];
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (z + j < z1) da = fmaf(v[j].x, v[j].y, da);
    }
    double v[1] = {(double)da};
    store_block_partials<1>(v, partials + blockIdx.y * stride, blockIdx.x);
}

template <class T, bool MASK, bool FINAL, bool XOUT, bool PAIR>
void launch_t(const ProblemArgs &p, int c, unsigned nb, const T *st, const float *mu_in,
              float *mu_out, const unsigned *bits, const float4 *wallg, float2 *x,
              const ReduceArgs &r, hipStream_t s)
{
    if constexpr (!XOUT && !PAIR) {
        if (c < 8) {
            k_adj_march<T, 0, MASK, FINAL, XOUT, PAIR><<<nb, NTHREADS, 0, s>>>(p, c, st, mu_in, mu_out, bits, wallg, x, r);
            return;
        }
    }
    // a loop of c + 2 iterations, its tail 3 + (c + 2) % 3
    switch ((c + 2) % 3) {
    case 0: k_adj_march<T, 3, MASK, FINAL, XOUT, PAIR><<<nb, NTHREADS, 0, s>>>(p, c, st, mu_in, mu_out, bits, wallg, x, r); break;
    case 1: k_adj_march<T, 4, MASK, FINAL, XOUT, PAIR><<<nb, NTHREADS, 0, s>>>(p, c, st, mu_in, mu_out, bits, wallg, x, r); break;
    default: k_adj_march<T, 5, MASK, FINAL, XOUT, PAIR><<<nb, NTHREADS, 0, s>>>(p, c, st, mu_in, mu_out, bits, wallg, x, r); break;
    }
}

template <class T, bool FINAL>
void dispatch(const ProblemArgs &p, const void *state, const float *mu_in, float *mu_out,
              const unsigned *bits, const float4 *wallg, float2 *x, const ReduceArgs &r,
              hipStream_t s)
{
    const T *st = static_cast<const T *>(state);
    const int c = x ? adj_split_depth(p) : adj_depth(p);
    const unsigned nb = adj_blocks(p, c);
    if (x) {
        launch_t<T, false, FINAL, true, false>(p, c, nb, st, mu_in, mu_out, bits, wallg, x, r, s);
        return;
    }
    // one round of two workgroups a CU, a sixteenth of it or less empty
    const bool pair = c >= 8 && 8LL * nb > 15LL * p.ncu && nb <= 2LL * p.ncu;
    if (p.mask) {
        if (pair) launch_t<T, true, FINAL, false, true>(p, c, nb, st, mu_in, mu_out, bits, wallg, nullptr, r, s);
        else launch_t<T, true, FINAL, false, false>(p, c, nb, st, mu_in, mu_out, bits, wallg, nullptr, r, s);
    } else {
        if (pair) launch_t<T, false, FINAL, false, true>(p, c, nb, st, mu_in, mu_out, bits, wallg, nullptr, r, s);
        else launch_t<T, false, FINAL, false, false>(p, c, nb, st, mu_in, mu_out, bits, wallg, nullptr, r, s);
    }
}

}  // namespace

bool adj_march_supported(const ProblemArgs &p)
{
    return p.Q == 19 && p.nx >= TX && p.ny >= TY && p.nx % TX == 0 && p.ny % TY == 0 &&
           p.nz >= 1 && p.n < (1LL << 28);
}

// Chunk depth: 64 planes.  A thread sums its planes' dL/da in FP32, so the
// depth is part of the result and stays as it is on every grid; sweeps on
// grids that it leaves half empty go through adj_split_depth.
int adj_depth(const ProblemArgs &p) { return p.nz < 64 ? p.nz : 64; }

int adj_split_depth(const ProblemArgs &p)
{
    const int c = p.march_deep > 0 ? p.march_deep : p.march_nzc;
    return c < p.nz ? c : p.nz;
}

unsigned adj_blocks(const ProblemArgs &p, int nzc)
{
    return (unsigned)((long long)(p.nx / TX) * (p.ny / TY) * ((p.nz + nzc - 1) / nzc));
}

unsigned adj_march_num_blocks(const ProblemArgs &p)
{
    return adj_march_supported(p) ? adj_blocks(p, adj_depth(p)) : 0;
}

hipError_t launch_adj_dadomega(const ProblemArgs &p, int nzc, int nsteps, const float2 *x,
                               double *partials, size_t stride, hipStream_t s)
{
    if (!adj_march_supported(p) || p.mask || nsteps < 1) return hipErrorInvalidValue;
    k_adj_dadomega<<<dim3(adj_blocks(p, nzc), (unsigned)nsteps), NINT, 0, s>>>(p, nzc, x, partials,
                                                                               stride);
    return hipGetLastError();
}

hipError_t launch_adj_march(const ProblemArgs &p, int storage, const void *state,
                            const float *mu_in, float *mu_out, const unsigned *bits,
                            const float4 *wallg, int final_t0, const ReduceArgs &r,
                            hipStream_t stream, float2 *x)
{
    if (!adj_march_supported(p) || (p.mask && (!bits || x))) return hipErrorNotSupported;
    if (storage) {
        if (final_t0) dispatch<__half, true>(p, state, mu_in, mu_out, bits, wallg, x, r, stream);
        else dispatch<__half, false>(p, state, mu_in, mu_out, bits, wallg, x, r, stream);
    } else {
        if (final_t0) dispatch<float, true>(p, state, mu_in, mu_out, bits, wallg, x, r, stream);
        else dispatch<float, false>(p, state, mu_in, mu_out, bits, wallg, x, r, stream);
    }
    const hipError_t e = hipGetLastError();
    // r.out null: the caller adds the block partials itself (lwacm_adjoint_sweep)
    if (e != hipSuccess || !r.out) return e;
    return launch_reduce(r, 1, adj_march_num_blocks(p), stream);
}

}  // namespace lwacm
