// resident.hip -- lattices of at most kResidentNodes nodes: every step of a
// call in one launch.
//
// Such a lattice keeps one launch per step busy for a few wavefronts' worth of
// work, and its time is the launch's and the serial chain of memory round
// trips in it.  Here one workgroup holds the whole lattice in LDS, one node
// per thread, and advances it any number of steps: a node pulls its
// populations from LDS, forms its moments, exchanges Phi with its neighbours
// through LDS, collides and writes its populations back -- two barriers per
// step and no global memory between the first step and the last.  The nodes'
// pull sources (periodic wrap, bounce-back from the link code) are LDS indices
// formed once per launch.  The state returns to the lattice it came from.
// Every node's arithmetic is the one-step sweep's on the values that sweep
// would store and load back, so the bits are the same.
//
// Bound: the dependent chain of one update (about 180 operations and two LDS
// round trips) while the nodes fill at most a wavefront per SIMD, then the one
// CU's issue rate.  Measured, us per step, against the best one-step launches
// (one-row blocks): FP64 4 x 34 0.58 / 3.3, 16 x 16 0.58 / 3.4, 32 x 32 1.33 /
// 3.3; FP32 0.48, 0.49, 0.79 / 3.05; FP16 0.50, 0.50, 0.88 / 3.1.  The ten
// 4 x 34 channels of a slip study, 200 steps and ten velocity changes: 447
// against 1173 us.
#include "wave.hpp"

namespace trt {

namespace {

constexpr int kEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int kEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// MAXN: the most nodes (and threads) of the variant.
template <int ST, int MAXN>
__device__ __forceinline__ void resident_steps(const InstDesc &d, int srcsel, int64_t steps) {
    using T = typename Store<ST>::T;
    using C = typename Store<ST>::C;
    constexpr bool SH = Store<ST>::shifted;
    __shared__ C pops[9 * MAXN];
    __shared__ C phis[2 * MAXN];

    const int nx = d.nx, ny = d.ny, n = nx * ny;
    const int t = threadIdx.x;
    const bool live = t < n;  // the others only meet the barriers
    const int node = live ? t : 0;
    const int y = node / nx, x = node - y * nx;
    T *lat = static_cast<T *>(srcsel ? d.buf[1] : d.buf[0]);
    T *own = lat + (int64_t)y * d.pitch + x;
    const uint32_t code =
        d.links ? d.links[(int64_t)y * d.lpitch + x] : 0u;  // solid, bounced pulls
    const bool solid = (code & 1u) != 0;

    const auto wrap = [](int v, int m) { return v < 0 ? v + m : (v >= m ? v - m : v); };
    // LDS indices of the pulls and of the neighbours' Phi
    int from[9];
    from[0] = node;
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const int s = wrap(y - kEy[i], ny) * nx + wrap(x - kEx[i], nx);
        from[i] = ((code >> i) & 1u) ? kOppDir[i] * MAXN + node : i * MAXN + s;
    }
    const int left = y * nx + wrap(x - 1, nx), right = y * nx + wrap(x + 1, nx);
    const int below = wrap(y - 1, ny) * nx + x, above = wrap(y + 1, ny) * nx + x;

    const C gx = uniform((C)d.gx), gy = uniform((C)d.gy);
    const C w1 = uniform((C)d.omega1), w2 = uniform((C)d.omega2), ph = uniform((C)d.phi);
    const bool open = d.xbc != 0;
    const C u_in = (C)d.u_in, rho_in = (C)d.rho_in, rho_out = (C)d.rho_out;
    const C phi_wall = rho_in * u_in * u_in * u_in;

    if (live) {
#pragma unroll
        for (int i = 0; i < 9; ++i) pops[i * MAXN + node] = to_c(own[i * d.plane]);
    }
    __syncthreads();
    for (int64_t k = 0; k < steps; ++k) {
        Moments<C, SH> m;
        C phix = C(0);
        if (live) {
            C f[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = pops[from[i]];
            if (open) open_x_fix<C, SH>(f, x, nx, u_in, rho_in, rho_out);
            m.compute(f, gx, gy);
            const C px = m.rho * m.ux * m.ux * m.ux;
            const C py = m.rho * m.uy * m.uy * m.uy;
            phix = solid ? C(0) : px;
            phis[node] = phix;
            phis[MAXN + node] = solid ? C(0) : py;
        }
        __syncthreads();  // every pull is done, every Phi written
        if (live) {
            C pl = phis[left], pr = phis[right];
            if (open) {
                if (x == 0) pl = phi_wall;
                if (x == nx - 1) pr = phix;
            }
            const C dphix = C(0.5) * (pr - pl);
            const C dphiy = C(0.5) * (phis[MAXN + above] - phis[MAXN + below]);
            const Coeffs<C> c = collide_coeffs<C, SH>(m, dphix, w1, w2, ph, gx, gy);
            C o[9];
            if constexpr (ST == ST_F16) {
                HalfPairs p;
                reconstruct_pairs(p, c.base, c.bx, c.by, c.bxx, c.byy - ph * dphiy, c.bxy, c.bxxy,
                                  c.bxyy);
                uint32_t h[9] = {half_out<0, false>(p), half_out<1, false>(p),
                                 half_out<2, false>(p), half_out<3, false>(p),
                                 half_out<4, false>(p), half_out<5, false>(p),
                                 half_out<6, false>(p), half_out<7, false>(p),
                                 half_out<8, false>(p)};
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    o[i] = (float)__builtin_bit_cast(_Float16, (unsigned short)(h[i] & 0xffffu));
            } else {
                reconstruct<C>(o, c.base, c.bx, c.by, c.bxx, c.byy - ph * dphiy, c.bxy, c.bxxy,
                               c.bxyy);
            }
            // a solid node's slots are never read; they keep zeros
#pragma unroll
            for (int i = 0; i < 9; ++i) pops[i * MAXN + node] = solid ? C(0) : o[i];
        }
        __syncthreads();  // every population written, every Phi read
    }
    if (live) {
#pragma unroll
        for (int i = 0; i < 9; ++i) own[i * d.plane] = (T)pops[i * MAXN + node];
    }
}

template <int ST, int MAXN>
__global__ __launch_bounds__(MAXN) void resident_kernel(InstDesc d, int srcsel, int64_t steps) {
    resident_steps<ST, MAXN>(d, srcsel, steps);
}

// Batched: workgroup b advances member members[b] of the table; a member
// advanced here stays on the lattice it was on when the table was built.
template <int ST, int MAXN>
__global__ __launch_bounds__(MAXN) void resident_batch_kernel(const InstDesc *__restrict__ descs,
                                                             const int4 *__restrict__ members,
                                                             int64_t steps) {
    const InstDesc d = descs[members[blockIdx.x].x];
    resident_steps<ST, MAXN>(d, d.cur, steps);
}

// one launch's steps: a call of many is cut so that a launch stays short
// (about 10 ms)
constexpr int64_t kLaunchSteps = 8192;

template <int ST, int MAXN>
hipError_t launch_t(const InstDesc *one, const InstDesc *descs, const int4 *members, int n, int src,
                    int64_t steps, hipStream_t s) {
    while (steps > 0) {
        const int64_t k = steps < kLaunchSteps ? steps : kLaunchSteps;
        if (one)
            resident_kernel<ST, MAXN><<<1, MAXN, 0, s>>>(*one, src, k);
        else
            resident_batch_kernel<ST, MAXN><<<n, MAXN, 0, s>>>(descs, members, k);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        steps -= k;
    }
    return hipSuccess;
}

template <int ST>
hipError_t launch_n(int nodes, const InstDesc *one, const InstDesc *descs, const int4 *members,
                    int n, int src, int64_t steps, hipStream_t s) {
    // as few threads as hold the nodes: idle ones would still meet every barrier
    if (nodes <= 128) return launch_t<ST, 128>(one, descs, members, n, src, steps, s);
    if (nodes <= 256) return launch_t<ST, 256>(one, descs, members, n, src, steps, s);
    if (nodes <= 512) return launch_t<ST, 512>(one, descs, members, n, src, steps, s);
    return launch_t<ST, 1024>(one, descs, members, n, src, steps, s);
}

hipError_t launch_s(int storage, int nodes, const InstDesc *one, const InstDesc *descs,
                    const int4 *members, int n, int src, int64_t steps, hipStream_t s) {
    if (nodes < 1 || nodes > kResidentNodes) return hipErrorInvalidValue;
    switch (storage) {
        case ST_F64: return launch_n<ST_F64>(nodes, one, descs, members, n, src, steps, s);
        case ST_F32: return launch_n<ST_F32>(nodes, one, descs, members, n, src, steps, s);
        case ST_F16: return launch_n<ST_F16>(nodes, one, descs, members, n, src, steps, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_resident(const InstDesc &d, int storage, int src, int64_t steps,
                           hipStream_t stream) {
    if ((int64_t)d.nx * d.ny > kResidentNodes) return hipErrorInvalidValue;
    return launch_s(storage, d.nx * d.ny, &d, nullptr, nullptr, 0, src, steps, stream);
}

hipError_t launch_resident_batch(const InstDesc *descs, const int4 *members, int n, int most_nodes,
                                 int storage, int64_t steps, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    return launch_s(storage, most_nodes, nullptr, descs, members, n, 0, steps, stream);
}

}  // namespace trt
