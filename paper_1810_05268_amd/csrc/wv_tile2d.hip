// Launches of the 2-D multi-step tiles (see wv_tile2d_dev.h), for one shot or a batch.
#include <hip/hip_ext.h>

#include "wv_tile2d_dev.h"

namespace wv {

namespace {

template <int K, bool GRAD>
__global__ __launch_bounds__(kTileThreads) void tile2d_kernel(const Grid g, const Tile2dArgs A, int tiles_x,
                                                              int tiles_z)
{
    __shared__ __align__(16) Tile2dShared<K> S;
    const int lid = xcd_remap(blockIdx.x, tiles_x * tiles_z);
    tile2d<K, GRAD>(g, A, lid % tiles_x, lid / tiles_x, S);
}

template <int K>
hipError_t launch_k(const Grid &g, const Tile2dArgs &A, hipStream_t s, LaunchEvents ev)
{
    const int core = kTileRegion - 2 * tile2d_halo(K, A.ns);
    const int tx = (g.nx + core - 1) / core, tz = (g.nz + core - 1) / core;
    auto go = [&](auto kern) {
        const dim3 grid(tx * tz), wg(kTileThreads);
        if (ev.start) hipExtLaunchKernelGGL(kern, grid, wg, 0, s, ev.start, ev.stop, 0, g, A, tx, tz);
        else hipLaunchKernelGGL(kern, grid, wg, 0, s, g, A, tx, tz);
    };
    if (A.G) go(tile2d_kernel<K, true>);
    else go(tile2d_kernel<K, false>);
    return hipGetLastError();
}

// The same steps of every shot of a batch (blockIdx.y).
template <int K, bool GRAD>
__global__ __launch_bounds__(kTileThreads) void tile2d_batch_kernel(const BatchArgs A, const BatchOp op,
                                                                    int tiles_x, int tiles_z)
{
    __shared__ __align__(16) Tile2dShared<K> S;
    const int lid = xcd_remap(blockIdx.x, tiles_x * tiles_z);
    const ShotTile<GRAD> T(A, A.shots[blockIdx.y], op, A.g.P);
    tile2d<K, GRAD>(A.g, T, lid % tiles_x, lid / tiles_x, S);
}

template <int K>
hipError_t launch_batch_k(const BatchArgs &A, const BatchOp &op, hipStream_t s)
{
    const int core = kTileRegion - 2 * tile2d_halo(K, op.ns);
    const int tx = (A.g.nx + core - 1) / core, tz = (A.g.nz + core - 1) / core;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(tx * tz, A.nshots), dim3(kTileThreads), 0, s, A, op, tx, tz);
    };
    if (op.kind == kOpAdj) go(tile2d_batch_kernel<K, true>);
    else go(tile2d_batch_kernel<K, false>);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_tile2d(const Grid &g, const Tile2dArgs &A, hipStream_t s, LaunchEvents ev)
{
    if (g.ndim != 2 || A.ns < 1 || A.ns > tile2d_steps(g.K)) return hipErrorInvalidValue;
    if (A.ns == 1 && A.out[0] && tile2d_march(g.K, g.nx, g.nz)) {
        hipError_t rc = A.gmask ? launch_gather(A.gat, A.u, A.rows, s) : hipSuccess;
        if (rc == hipSuccess)
            rc = A.G ? launch_adj_step(g, A.u, A.up, A.out[0], A.w, A.uk[0], A.G, A.gscale, s, ev, nullptr, kGAdd, {})
                     : launch_fwd_step(g, A.u, A.up, A.out[0], A.w, s, ev, {});
        if (rc == hipSuccess) rc = launch_inject_res(g, A.inj, A.vals, A.w, A.out[0], A.uk[0], A.G, A.gscale, s);
        return rc;
    }
    switch (g.K) {
    case 1: return launch_k<1>(g, A, s, ev);
    case 2: return launch_k<2>(g, A, s, ev);
    case 3: return launch_k<3>(g, A, s, ev);
    case 4: return launch_k<4>(g, A, s, ev);
    case 5: return launch_k<5>(g, A, s, ev);
    case 6: return launch_k<6>(g, A, s, ev);
    case 7: return launch_k<7>(g, A, s, ev);
    case 8: return launch_k<8>(g, A, s, ev);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_batch_steps(const BatchArgs &A, const BatchOp &op, hipStream_t s)
{
    if ((op.kind != kOpStep && op.kind != kOpAdj) || op.ns < 1 || op.ns > tile2d_steps(A.g.K))
        return hipErrorInvalidValue;
    switch (A.g.K) {
    case 1: return launch_batch_k<1>(A, op, s);
    case 2: return launch_batch_k<2>(A, op, s);
    case 3: return launch_batch_k<3>(A, op, s);
    case 4: return launch_batch_k<4>(A, op, s);
    case 5: return launch_batch_k<5>(A, op, s);
    case 6: return launch_batch_k<6>(A, op, s);
    case 7: return launch_batch_k<7>(A, op, s);
    case 8: return launch_batch_k<8>(A, op, s);
    default: return hipErrorInvalidValue;
    }
}

int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return 256;
    return cus;
}

// Whether a shot's steps are marched one by one (stencil2d) instead: for operators wider than
// order 8 on grids of more than 4 regions a CU, where a region's rim is most of it and its
// loads are no longer hidden.  At order 16 on 4000 x 3000 points a forward step takes 112 us in
// tiles and 76 marched, on 2000 x 1500 an adjoint one 61 and 43 (a forward one 31 either way);
// at order 8 tiles are faster on both (66 and 74 us, 19 and 28).
bool tile2d_march(int K, int nx, int nz)
{
    const int core = kTileRegion - 2 * tile2d_halo(K, 1);
    return K > 4 && (long long)((nx + core - 1) / core) * ((nz + core - 1) / core) > 4LL * device_cus();
}

// Steps per group.  A group of ns steps costs a launch with its first regions, 5 + (0.9 + K / 6) ns
// us, and every further region that a CU gets 3.8 + (0.7 + K / 20) ns us (fitted to forward steps
// of orders 4, 8, 12 and 16 on 100 x 90 to 4000 x 3000 points, each at every ns; it picks the fastest
// ns or one within 5 % of it on all of them).  More steps mean a wider rim and so more regions.
int tile2d_choose(int K, int nx, int nz, int nshots)
{
    if (nshots == 1 && tile2d_march(K, nx, nz)) return 1;
    const int cus = device_cus();
    int best = 1;
    double best_t = 0.0;
    for (int ns = 1; ns <= tile2d_steps(K); ++ns) {
        const int core = kTileRegion - 2 * tile2d_halo(K, ns);
        const long long n = (long long)((nx + core - 1) / core) * ((nz + core - 1) / core) * nshots;
        const double r = (double)((n + cus - 1) / cus);
        const double t = (5.0 + (0.9 + K / 6.0) * ns + (r - 1.0) * (3.8 + (0.7 + 0.05 * K) * ns)) / ns;
        if (ns == 1 || t < best_t) {
            best = ns;
            best_t = t;
        }
    }
    return best;
}

}  // namespace wv
