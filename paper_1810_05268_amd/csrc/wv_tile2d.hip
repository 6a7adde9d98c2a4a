// Launches of the 2-D multi-step tiles (see wv_tile2d_dev.h), for one shot or a batch.
#include <hip/hip_ext.h>

#include "wv_tile2d_dev.h"

namespace wv {

namespace {

template <int K, bool GRAD>
__global__ __launch_bounds__(kTileThreads) void tile2d_kernel(const Grid g, const Tile2dArgs A, int tiles_x,
                                                              int tiles_z)
{
    __shared__ __align__(16) Tile2dShared S;
    __shared__ __align__(16) typename Tile2dShared::template Levels<K> L;
    const int lid = xcd_remap(blockIdx.x, tiles_x * tiles_z);
    tile2d<K, GRAD>(g, A, lid % tiles_x, lid / tiles_x, S, L);
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
    __shared__ __align__(16) Tile2dShared S;
    __shared__ __align__(16) typename Tile2dShared::template Levels<K> L;
    const int lid = xcd_remap(blockIdx.x, tiles_x * tiles_z);
    const ShotTile<GRAD> T(A, A.shots[blockIdx.y], op, A.g.P);
    tile2d<K, GRAD>(A.g, T, lid % tiles_x, lid / tiles_x, S, L);
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

// A group of ns steps costs a launch and its loads, about 4 us, and ns times the work of the
// regions a CU gets, r = ceil(regions / CUs): (0.8 + K / 4) us for one, three quarters of that
// for each of several (measured at orders 4, 8 and 16 on 141^2 and 552^2 points; in a batch
// a device-wide barrier stands for the launch).  More steps mean a wider rim and so more
// regions; the least time per step over the counts a region allows.
int tile2d_choose(int K, int nx, int nz, int nshots)
{
    const int cus = device_cus();
    const double start = nshots > 1 ? 8.0 : 4.0;
    int best = 1;
    double best_t = 0.0;
    for (int ns = 1; ns <= tile2d_steps(K); ++ns) {
        const int core = kTileRegion - 2 * tile2d_halo(K, ns);
        const long long n = (long long)((nx + core - 1) / core) * ((nz + core - 1) / core) * nshots;
        const double r = (double)((n + cus - 1) / cus);
        const double t = start / ns + (0.8 + 0.25 * K) * (r > 1.0 ? 0.75 * r : 1.0);
        if (ns == 1 || t < best_t) {
            best = ns;
            best_t = t;
        }
    }
    return best;
}

}  // namespace wv
