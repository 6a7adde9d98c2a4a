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

constexpr int kMarchPoints = 4096;   // at most so many are injected by the marching workgroups

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
    if (A.march && A.ns == 1 && A.out[0]) {
        // every workgroup looks through the injected points
        const bool fused = A.inj.npts <= kMarchPoints;
        StepSide side;
        if (fused) {
            side.inj = &A.inj;
            side.vals = A.vals;
        }
        if (A.gmask) {
            side.gat = &A.gat;
            side.row = A.rows;
        }
        hipError_t rc = A.G ? launch_adj_step(g, A.u, A.up, A.out[0], A.w, A.uk[0], A.G, A.gscale, s, ev, nullptr,
                                              kGAdd, side)
                            : launch_fwd_step(g, A.u, A.up, A.out[0], A.w, s, ev, side);
        if (rc == hipSuccess && !fused)
            rc = launch_inject_res(g, A.inj, A.vals, A.w, A.out[0], A.uk[0], A.G, A.gscale, s);
        return rc;
    }
    for (int j = 0; j < A.ns; ++j)   // a tile's neighbours read what it writes over
        if (A.out[j] && (A.out[j] == A.u || A.out[j] == A.up)) return hipErrorInvalidValue;
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
    // a tile's neighbours read what it writes over
    const int32_t *out = op.kind == kOpAdj ? op.d : op.c;
    for (int j = 0; j < (op.kind == kOpAdj ? 2 : op.ns); ++j)
        if (out[j] != kBufNone && (out[j] == op.a || out[j] == op.b)) return hipErrorInvalidValue;
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

// Whether the steps of a call march one by one (stencil2d) instead of running in tiles, which a
// region's rim and its loads, no longer hidden behind each other, make slower on large grids, the
// wider the operator the sooner.  By the regions of one step a CU would get; microseconds a step,
// marched / in the best groups:
//   forward calls: order 10, 1200 x 900 points (1.9) 14.6 / 15.7; order 16, 1500 x 1200 (3.1)
//     22.7 / 27.0; order 8, 3000 x 2200 (8.4) 41.6 / 41.9 and 4000 x 3000 (15) 65.4 / 70.7; order 6,
//     4000 x 3000 64.3 / 64.0 and 6000 x 5000 (38) 146 / 166; orders 2 and 4 there 116 / 74 and
//     147 / 113.
//   gradients (a forward and an adjoint step): order 8, 4000 x 3000 167 / 164 and 6000 x 5000
//     396 / 416; order 6 there 396 / 353; order 10, 1500 x 1200 43.8 / 42.8, 2000 x 1500 (5.2)
//     57.5 / 61.6; order 16, 1200 x 900 43.4 / 35.4 and 1500 x 1200 51.9 / 55.0.
//   the adjoint of the source, whose every level is sampled, goes step by step: order 4, 250 x 200
//     (0.1) 13.4 / 14.8, 1200 x 900 (1.5) 17.6 / 20.2, 6000 x 5000 155 / 224; order 16, 552 x 552
//     (0.6) 19.0 / 15.6, 1500 x 1200 27.6 / 30.7.
bool tile2d_march(int K, int nx, int nz, int run)
{
    const int core = kTileRegion - 2 * tile2d_halo(K, 1);
    const double r = (double)((nx + core - 1) / core) * ((nz + core - 1) / core) / device_cus();
    if (run == kRunAdjointSrc) return K <= 4 || r > 1.0;
    if (K <= 2) return false;
    if (run == kRunForward) return r > (K == 3 ? 16.0 : (K == 4 ? 10.0 : 1.5));
    return K > 3 && r > (K == 4 ? 20.0 : (K <= 6 ? 4.0 : 2.5));
}

// Steps per group.  A group of ns steps costs a launch with its first regions, 5 + (0.9 + K / 6) ns
// us, and every further region that a CU gets 3.8 + (0.7 + K / 20) ns us (fitted to forward steps
// of orders 4, 8, 12 and 16 on 100 x 90 to 4000 x 3000 points, each at every ns; it picks the fastest
// ns or one within 5 % of it on all of them).  More steps mean a wider rim and so more regions.
int tile2d_choose(int K, int nx, int nz, int nshots)
{
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
