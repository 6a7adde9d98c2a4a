// How the planes of a 3-D grid are split over the workgroups of a stencil launch.  Host only.
#pragma once

#include <algorithm>
#include <cmath>

namespace wv {

// Planes of a chunk, for `tiles` 32 x 32 tiles a plane and a kernel of which per_cu workgroups
// fit a CU.  A workgroup reads the 2K + 1 planes of its queue together, and then marches its
// chunk; what counts is how many workgroups a CU gets, r = ceil(workgroups / CUs), not whether
// they all fit at once.  Counted in planes marched, a CU with r workgroups that are resident
// together takes max(r, 2.05) zlen (two marches hide each other's latency, more share its
// throughput; 2.03 at orders 2 and 4, where three are about even with two) and for their starts
// 0.7 (2K + 1) sqrt(r) + 0.4 r (0.8 r at order 2); a plane of a step with a gradient is twice the
// traffic, so that 1.3 marches fill a CU and a start counts half.  The least of that over all
// chunk counts.
// Fitted to 47 grids of 24^3 to 400^3 points, cubes and slabs, at orders 2 to 16, each at up to
// 16 chunk lengths: within 0.7 % of the best of them on average.  On 170 other grids 12 kernels of
// 2040 take over 3 % longer than with chunks that fill the resident workgroups once and hold at
// least 4K planes, most of them forward steps at order 2.  An earlier fit, to 168^3 and 200^3
// points at order 8 and 296^3 at order 12, weighed starts three times as much: where the chunks
// differ, kernels take 7 % less on average.  Microseconds a forward / adjoint step:
//                             filled once    earlier fit    this
//   168^3, order 8            27.1 / 42.0    22.8 / 34.4    22.8 / 34.5
//   168^3, order 16           45.0 / 53.1    34.4 / 40.9    26.6 / 35.7
//   183 x 139 x 125, 12       31.4 / 39.1    22.9 / 27.6    19.0 / 25.9
//   300 x 40 x 480, order 4   26.2 / 42.5    28.3 / 48.2    26.4 / 42.5
//   296^3, order 12           92.1 / 177     92.2 / 178     91.7 / 177
inline int chunks3d(long long tiles, int nz, int K, bool grad, int per_cu, int cus)
{
    double best = 0.0;
    int zlen = 0;
    // each length that some chunk count has, the longest first: about 2 sqrt(nz) of them (this
    // runs at every launch: all counts of 1000 planes took 9 us, against 17 us of such a step)
    for (int zl = nz; zl >= 1;) {
        const int n = (nz + zl - 1) / zl;
        const long long r = (tiles * n + cus - 1) / cus;
        auto cost = [&](long long c) {
            const double start = 0.7 * (2 * K + 1) * std::sqrt((double)c) + (K == 1 ? 0.8 : 0.4) * (double)c;
            return c ? std::max((double)c, grad ? 1.3 : (K <= 2 ? 2.03 : 2.05)) * zl + (grad ? 0.5 : 1.0) * start : 0.0;
        };
        const double t = (double)(r / per_cu) * cost(per_cu) + cost(r % per_cu);
        if (!zlen || t < best) {
            best = t;
            zlen = zl;
        }
        if (zl == 1 || r > 8LL * per_cu) break;          // only more starts from here
        const int zc = (nz + zl - 2) / (zl - 1);         // the least count with shorter chunks
        zl = (nz + zc - 1) / zc;
    }
    return zlen;
}

}  // namespace wv
