// Several 2-D OT2 steps in one pass over a tile, shared by the solo launches and the
// batched solver (one definition, so that a shot gives the same bits either way).
//
// A 2-D field is a few MB, so a step launched by itself is bound by latency: the launch, a
// workgroup's first loads and its march down the rows (7.1 us a forward step on 552^2 points
// at order 8, 0.7 us of which its bytes need; 8.7 us an adjoint step).  Three steps in tiles
// take 8.5 and 9.9 us, over half of it arithmetic.  Here a workgroup takes a 64 x 64 region of
// the grid into LDS and its registers and advances it by up to kTileSteps(K) steps; each
// step makes K more rows and columns at the region's rim invalid, and the core that is left
// is written.  The rim is computed by the neighbouring workgroups too (with 4 steps of order
// 8 a core of 32 x 32: twice the arithmetic), which costs less than a launch per step.
//   * A lane owns 4 points of a row (16 waves, one region a CU at a time): the two levels are in
//     LDS (a step overwrites the older one, each lane its own points: one barrier a step), w and
//     the damping in registers; a step reads 1 + 2K rows of 16 bytes for the z neighbours of its
//     points and 2 ceil(K/4) more for the x neighbours.  More rows a lane read less, but leave
//     fewer waves, whose latency shows: three forward steps (196 regions) take 9.5 us with one
//     row a lane, 11.8 with two, 15.2 with four, and an adjoint group of eight such shots 47 with
//     one and 84 with two, which spill.
//   * A region is bound by latency (its loads, then a chain of steps) and by the set-up of its
//     lanes.  Regions inside the grid and its absorbing layer skip the damping and the masks
//     (4 to 10 % of a step from 100 x 90 to 4000 x 3000 points); a persistent workgroup that loads
//     its next region ahead took 7 % longer with one region a CU and 2 to 10 % less with many.
//   * Injected samples are summed before the steps, for all of them, by the lanes that find the
//     points, while the fields load; each step's go to one of two LDS planes of the region a step
//     ahead, and the owner of a point adds its own in the step's order (the
//     binary64 gradient too), so results do not depend on how steps are grouped.
//   * Divisions by 1 + a (in the absorbing layer) multiply by the reciprocal, formed once a
//     region, and correct twice, which rounds as the division does (5 operations for 13);
//     waves whose points all lie outside the layer have none.
//   * Points outside the grid hold zeros and have w = 0, so they stay zero (but for a field that
//     is no longer finite, which the caller refuses).
//   * Receivers are read from the LDS level: those whose first corner lies in the core.
#pragma once

#include "wv_stencil_dev.h"

namespace wv {

namespace {

constexpr int kTileEX = kTileRegion, kTileEY = kTileRegion;
constexpr int kTileThreads = 16 * kTileRegion;
constexpr int kTileCap = 256;                // injected points and receivers of a region kept in LDS

// A workgroup's LDS.  All of it stays under half a CU's: not for a second workgroup, but because
// the compiler takes less to mean that registers are free, and spills at K >= 6.
template <int K>
struct Tile2dShared {
    // two levels of the region with a guard rim for the lanes at its edge, whose results
    // are not used
    float u[2][kTileEY + 2 * K][kTileEX + 2 * ((K + 3) & ~3)];
    // the summed samples of a step and of the next one, 0 where there is no point, of the rows
    // that are stepped at all
    float inj[2][kTileEY - 2 * K][kTileEX];
    float val[tile2d_steps(K)][kTileCap];    // those of the listed points for every step,
    int loc[kTileCap];                       // and the points' places in a plane of inj
    int rec[kTileCap];
    int n, nrec;
};
static_assert(sizeof(Tile2dShared<1>) <= 81920 && sizeof(Tile2dShared<2>) <= 81920 &&
              sizeof(Tile2dShared<5>) <= 81920 && sizeof(Tile2dShared<8>) <= 81920);

// n[i] / b[i], r the binary32 reciprocals of b (b >= 1: 1 + a, at most 8.4 in the corners of a
// layer one cell thick).  The first correction leaves less than an ulp and the second rounds
// correctly, as long as the remainders are exact and nothing overflows: for |n| below 2^-100 they
// may not be, and a wave with such a value divides (a long run is sensitive to a single bit: the
// smallest values are those ahead of a wavefront, which grow by many orders).
__device__ __forceinline__ void div4(const float *n, const float *b, const float *r, float *q)
{
#pragma clang fp contract(off)
    unsigned least = ~0u;      // of the magnitudes, 0 taken as the largest
#pragma unroll
    for (int i = 0; i < 4; ++i) least = min(least, (__float_as_uint(n[i]) << 1) - 1u);
    if (__any(least < (__float_as_uint(0x1p-100f) << 1) - 1u)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = n[i] / b[i];
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float t = n[i] * r[i];
            t = fmaf(fmaf(-t, b[i], n[i]), r[i], t);
            q[i] = fmaf(fmaf(-t, b[i], n[i]), r[i], t);
        }
    }
}

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length: 4-byte aligned
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// 4 values of row z from column x on (inside the grid).  x is a multiple of 4, so only a row's
// last lane straddles its end; it reads on into the next row (after the last row, into the
// workspace behind the array, which is padded).
__device__ __forceinline__ f4u tile_load4(const Grid &g, const float *f, int x, int z)
{
    return *reinterpret_cast<const f4u *>(f + (long long)z * g.nx + x);
}

// As tile_load4 for the caller's gradient, behind which nothing may be read: the last lane
// of a row reads its last four values and moves them down (grids under 4 wide: one by one).
__device__ __forceinline__ void tile_load_grad(const Grid &g, const double *f, int gx, int gz, double *v)
{
    const double *row = f + (long long)gz * g.nx;
    if (g.nx < 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = row[min(gx + i, g.nx - 1)];
        return;
    }
    const int x = min(gx, g.nx - 4), sh = gx - x;
    const d2u a = *reinterpret_cast<const d2u *>(row + x), b = *reinterpret_cast<const d2u *>(row + x + 2);
    const double t0 = sh & 1 ? a.y : a.x, t1 = sh & 1 ? b.x : a.y, t2 = sh & 1 ? b.y : b.x, t3 = b.y;
    v[0] = sh & 2 ? t2 : t0;
    v[1] = sh & 2 ? t3 : t1;
    v[2] = t2;
    v[3] = t3;
}

// Region (tix, tiz) of the steps A describes (a Tile2dArgs, or a view of a batched shot with
// the same members); every lane of the kTileThreads calls it.
template <int K, bool GRAD, typename Args>
__device__ __forceinline__ void tile2d(const Grid &g, const Args &A, int tix, int tiz, Tile2dShared<K> &S)
{
#pragma clang fp contract(off)
    constexpr int HXK = (K + 3) & ~3;
    constexpr int NXV = 1 + 2 * (HXK / 4);
    constexpr int NT = kTileThreads;
    static_assert(NT >= kTileCap, "a lane per listed point");
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int nx = g.nx, nz = g.nz, ns = A.ns;
    const int H = tile2d_halo(K, ns), C = kTileEX - 2 * H;     // rim and core (both axes)
    const int gx0 = tix * C - H, gz0 = tiz * C - H;
    const int gx = gx0 + 4 * tx, gz = gz0 + ty;
    const bool core = tx >= H / 4 && tx < (H + C) / 4 && ty >= H && ty < H + C;
    // Where a lane loads from: its points, moved into the grid and into what is needed of an
    // array, the region less a rim (u: none, u^{n-1} and w: K, the gradient and its states: H).
    // So no load has a branch and all of a lane's are in flight together, and lanes outside
    // repeat addresses of lanes inside.  What lies outside the grid is zeroed below; an array's
    // rim is not used.
    auto xin = [&](int rim) {
        return min(max(gx, max(gx0 + (rim & ~3), 0)), min(gx0 + kTileEX - 4 - (rim & ~3), (nx - 1) & ~3));
    };
    auto zin = [&](int rim) { return min(max(gz, max(gz0 + rim, 0)), min(gz0 + kTileEY - 1 - rim, nz - 1)); };

    f4u un = tile_load4(g, A.u, xin(0), zin(0));
    f4u up = tile_load4(g, A.up, xin(K), zin(K));
    f4u w4 = tile_load4(g, A.w, xin(K), zin(K));
    double G[4];
    if constexpr (GRAD) tile_load_grad(g, A.G, xin(H), zin(H), G);
    // regions that reach out of the grid or into its absorbing layer
    const bool edge = gx0 < max(g.ix0[0], 0) || gx0 + kTileEX - 1 > min(g.ix1[0], nx - 1) ||
                      gz0 < max(g.ix0[2], 0) || gz0 + kTileEY - 1 > min(g.ix1[2], nz - 1);
    if (tid == 0) S.n = S.nrec = 0;
    __syncthreads();
    // injected points of the region and receivers of the core
    for (int i = tid; i < A.inj.npts; i += NT) {
        const int p = A.inj.s_pts[i], q0 = A.inj.s_start[i], q1 = A.inj.s_start[i + 1];
        const int z = p / nx, lx = p - z * nx - gx0, lz = z - gz0;
        if (lx < 0 || lx >= kTileEX || lz < K || lz >= kTileEY - K) continue;
        const int e = atomicAdd(&S.n, 1);
        if (e >= kTileCap) continue;
        float v[tile2d_steps(K)];
#pragma unroll
        for (int j = 0; j < tile2d_steps(K); ++j) v[j] = 0.0f;
        for (int q = q0; q < q1; ++q) {   // as scatter_sum, all steps at once
            const float wt = A.inj.s_wt[q];
            const float *f = A.vals + A.inj.s_col[q];
#pragma unroll
            for (int j = 0; j < tile2d_steps(K); ++j) v[j] = fmaf(wt, f[min(j, ns - 1) * A.vstride], v[j]);
        }
        S.loc[e] = (lz - K) * kTileEX + lx;
#pragma unroll
        for (int j = 0; j < tile2d_steps(K); ++j) S.val[j][e] = v[j];
    }
    if (!GRAD && A.gmask) {
        for (int i = tid; i < A.gat.n; i += NT) {
            const int p = A.gat.g_idx[i * A.gat.nc];
            const int z = p / nx, lx = p - z * nx - gx0, lz = z - gz0;
            if (lx < H || lx >= H + C || lz < H || lz >= H + C) continue;
            const int e = atomicAdd(&S.nrec, 1);
            if (e < kTileCap) S.rec[e] = i;
        }
    }
    // u^n and u^{n-1} go to LDS; w and the damping (1 - a, 1 + a, 1 / (1 + a)) stay
    float wr[4], am[4], ap[4], rp[4];
    bool damp = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        wr[i] = w4[i];
        am[i] = ap[i] = 1.0f;
    }
    if (edge) {
        const bool zok = (unsigned)gz < (unsigned)nz;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = zok & ((unsigned)(gx + i) < (unsigned)nx);
            const float a0 = damping(g, gx + i, 0, gz);
            const float a = in ? a0 : 0.0f;
            un[i] = in ? un[i] : 0.0f;
            up[i] = in ? up[i] : 0.0f;
            wr[i] = in ? wr[i] : 0.0f;
            damp |= a != 0.0f;
            am[i] = 1.0f - a;
            ap[i] = 1.0f + a;
        }
    }
    *reinterpret_cast<float4 *>(&S.u[0][ty + K][4 * tx + HXK]) = make_float4(un[0], un[1], un[2], un[3]);
    *reinterpret_cast<float4 *>(&S.u[1][ty + K][4 * tx + HXK]) = make_float4(up[0], up[1], up[2], up[3]);
    __syncthreads();
    const int ninj = S.n, nrec = S.nrec;
    const bool damped = __any(damp);
    // step j's samples go to its plane (the same places every step)
    const bool listed = ninj <= kTileCap;
    auto place = [&](int j) {
        float *plane = &S.inj[j & 1][0][0];
        if (listed) {
            if (tid < ninj) plane[S.loc[tid]] = S.val[j][tid];
        } else {
            for (int i = tid; i < A.inj.npts; i += NT) {
                const int p = A.inj.s_pts[i];
                const int z = p / nx, lx = p - z * nx - gx0, lz = z - gz0;
                if (lx >= 0 && lx < kTileEX && lz >= K && lz < kTileEY - K)
                    plane[(lz - K) * kTileEX + lx] = scatter_sum(A.inj, i, A.vals + j * A.vstride);
            }
        }
    };
    if (ninj) {
        if (ty >= K && ty < kTileEY - K) {
            const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            *reinterpret_cast<float4 *>(&S.inj[0][ty - K][4 * tx]) = zero;
            *reinterpret_cast<float4 *>(&S.inj[1][ty - K][4 * tx]) = zero;
        }
        __syncthreads();
        place(0);
        __syncthreads();
    }
    if (damped) {
#pragma unroll
        for (int i = 0; i < 4; ++i) rp[i] = 1.0f / ap[i];
    }
    // the lane's receiver: its corners' places in the region and their weights
    int goff[4] = {0, 0, 0, 0};
    float gwt[4] = {0.f, 0.f, 0.f, 0.f};
    const int rr = (!GRAD && nrec <= kTileCap && tid < nrec) ? S.rec[tid] : -1;
    if (rr >= 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c < A.gat.nc) {
                const int p = A.gat.g_idx[rr * A.gat.nc + c];
                const int z = p / nx;
                goff[c] = (z - gz0 + K) * (kTileEX + 2 * HXK) + p - z * nx - gx0 + HXK;
                gwt[c] = A.gat.g_wt[rr * A.gat.nc + c];
            }
    }

#pragma unroll 1
    for (int j = 0; j < ns; ++j) {
        const int cur = j & 1;
        if (ninj && j + 1 < ns) place(j + 1);
        if (!GRAD && (A.gmask >> j & 1)) {
            const float *lev = &S.u[cur][0][0];
            float *row = A.rows + (long long)j * A.gat.n;
            if (nrec <= kTileCap) {
                if (rr >= 0) {
                    float s = 0.0f;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (c < A.gat.nc) s = fmaf(gwt[c], lev[goff[c]], s);
                    row[rr] = s;
                }
            } else {
                for (int i = tid; i < A.gat.n; i += NT) {
                    const int p0 = A.gat.g_idx[i * A.gat.nc];
                    const int z0 = p0 / nx, lx0 = p0 - z0 * nx - gx0, lz0 = z0 - gz0;
                    if (lx0 < H || lx0 >= H + C || lz0 < H || lz0 >= H + C) continue;
                    float s = 0.0f;
                    for (int c = 0; c < A.gat.nc; ++c) {
                        const int p = A.gat.g_idx[i * A.gat.nc + c];
                        const int z = p / nx;
                        s = fmaf(A.gat.g_wt[i * A.gat.nc + c], S.u[cur][z - gz0 + K][p - z * nx - gx0 + HXK], s);
                    }
                    row[i] = s;
                }
            }
        }
        const int m = K * (j + 1);     // the rim that is invalid after this step
        if (ty >= m && ty < kTileEY - m && 4 * tx + 4 > m && 4 * tx < kTileEX - m) {
            f4u uk;      // used in the core only
            if constexpr (GRAD) uk = tile_load4(g, A.level(j), xin(H), zin(H));
            float q[4][1 + 2 * K];
#pragma unroll
            for (int r = 0; r < 1 + 2 * K; ++r) {
                const float4 t = *reinterpret_cast<const float4 *>(&S.u[cur][ty + r][4 * tx + HXK]);
                q[0][r] = t.x; q[1][r] = t.y; q[2][r] = t.z; q[3][r] = t.w;
            }
            float xr[4 * NXV];
#pragma unroll
            for (int v = 0; v < NXV; ++v) {
                if (v == HXK / 4) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) xr[4 * v + i] = q[i][K];
                } else {
                    const float4 t = *reinterpret_cast<const float4 *>(&S.u[cur][ty + K][4 * tx + 4 * v]);
                    xr[4 * v] = t.x; xr[4 * v + 1] = t.y; xr[4 * v + 2] = t.z; xr[4 * v + 3] = t.w;
                }
            }
            // the level before is the lane's own in the other buffer, about to be overwritten
            const float4 p4 = *reinterpret_cast<const float4 *>(&S.u[cur ^ 1][ty + K][4 * tx + HXK]);
            const float pv[4] = {p4.x, p4.y, p4.z, p4.w};
            float on[4], num[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float lap = lap2d<K>(g, q[i], &xr[HXK + i - K]);
                const float wl = wr[i] * lap;
                const float d = q[i][K] - pv[i];
                num[i] = damped ? fmaf(am[i], d, wl) : d + wl;   // (1 - 0) d + wl rounds as d + wl
                if constexpr (GRAD) G[i] = fma(A.gscale * (double)uk[i], (double)wl, G[i]);
            }
            if (damped) div4(num, ap, rp, num);
#pragma unroll
            for (int i = 0; i < 4; ++i) on[i] = q[i][K] + num[i];
            if (ninj) {
                const float4 s4 = *reinterpret_cast<const float4 *>(&S.inj[cur][ty - K][4 * tx]);
                const float sv[4] = {s4.x, s4.y, s4.z, s4.w};
                if (sv[0] != 0.0f || sv[1] != 0.0f || sv[2] != 0.0f || sv[3] != 0.0f) {
                    float wi[4], di[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) wi[i] = di[i] = wr[i] * sv[i];
                    if (damped) div4(wi, ap, rp, di);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bool here = sv[i] != 0.0f;
                        on[i] = here ? on[i] + di[i] : on[i];
                        if constexpr (GRAD) {
                            const double t = fma(A.gscale * (double)uk[i], (double)wi[i], G[i]);
                            G[i] = here ? t : G[i];
                        }
                    }
                }
            }
            *reinterpret_cast<float4 *>(&S.u[cur ^ 1][ty + K][4 * tx + HXK]) = make_float4(on[0], on[1], on[2], on[3]);
            float *const out = A.dest(j);
            if (core && out && gz < nz) {
                float *p = out + (long long)gz * nx + gx;
                if (gx + 3 < nx) {
                    const f4u t = {on[0], on[1], on[2], on[3]};
                    *reinterpret_cast<f4u *>(p) = t;
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (gx + i < nx) p[i] = on[i];
                }
            }
        }
        __syncthreads();
    }
    if constexpr (GRAD) {
        if (core && gz < nz && gx < nx) {
            double *p = A.G + (long long)gz * nx + gx;
            if (gx + 3 < nx) {
                const d2u a = {G[0], G[1]}, b = {G[2], G[3]};
                *reinterpret_cast<d2u *>(p) = a;
                *reinterpret_cast<d2u *>(p + 2) = b;
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (gx + i < nx) p[i] = G[i];
            }
        }
    }
}

// The array a batched shot holds for a buffer id.
__device__ __forceinline__ float *batch_buf(const BatchArgs &A, const BatchShot &S, int id, long long P)
{
    if (id < 0) return nullptr;
    if (id >= kBufSlot)
        return reinterpret_cast<float *>(S.arena) + (long long)((id - kBufSlot) / 2 - 1) * A.slot_elems +
               (long long)(id & 1) * P;
    if (id >= kBufUB) return S.UB + (id - kBufUB) * A.fstride;
    if (id >= kBufU) return S.U + (id - kBufU) * A.fstride;
    if (id >= kBufL) return S.Lm + (id - kBufL) * A.fstride;
    return id == kBufDB ? S.DB : S.Z;
}

// The steps of one batched shot, as tile2d takes them.
template <bool GRAD>
struct ShotTile {
    const BatchArgs &A;
    const BatchShot &S;
    const BatchOp &op;
    long long P;
    const float *u, *up, *w;
    int ns;
    const Sparse &inj;
    const float *vals;
    long long vstride;
    const Sparse &gat;
    float *rows;
    unsigned gmask;
    double *G;
    double gscale;
    __device__ ShotTile(const BatchArgs &A_, const BatchShot &S_, const BatchOp &op_, long long P_)
        : A(A_), S(S_), op(op_), P(P_), u(batch_buf(A_, S_, op_.a, P_)), up(batch_buf(A_, S_, op_.b, P_)), w(S_.W),
          ns(op_.ns), inj(GRAD ? S_.rec : S_.src),
          vals(GRAD ? S_.res + (long long)op_.n * A_.nrec : S_.wavelet + op_.n), vstride(GRAD ? -A_.nrec : 1),
          gat(S_.rec), rows(S_.dsim + (long long)op_.n * A_.nrec), gmask(GRAD ? 0u : (unsigned)op_.e), G(S_.G),
          gscale(A_.gscale)
    {
    }
    __device__ const float *level(int j) const { return batch_buf(A, S, op.c[j], P); }
    __device__ float *dest(int j) const
    {
        if (!GRAD) return batch_buf(A, S, op.c[j], P);
        return j == ns - 1 ? batch_buf(A, S, op.d[0], P) : (j == ns - 2 ? batch_buf(A, S, op.d[1], P) : nullptr);
    }
};

}  // namespace

}  // namespace wv
