// Stencil kernels of the forward and adjoint acoustic solver (gfx950, wave64).
//
// The discrete problem is eq. (7) of the paper with the OT2 (second order in time)
// leapfrog on two time levels, updated in place (u^{n+1} overwrites u^{n-1}):
//   u^{n+1} = [2u^n - (1-a)u^{n-1} + w(lap u^n + s^n)]/(1+a),   w = dt^2 c^2,
// so a step moves exactly three reads and one write per point.  It is evaluated as
//   u^{n+1} = u^n + [(1-a)(u^n - u^{n-1}) + w lap u^n]/(1+a)
// (the source term is added after it, by the same launch where it can be): the small per-step
// change is formed first and added once, which keeps binary32 rounding near 5e-6 relative over
// thousands of steps.  The adjoint of the recursion has the same form run backward
// in time (lam^{k-1} overwrites lam^{k+1}) with the residual injected at the
// receivers; the gradient of the misfit with respect to m accumulates
// -(1/dt^2) u^k w (lap lam^k + R^T r^k), which equals
// -(1/dt^2) u^k [(1+a)lam^{k-1} - 2lam^k + (1-a)lam^{k+1}].
//
// Operands read or written once per step (u^{n-1}, w, u^k, the new level) use
// nontemporal loads and stores, so they stream past the caches and leave L2 to the
// centre field, whose halos are re-read by neighbouring tiles.  The binary64 gradient
// takes two 16-byte accesses per lane; it is cached normally, so that a line is
// fetched and written once although each access covers only half of it.
//
// Laplacian along one axis, in binary32 without the cancellation of a direct sum:
//   c_1 ((u_{+1} - u) + (u_{-1} - u)) + [sum_{k>=2} c_k (u_{+k} + u_{-k}) - 2 (sum_{k>=2} c_k) u].
// The dominant k = 1 term is formed from differences, which are small and nearly
// exact for smooth fields; the far weights are small (|c_k| <= 0.18 c_1 for k >= 2 at
// every order up to 16, falling fast), so their plain sum, folded once against u, adds only
// a fraction of an ulp of the result.  In a 3000-step binary32 run this matches the
// all-difference form (about 5e-6 against binary64; a direct sum of all terms loses
// about two digits) at 20 instead of 32 operations per axis for order 16.
//
// Workgroup ids are remapped so that every XCD (each has its own L2) receives a
// contiguous run of neighbouring tiles, whose halos then hit the same L2.
//
// Field arrays are pitched (rows of px >= nx elements, px a multiple of 32 in 3-D):
// a 32-wide tile row is then exactly one 128-byte line.  With a row length that is
// not a multiple of 32 (e.g. 400), every other tile row straddles two lines, which
// measured 10-15 % slower.  The binary64 gradient belongs to the caller and is dense.
#include <algorithm>

#include <hip/hip_ext.h>

#include "wv_chunks3d.h"
#include "wv_stencil_dev.h"

namespace wv {

namespace {


typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 ntload4(const float *p)
{
    const f4v t = __builtin_nontemporal_load(reinterpret_cast<const f4v *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}

__device__ __forceinline__ void ntstore4(float *p, float a, float b, float c, float d)
{
    f4v t = {a, b, c, d};
    __builtin_nontemporal_store(t, reinterpret_cast<f4v *>(p));
}

// What a 3-D launch does beside the step (see StepSide).
struct Side3d {
    const float *plane, *scale;      // injected values: np planes, times *scale if set
    int np, pz[kInjPlanes];
    Sparse gat;                      // receiver gather of the input level into row
    float *row;
    Sparse next;                     // sums for a later step's injection
    const float *next_vals;
    float *next_plane;
    int gat_wg, next_wg;             // workgroups of each
};
constexpr int kSidePerWg = 1024;     // points of a side workgroup

__device__ __forceinline__ void side_work(const Side3d &S, const float *__restrict__ f, int b)
{
    const bool next = b >= S.gat_wg;
    const int i0 = (next ? b - S.gat_wg : b) * kSidePerWg + (int)threadIdx.x;
    if (!next) {
#pragma unroll
        for (int j = 0; j < kSidePerWg / 256; ++j) {
            const int r = i0 + 256 * j;
            if (r < S.gat.n) S.row[r] = gather_point(S.gat, r, f);
        }
    } else {
#pragma unroll
        for (int j = 0; j < kSidePerWg / 256; ++j) {
            const int i = i0 + 256 * j;
            if (i < S.next.npts) S.next_plane[S.next.s_pos[i]] = scatter_sum(S.next, i, S.next_vals);
        }
    }
}

// 3-D step.  A workgroup owns a 32 x 32 tile of the x-y plane and marches down z
// over a chunk of planes; each lane owns four consecutive x points of one row.
//   * z neighbours: a register queue of 2K+1 planes per point, shifted once per plane;
//   * x, y neighbours: the centre plane staged in LDS with its halos (x halo padded to
//     a multiple of four columns so that every LDS access is an aligned float4),
//     double buffered, one barrier per plane;
//   * software pipeline: the global loads a plane needs (its point operands, its
//     halo and the queue front K planes further on) are issued into a register
//     stage AHEAD planes before the plane is computed (two where a third stage fits
//     in the registers, else one);
//   * the halo of plane z+1 goes from its stage straight into the next LDS buffer;
//   * interior LDS values come from the queue, so HBM is read once per value
//     (plus the 2K-plane warm-up of each z chunk); halos are lines the neighbouring
//     tiles of the same XCD read as their interior.
// Rows are pitched to a multiple of four and their pad columns hold zeros, so every field
// access is an aligned float4 at any nx.  WHOLE: nx % 4 == 0, no float4 reaches past nx;
// otherwise the last lane of a row stores zeros to its pad columns, and the dense binary64
// gradient is accessed one value at a time.  (Scalar field accesses for such rows took
// 32.9 us for a forward step of a 183 x 139 x 125 grid at order 8, 49.8 us for an adjoint
// step that updates the gradient.)
// `prev` (u^{n-1}) and `fout` (u^{n+1}) may be the same array: each point of it is
// read and then written by the same lane only.
//
// MODE selects what is done with the Laplacian L of the marched field `fin`:
//   kOT2:  the OT2 step above: out = c + ((1-a)(c - prev) + w L)/(1+a), c = fin's
//          centre; GRAD adds gscale u^k (w L) to G.
//   kLapW: out = w L (the first pass of an OT4 step; no gradient).
//   kOT4:  the second pass of an OT4 step: fin is v = w lap u^n, the centre
//          c = u^n comes pointwise from xtra, and
//          out = c + ((1-a)(c - prev) + v + (w/12) L)/(1+a);
//          GRAD adds both OT4 gradient terms in one update,
//          gscale [u^k (v + (w/12) L) + v vu / 12], where vu = w lap u^k comes pointwise
//          from xtra2 (the second is the term of the m inside the OT4 operator).
// GM selects how the gradient term t = u^k (w L) of an OT2 step reaches G:
//   kGNone: no gradient;  kGAdd: G += gscale t;
//   kGCarryOut: cr = t rounded to binary32, G untouched;
//   kGCarryIn:  G += gscale (t + cr), cr from the kGCarryOut step before.
// A pair of adjoint steps thus reads and writes the binary64 gradient once.
//
// S is what the launch does beside the step, each formerly a launch of its own (4.4 and
// 3.8 us of a 35 us step on 168^3 points at order 8 with 16384 receivers, and 3 us of gaps):
//   * injection into the level it writes (and its gradient term), as inject_kernel would
//     after it, with the same operations in the same order.  The points lie in few planes;
//     a workgroup whose chunk holds one reads its tile of the plane's values before the
//     march, into LDS, so that the march waits for nothing;
//   * the receivers of `fin`, and the sums a later step injects, by further workgroups at
//     the end of the grid.  Their chains of dependent loads then run beside the march; done
//     by the marching workgroups themselves they cost 5-10 us a step.
template <int K, int GM, bool WHOLE, int MODE>
__global__ __launch_bounds__(256, 2) void stencil3d(const Grid g, const float *__restrict__ fin,
                                                 const float *prev, float *fout, const float *__restrict__ w,
                                                 const float *__restrict__ uk, const float *__restrict__ xtra,
                                                 const float *__restrict__ xtra2, double *__restrict__ G,
                                                 float *__restrict__ cr, double gscale, int tiles_x, int tiles_y,
                                                 int zchunks, int zlen, const Side3d S3)
{
    constexpr bool GRAD = GM != kGNone;                    // u^k is read
    constexpr bool GRW = GM == kGAdd || GM == kGCarryIn;    // G is read and written
    static_assert(!(GRAD && MODE == kLapW), "the w lap pass carries no gradient term");
    static_assert(MODE == kOT2 || GM == kGNone || GM == kGAdd, "carried gradient terms are OT2 only");
    constexpr int TX = 32, TY = 32;
    constexpr int HX = (K + 3) / 4 * 4;          // x halo columns (>= K, multiple of 4)
    constexpr int LX = TX + 2 * HX, LY = TY + 2 * K;
    constexpr int NXV = 1 + 2 * ((K + 3) / 4);   // float4 reads for the x neighbours
    constexpr int XC = 4 * ((K + 3) / 4);        // index of the lane's first point in them
    constexpr int NHX = 2 * TY * (HX / 4);        // x-halo float4s per plane
    constexpr int NH = NHX + 2 * K * (TX / 4);    // all halo float4s per plane (<= 256)
    static_assert(NH <= 256, "one halo float4 per lane at most");
    // planes between a stage's loads and its use: two where three stages fit in 256
    // registers without spilling (no gradient, not the OT4 update)
    constexpr int AHEAD = (!GRAD && MODE != kOT4) ? 2 : 1;
    constexpr bool INJ = MODE != kLapW;                     // may inject
    __shared__ __align__(16) float tile[2][LY][LX];
    __shared__ __align__(16) float s_inj[INJ ? kInjPlanes : 1][INJ ? 256 : 1][4];

    const int nwg = tiles_x * tiles_y * zchunks;
    if ((int)blockIdx.x >= nwg) {
        side_work(S3, fin, (int)blockIdx.x - nwg);
        return;
    }
    const int lid = xcd_remap(blockIdx.x, nwg);
    const int tix = lid % tiles_x;
    const int tiy = (lid / tiles_x) % tiles_y;
    const int zc = lid / (tiles_x * tiles_y);
    const int z0 = zc * zlen;
    const int z1 = min(z0 + zlen, g.nz);

    const int tid = threadIdx.x;
    const int tx4 = tid & 7, ty = tid >> 3;
    const int nx = g.nx, ny = g.ny, nz = g.nz, px = g.px;
    const int nxl = (nx - 1) & ~3;                // first column of a row's last float4
    const long long sxy = (long long)px * ny;     // pitched field plane
    const int x0 = tix * TX + 4 * tx4;
    const int y = tiy * TY + ty;
    const bool rowin = y < ny;
    const bool ptin = rowin && x0 < nx;
    const long long rowoff = (long long)(rowin ? y : 0) * px;

    // halo float4 of this lane: source in the plane and place in the tile
    int hrow = 0, hcol = 0, hgx = -1, hgy = -1;
    if (tid < NHX) {
        const int side = tid / (TY * (HX / 4));
        const int rem = tid - side * (TY * (HX / 4));
        const int r = rem / (HX / 4), c4 = rem - (rem / (HX / 4)) * (HX / 4);
        hrow = r + K;
        hcol = side ? (TX + HX + 4 * c4) : (4 * c4);
        hgx = tix * TX - HX + hcol;
        hgy = tiy * TY + r;
    } else if (tid < NH) {
        const int e = tid - NHX;
        const int side = e / (K * (TX / 4));
        const int rem = e - side * (K * (TX / 4));
        const int r = rem / (TX / 4), c4 = rem - (rem / (TX / 4)) * (TX / 4);
        hrow = side ? (TY + K + r) : r;
        hcol = HX + 4 * c4;
        hgx = tix * TX + 4 * c4;
        hgy = tiy * TY - K + hrow;
    }
    const bool hact = tid < NH && hgy >= 0 && hgy < ny;

    // Branch-free float4 load of (gx..gx+3, yy, z): the address is clamped into the
    // grid and the value zeroed outside, so every lane issues its load and no wait
    // is forced at a control-flow join (the pipeline depends on that).
    auto load4 = [&](const float *base, int z, int yy, int gx, bool ok) -> float4 {
        const bool in = ok && z >= 0 && z < nz && yy >= 0 && yy < ny;
        const int zc = min(max(z, 0), nz - 1), yc = min(max(yy, 0), ny - 1);
        const float *row = base + (long long)zc * sxy + (long long)yc * px;
        const bool inx = in && gx >= 0 && gx < nx;
        const float4 t = *reinterpret_cast<const float4 *>(row + min(max(gx, 0), nxl));
        float4 v;
        v.x = inx ? t.x : 0.0f;
        v.y = inx ? t.y : 0.0f;
        v.z = inx ? t.z : 0.0f;
        v.w = inx ? t.w : 0.0f;
        return v;
    };

    struct Stage {
        float4 p, w, u, c, h, f, t;
        double g[GRW ? 4 : 1];
    };
    // loads that computing plane z needs: its point operands (with GRAD also u^k and
    // the gradient), the halo of plane z+1+K and the queue front of plane z+1+K
    // point operands feed only values stored under the same in-range predicate, so
    // they are loaded from the clamped address without zeroing
    auto load4p = [&](const float *base, int z, int gx) -> float4 {
        const int zc = min(z, nz - 1), yc = min(y, ny - 1);
        const float *row = base + (long long)zc * sxy + (long long)yc * px;
        return ntload4(row + min(gx, nxl));
    };
    auto fill = [&](Stage &S, int z) {
        if constexpr (MODE != kLapW) S.p = load4p(prev, z, x0);
        S.w = load4p(w, z, x0);
        if constexpr (MODE == kOT4) S.c = load4p(xtra, z, x0);
        if constexpr (GRAD) S.u = load4p(uk, z, x0);
        if constexpr (GM == kGCarryIn) S.t = load4p(cr, z, x0);
        if constexpr (GRW) {
            const long long pg = ((long long)min(z, nz - 1) * ny + min(y, ny - 1)) * nx;   // dense
            if constexpr (WHOLE) {
                // two 16-byte loads per lane, normally cached: the line a lane pair shares
                // stays in L2 between them
                const double2 g0 = *reinterpret_cast<const double2 *>(&G[pg + min(x0, nx - 4)]);
                const double2 g1 = *reinterpret_cast<const double2 *>(&G[pg + min(x0, nx - 4) + 2]);
                S.g[0] = g0.x; S.g[1] = g0.y; S.g[2] = g1.x; S.g[3] = g1.y;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) S.g[i] = G[pg + min(x0 + i, nx - 1)];
            }
        }
        const bool more = z + 1 < z1;
        S.h = load4(fin, z + 1, hgy, hgx, hact && more);
        S.f = load4(fin, z + 1 + K, y, x0, more && rowin);
    };

    // register queue: q[i][j] = u(x0+i, y, z-K+j)
    float q[4][2 * K + 1];
#pragma unroll
    for (int j = 0; j < 2 * K + 1; ++j) {
        const float4 v = load4(fin, z0 - K + j, y, x0, rowin);
        q[0][j] = v.x; q[1][j] = v.y; q[2][j] = v.z; q[3][j] = v.w;
    }
    if constexpr (INJ) {
        for (int j = 0; j < S3.np; ++j) {
            if (S3.pz[j] < z0 || S3.pz[j] >= z1) continue;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (ptin) v = *reinterpret_cast<const float4 *>(S3.plane + j * sxy + rowoff + x0);
            if (S3.scale) {
                const float q = *S3.scale;
                v = make_float4(v.x * q, v.y * q, v.z * q, v.w * q);
            }
            *reinterpret_cast<float4 *>(&s_inj[j][tid][0]) = v;
        }
    }
    Stage A, B, C;
    fill(A, z0);
    if constexpr (AHEAD == 2) fill(B, z0 + 1);
    {
        const float4 hv = load4(fin, z0, hgy, hgx, hact);
        *reinterpret_cast<float4 *>(&tile[0][ty + K][HX + 4 * tx4]) = make_float4(q[0][K], q[1][K], q[2][K], q[3][K]);
        if (tid < NH) *reinterpret_cast<float4 *>(&tile[0][hrow][hcol]) = hv;
    }
    __syncthreads();

    const float c1 = g.cy[0], c2 = g.cz[0];   // h_x^2/h_y^2, h_x^2/h_z^2
    auto step = [&](int z, Stage &S, Stage &N) {
        // the binary64 gradient of this plane arrived with the stage (clamped address,
        // no branch; only in-range lanes store the update)
        double gold[4] = {0.0, 0.0, 0.0, 0.0};
        if constexpr (GRW) {
#pragma unroll
            for (int i = 0; i < 4; ++i) gold[i] = S.g[i];
        }
        // OT4 adjoint: w lap u^k of this plane, loaded here rather than staged (a staged
        // copy would not fit the registers); the Laplacian below covers its latency
        float4 vu4 = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (MODE == kOT4 && GRAD) vu4 = load4p(xtra2, z, x0);
        fill(N, z + AHEAD);
        const int cur = (z - z0) & 1;
        // x neighbours: NXV aligned float4 around the lane's four points
        float xr[4 * NXV];
        const float *trow = &tile[cur][ty + K][0];
#pragma unroll
        for (int v = 0; v < NXV; ++v) {
            const float4 t = *reinterpret_cast<const float4 *>(trow + HX + 4 * tx4 - XC + 4 * v);
            xr[4 * v + 0] = t.x; xr[4 * v + 1] = t.y; xr[4 * v + 2] = t.z; xr[4 * v + 3] = t.w;
        }
        // per axis: near (k = 1, differences) + far (k >= 2, plain sum) - cf2 * centre;
        // the 3-D kernel applies cx on every axis and scales y and z afterwards
        const float cf2 = g.cf2[0];
        float lap[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float c = q[i][K];
            float sx = g.cx[1] * ((xr[XC + i + 1] - c) + (xr[XC + i - 1] - c));
            float sz = g.cx[1] * ((q[i][K + 1] - c) + (q[i][K - 1] - c));
            if constexpr (K > 1) {
                float fx = 0.0f, fz = 0.0f;
#pragma unroll
                for (int k = 2; k <= K; ++k) {
                    fx = fmaf(g.cx[k], xr[XC + i + k] + xr[XC + i - k], fx);
                    fz = fmaf(g.cx[k], q[i][K + k] + q[i][K - k], fz);
                }
                sx += fmaf(-cf2, c, fx);
                sz += fmaf(-cf2, c, fz);
            }
            lap[i] = fmaf(c2, sz, sx);
        }
        float sy[4];
        {
            const float4 a = *reinterpret_cast<const float4 *>(&tile[cur][ty + K + 1][HX + 4 * tx4]);
            const float4 b = *reinterpret_cast<const float4 *>(&tile[cur][ty + K - 1][HX + 4 * tx4]);
            sy[0] = g.cx[1] * ((a.x - q[0][K]) + (b.x - q[0][K]));
            sy[1] = g.cx[1] * ((a.y - q[1][K]) + (b.y - q[1][K]));
            sy[2] = g.cx[1] * ((a.z - q[2][K]) + (b.z - q[2][K]));
            sy[3] = g.cx[1] * ((a.w - q[3][K]) + (b.w - q[3][K]));
        }
        if constexpr (K > 1) {
            float fy[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 2; k <= K; ++k) {
                const float4 a = *reinterpret_cast<const float4 *>(&tile[cur][ty + K + k][HX + 4 * tx4]);
                const float4 b = *reinterpret_cast<const float4 *>(&tile[cur][ty + K - k][HX + 4 * tx4]);
                fy[0] = fmaf(g.cx[k], a.x + b.x, fy[0]);
                fy[1] = fmaf(g.cx[k], a.y + b.y, fy[1]);
                fy[2] = fmaf(g.cx[k], a.z + b.z, fy[2]);
                fy[3] = fmaf(g.cx[k], a.w + b.w, fy[3]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) sy[i] += fmaf(-cf2, q[i][K], fy[i]);
        }
        // damping a = dampx dx^2 + dampy dy^2 + dampz dz^2; the change of this step is
        // formed from the two levels and added once.  Which product is fused with a sum is written
        // out where the compiler could choose: it did so by the unrolled copy of the plane, and the
        // corners of the layer came to depend, in their last bit, on how z is split
        const int dy_ = layer_depth(y, g.ix0[1], g.ix1[1]);
        const int dz_ = layer_depth(z, g.ix0[2], g.ix1[2]);
        const float ayz = fmaf(g.dampz, (float)(dz_ * dz_), g.dampy * (float)(dy_ * dy_));
        const float pin[4] = {S.p.x, S.p.y, S.p.z, S.p.w};
        const float win[4] = {S.w.x, S.w.y, S.w.z, S.w.w};
        const float uin[4] = {S.u.x, S.u.y, S.u.z, S.u.w};
        const float cin[4] = {S.c.x, S.c.y, S.c.z, S.c.w};
        const float c2in[4] = {vu4.x, vu4.y, vu4.z, vu4.w};
        float on[4], wl[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float l = fmaf(c1, sy[i], lap[i]);
            if constexpr (MODE == kLapW) {
                on[i] = win[i] * l;
            } else {
                // wl: w B u^n, the whole spatial term of the step
                const float ctr = MODE == kOT4 ? cin[i] : q[i][K];
                wl[i] = MODE == kOT4 ? fmaf(win[i] * (1.0f / 12.0f), l, q[i][K]) : win[i] * l;
                const int dx_ = layer_depth(x0 + i, g.ix0[0], g.ix1[0]);
                const float a = fmaf(g.dampx, (float)(dx_ * dx_), ayz);
                const float r = __builtin_amdgcn_rcpf(1.0f + a);
                on[i] = fmaf(fmaf(1.0f - a, ctr - pin[i], wl[i]), r, ctr);
            }
        }
        // injected values of this plane (0 where a point has none): w s and w s / (1+a)
        float wi[4] = {0.f, 0.f, 0.f, 0.f};
        bool inj = false;
        if constexpr (INJ) {
            {
                int j = S3.np;
#pragma unroll
                for (int i = 0; i < kInjPlanes; ++i)
                    if (i < S3.np && S3.pz[i] == z) j = i;
                if (j < S3.np) {
                    const float4 s4 = *reinterpret_cast<const float4 *>(&s_inj[j][tid][0]);   // the lane's own
                    const float sv[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (sv[i] != 0.0f) {
                            inj = true;
                            wi[i] = win[i] * sv[i];
                            on[i] += injected(g, x0 + i, y, z, wi[i]);
                        }
                    }
                }
            }
        }
        if (ptin) {
            const long long p0 = (long long)z * sxy + rowoff + x0;
            const long long p0g = ((long long)z * ny + y) * nx + x0;   // dense gradient
            if constexpr (!WHOLE) {
#pragma unroll
                for (int i = 1; i < 4; ++i) on[i] = x0 + i < nx ? on[i] : 0.0f;   // pad columns stay zero
            }
            ntstore4(fout + p0, on[0], on[1], on[2], on[3]);
            if constexpr (GM == kGCarryOut) {
                float t[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = uin[i] * wl[i];
                ntstore4(cr + p0, t[0], t[1], t[2], t[3]);
                if (inj) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (wi[i] != 0.0f) G[p0g + i] += gscale * (double)uin[i] * (double)wi[i];
                }
            }
            if constexpr (GRW) {
                const float tin[4] = {S.t.x, S.t.y, S.t.z, S.t.w};
                double gn[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (MODE == kOT4)   // v vu / 12 rounded once in binary32
                        gn[i] = gold[i] + gscale * ((double)uin[i] * (double)wl[i] +
                                                    (double)(q[i][K] * c2in[i] * (1.0f / 12.0f)));
                    else if constexpr (GM == kGCarryIn)
                        gn[i] = gold[i] + gscale * ((double)uin[i] * (double)wl[i] + (double)tin[i]);
                    else
                        gn[i] = gold[i] + gscale * (double)uin[i] * (double)wl[i];
                }
                if (inj) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) gn[i] += gscale * (double)uin[i] * (double)wi[i];
                }
                if constexpr (WHOLE) {
                    *reinterpret_cast<double2 *>(&G[p0g]) = make_double2(gn[0], gn[1]);
                    *reinterpret_cast<double2 *>(&G[p0g + 2]) = make_double2(gn[2], gn[3]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (x0 + i < nx) G[p0g + i] = gn[i];
                }
            }
        }
        // stage plane z+1 (after the last plane this buffer is simply not read)
        *reinterpret_cast<float4 *>(&tile[cur ^ 1][ty + K][HX + 4 * tx4]) =
            make_float4(q[0][K + 1], q[1][K + 1], q[2][K + 1], q[3][K + 1]);
        if (tid < NH) *reinterpret_cast<float4 *>(&tile[cur ^ 1][hrow][hcol]) = S.h;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 2 * K; ++j) q[i][j] = q[i][j + 1];
        }
        q[0][2 * K] = S.f.x; q[1][2 * K] = S.f.y; q[2][2 * K] = S.f.z; q[3][2 * K] = S.f.w;
    };
    // AHEAD = 2: three stages in rotation, six planes per trip; otherwise without the
    // binary64 gradient two stages, four planes per trip (the wait pass drains
    // outstanding loads at the back-edge); with it, whose stage also carries u^k and
    // the gradient, one plane per trip and the stage handed over by copy, which keeps
    // it within 256 registers without spilling
    int z = z0;
    if constexpr (AHEAD == 2) {
        for (; z + 5 < z1; z += 6) {
            step(z, A, C);
            step(z + 1, B, A);
            step(z + 2, C, B);
            step(z + 3, A, C);
            step(z + 4, B, A);
            step(z + 5, C, B);
        }
        for (; z + 2 < z1; z += 3) {
            step(z, A, C);
            step(z + 1, B, A);
            step(z + 2, C, B);
        }
        if (z < z1) step(z, A, C);
        if (z + 1 < z1) step(z + 1, B, A);
    } else if constexpr (!GRW) {
        (void)C;
        for (; z + 3 < z1; z += 4) {
            step(z, A, B);
            step(z + 1, B, A);
            step(z + 2, A, B);
            step(z + 3, B, A);
        }
        for (; z + 1 < z1; z += 2) {
            step(z, A, B);
            step(z + 1, B, A);
        }
        if (z < z1) step(z, A, B);
    } else {
        (void)C;
        for (; z < z1; ++z) {
            step(z, A, B);
            A = B;
        }
    }
}

// What a marched 2-D OT2 step's launch does beside the step (see StepSide): both as launches of
// their own took 2.7 us more, of 60 for a forward step of 4000 x 3000 points at order 16.
struct Side2d {
    Sparse inj;                      // samples inj_vals at its points, when set
    const float *inj_vals;
    Sparse gat;                      // receivers of the input level into row, by gat_wg workgroups
    float *row;
    int gat_wg;
};

// 2-D march: OT4, and OT2 where tiles are slower (see tile2d_march): a workgroup owns 256
// consecutive x and marches down z (the second axis).  `prev` and `fout` may be the same array
// (read, then written, by the same lane).  MODE as for the 3-D kernel.
// With samples to inject, an OT2 workgroup then adds those of its strip and rows to the level it
// has just written, as inject_kernel would after the step (the same arithmetic in the same
// order).  Further workgroups gather the receivers.
template <int K, bool GRAD, int MODE>
__global__ __launch_bounds__(256) void stencil2d(Grid g, const float *__restrict__ fin, const float *prev,
                                                 float *fout, const float *__restrict__ w,
                                                 const float *__restrict__ uk, const float *__restrict__ xtra,
                                                 const float *__restrict__ xtra2, double *__restrict__ G,
                                                 double gscale, int tiles_x, int zchunks, int zlen, Side2d S)
{
    static_assert(MODE != kLapW || !GRAD, "w lap carries no gradient term");
    __shared__ float row[256 + 2 * K];
    const int nwg = tiles_x * zchunks;
    if constexpr (MODE == kOT2) {
        if ((int)blockIdx.x >= nwg) {
            const int r = ((int)blockIdx.x - nwg) * 256 + (int)threadIdx.x;
            if (r < S.gat.n) S.row[r] = gather_point(S.gat, r, fin);
            return;
        }
    }
    const int lid = xcd_remap(blockIdx.x, nwg);
    const int tix = lid % tiles_x, zc = lid / tiles_x;
    const int z0 = zc * zlen, z1 = min(z0 + zlen, g.nz);
    march2d<K, GRAD, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, gscale, tix, z0, z1, row);
    if constexpr (MODE == kOT2) {
        if (S.inj_vals) {
            __syncthreads();
            const int nx = g.nx, x0 = tix * 256, x1 = min(x0 + 256, nx);
            for (int i = threadIdx.x; i < S.inj.npts; i += 256) {
                const int p = S.inj.s_pts[i];
                const int z = p / nx, x = p - z * nx;
                if (z < z0 || z >= z1 || x < x0 || x >= x1) continue;
                inject_point<GRAD>(g, S.inj, i, p, x, 0, z, S.inj_vals, w, fout, uk, G, p, gscale);
            }
        }
    }
}

// Adds w s / (1+a) at the source (or receiver) points of the level just written.
template <bool GRAD>
__global__ void inject_kernel(Grid g, Sparse sp, const float *__restrict__ vals, const float *__restrict__ w,
                              float *__restrict__ fout, const float *__restrict__ uk, double *__restrict__ G,
                              double gscale)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= sp.npts) return;
    const int p = sp.s_pts[i];
    const long long sxy = (long long)g.px * g.ny;   // p indexes the pitched field arrays
    const int z = (int)(p / sxy);
    const int rem = (int)(p - z * sxy);
    const int y = rem / g.px, x = rem - (rem / g.px) * g.px;
    inject_point<GRAD>(g, sp, i, p, x, y, z, vals, w, fout, uk, G, ((long long)z * g.ny + y) * g.nx + x, gscale);
}

// each point's place in the planes of its table, and (with weights) its weight there
__global__ void plane_setup_kernel(Sparse sp, int plane, float *__restrict__ weights)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < sp.npts; i += gridDim.x * blockDim.x) {
        const int p = sp.s_pts[i];
        const int z = p / plane;
        int pos = p - z * plane;
        for (int j = 0; j < sp.np; ++j)
            if (sp.pz[j] == z) pos += j * plane;
        sp.s_pos[i] = pos;
        if (weights) weights[pos] = sp.s_wt[sp.s_start[i]];
    }
}

__global__ void plane_sums_kernel(Sparse sp, const float *__restrict__ vals, float *__restrict__ plane)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < sp.npts; i += gridDim.x * blockDim.x)
        plane[sp.s_pos[i]] = scatter_sum(sp, i, vals);
}

__global__ void gather_kernel(Sparse sp, const float *__restrict__ f, float *__restrict__ out)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= sp.n) return;
    out[r] = gather_point(sp, r, f);
}

__global__ void gather_sum_kernel(Sparse sp, const float *__restrict__ f, float *__restrict__ out)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    float tot = 0.0f;
    for (int r = 0; r < sp.n; ++r) {
        float s = 0.0f;
        for (int c = 0; c < sp.nc; ++c) s = fmaf(sp.g_wt[r * sp.nc + c], f[sp.g_idx[r * sp.nc + c]], s);
        tot += s;
    }
    out[0] = tot;
}

// w over the pitched field array from the dense velocity; pad columns get 0
__global__ void setup_w_kernel(const float *__restrict__ vel, float *__restrict__ w, long long P, int nx, int px,
                               double dt, double vmax, unsigned *err)
{
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < P;
         p += (long long)gridDim.x * blockDim.x) {
        const long long row = p / px;
        const int x = (int)(p - row * px);
        if (x >= nx) {
            w[p] = 0.0f;
            continue;
        }
        const float v = vel[row * nx + x];
        const double vd = (double)v;
        if (!(vd > 0.0) || !(vd <= vmax)) atomicOr(err, 1u);
        w[p] = (float)(dt * dt * vd * vd);
    }
}

template <typename T>
__global__ void fill_kernel(T *p, long long n, T v)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void check_finite_kernel(const float *__restrict__ f, long long n, unsigned *err)
{
    bool bad = false;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        bad |= !isfinite(f[i]);
    if (bad) atomicOr(err, 8u);
}

constexpr int kRedThreads = 256;

__global__ __launch_bounds__(kRedThreads) void residual_kernel(const float *__restrict__ dsim,
                                                               const float *__restrict__ dobs,
                                                               float *__restrict__ res, long long n,
                                                               long long nrec, double *partials)
{
    __shared__ double sh[kRedThreads];
    double acc = 0.0;
    for (long long e = blockIdx.x * (long long)kRedThreads + threadIdx.x; e < n;
         e += (long long)gridDim.x * kRedThreads) {
        if (e < nrec) {
            res[e] = 0.0f;
            continue;
        }
        const double r = (double)dsim[e] - (double)dobs[e];
        res[e] = (float)r;
        acc += r * r;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kRedThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(kRedThreads) void final_sum_kernel(const double *partials, int n, double *out)
{
    __shared__ double sh[kRedThreads];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kRedThreads) acc += partials[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kRedThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = 0.5 * sh[0];
}

struct Dims3 { int n[3]; int N[3]; int nbl; int nd; };

__global__ void pad_kernel(Dims3 d, const float *__restrict__ vin, float *__restrict__ vout, long long P)
{
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < P;
         p += (long long)gridDim.x * blockDim.x) {
        long long r = p;
        long long src = 0, stride = 1;
        for (int a = 0; a < d.nd; ++a) {
            int i = (int)(r % d.N[a]);
            r /= d.N[a];
            int j = i - d.nbl;
            j = j < 0 ? 0 : (j > d.n[a] - 1 ? d.n[a] - 1 : j);
            src += (long long)j * stride;
            stride *= d.n[a];
        }
        vout[p] = vin[src];
    }
}

__global__ void velgrad_kernel(Dims3 d, const float *__restrict__ vpad, const double *__restrict__ gm,
                               double *__restrict__ gv, long long Pint)
{
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < Pint;
         q += (long long)gridDim.x * blockDim.x) {
        int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
        long long r = q;
        for (int a = 0; a < d.nd; ++a) {
            int j = (int)(r % d.n[a]);
            r /= d.n[a];
            lo[a] = (j == 0) ? 0 : j + d.nbl;
            hi[a] = (j == d.n[a] - 1) ? d.N[a] - 1 : j + d.nbl;
        }
        double s = 0.0;
        const int z1 = d.nd == 3 ? hi[2] : 0, zl = d.nd == 3 ? lo[2] : 0;
        for (int k = zl; k <= z1; ++k)
            for (int j = lo[1]; j <= hi[1]; ++j)
                for (int i = lo[0]; i <= hi[0]; ++i) {
                    const long long p = ((long long)k * d.N[1] + j) * d.N[0] + i;
                    const double c = (double)vpad[p];
                    s += gm[p] * (-2.0 / (c * c * c));
                }
        gv[q] = s;
    }
}

int grid_for(long long n, int threads)
{
    long long b = (n + threads - 1) / threads;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    return (int)b;
}

// z chunking: about `target` workgroups, chunks no shorter than min_len planes.
void choose_chunks(long long tiles, int nz, int min_len, int target, int &zchunks, int &zlen)
{
    long long want = target / tiles;
    long long maxc = nz / (min_len > 0 ? min_len : 1);
    if (maxc < 1) maxc = 1;
    if (want > maxc) want = maxc;
    if (want < 1) want = 1;
    zlen = (int)((nz + want - 1) / want);
    zchunks = (nz + zlen - 1) / zlen;
}

// z chunks of a 3-D launch (see chunks3d).
template <typename Kern>
void choose_chunks3d(Kern kern, long long tiles, int nz, int K, bool grad, int &zchunks, int &zlen)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    zlen = chunks3d(tiles, nz, K, grad, per_cu, device_cus());
    zchunks = (nz + zlen - 1) / zlen;
}

// Kernel launch; with events, the dispatch itself records them around the kernel.
template <typename Kern, typename... Args>
void launch_timed(Kern kern, dim3 grid, hipStream_t s, LaunchEvents ev, Args... args)
{
    if (ev.start)
        hipExtLaunchKernelGGL(kern, grid, dim3(256), 0, s, ev.start, ev.stop, 0, args...);
    else
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, args...);
}

template <int K, int GM, bool WHOLE, int MODE>
hipError_t launch3d(const Grid &g, const float *fin, const float *prev, float *fout, const float *w,
                    const float *uk, const float *xtra, const float *xtra2, double *G, float *cr, double gscale,
                    hipStream_t s, LaunchEvents ev, const StepSide &side)
{
    auto kern = stencil3d<K, GM, WHOLE, MODE>;
    const int tiles_x = (g.nx + 31) / 32, tiles_y = (g.ny + 31) / 32;
    int zchunks, zlen;
    choose_chunks3d(kern, (long long)tiles_x * tiles_y, g.nz, K, GM != kGNone, zchunks, zlen);
    const int nwg = tiles_x * tiles_y * zchunks;
    Side3d S{};
    if (side.inj) {
        if (side.inj->np < 1 || !side.plane || MODE == kLapW) return hipErrorInvalidValue;
        S.plane = side.plane;
        S.scale = side.scale;
        S.np = side.inj->np;
        std::copy(side.inj->pz, side.inj->pz + S.np, S.pz);
    }
    if (side.gat && side.row) {
        if (MODE == kOT4) return hipErrorInvalidValue;   // its input is not the wavefield
        S.gat = *side.gat;
        S.row = side.row;
        S.gat_wg = (S.gat.n + kSidePerWg - 1) / kSidePerWg;
    }
    if (side.next) {
        S.next = *side.next;
        S.next_vals = side.next_vals;
        S.next_plane = side.next_plane;
        S.next_wg = (S.next.npts + kSidePerWg - 1) / kSidePerWg;
    }
    launch_timed(kern, dim3(nwg + S.gat_wg + S.next_wg), s, ev, g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale,
                 tiles_x, tiles_y, zchunks, zlen, S);
    return hipGetLastError();
}

template <int K, int GM, int MODE>
hipError_t launch_k(const Grid &g, const float *fin, const float *prev, float *fout, const float *w,
                    const float *uk, const float *xtra, const float *xtra2, double *G, float *cr, double gscale,
                    hipStream_t s, LaunchEvents ev, const StepSide &side)
{
    if (g.ndim == 3) {
        if (g.nx % 4 == 0)
            return launch3d<K, GM, true, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
        return launch3d<K, GM, false, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    }
    // 2-D grids are small (a few MB): a step is bound by the latency of each workgroup's
    // plane-by-plane march, not by bandwidth, so chunks are short (down to K planes, whose
    // 2K-plane warm-up loads are issued together) and the workgroups many
    const int tiles_x = (g.nx + 255) / 256;
    int zchunks, zlen;
    choose_chunks(tiles_x, g.nz, K, 2048, zchunks, zlen);
    Side2d S{};
    if (side.next || (MODE != kOT2 && (side.inj || side.row))) return hipErrorInvalidValue;
    if (side.inj) {
        S.inj = *side.inj;
        S.inj_vals = side.vals;
    }
    if (side.gat && side.row) {
        S.gat = *side.gat;
        S.row = side.row;
        S.gat_wg = (S.gat.n + 255) / 256;
    }
    launch_timed(stencil2d<K, GM == kGAdd, MODE>, dim3(tiles_x * zchunks + S.gat_wg), s, ev, g, fin, prev, fout, w, uk,
                 xtra, xtra2, G, gscale, tiles_x, zchunks, zlen, S);
    return hipGetLastError();
}

template <int GM, int MODE>
hipError_t launch_any(const Grid &g, const float *fin, const float *prev, float *fout, const float *w,
                      const float *uk, const float *xtra, const float *xtra2, double *G, double gscale, hipStream_t s,
                      LaunchEvents ev, const StepSide &side, float *cr = nullptr)
{
    switch (g.K) {
    case 1: return launch_k<1, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 2: return launch_k<2, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 3: return launch_k<3, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 4: return launch_k<4, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 5: return launch_k<5, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 6: return launch_k<6, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 7: return launch_k<7, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    case 8: return launch_k<8, GM, MODE>(g, fin, prev, fout, w, uk, xtra, xtra2, G, cr, gscale, s, ev, side);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_fwd_step(const Grid &g, const float *u_in, const float *u_prev, float *u_out, const float *w,
                           hipStream_t s, LaunchEvents ev, const StepSide &side)
{
    return launch_any<kGNone, kOT2>(g, u_in, u_prev, u_out, w, nullptr, nullptr, nullptr, nullptr, 0.0, s, ev, side);
}

hipError_t launch_adj_step(const Grid &g, const float *lam_in, const float *lam_next, float *lam_out,
                           const float *w, const float *uk, double *G, double gscale, hipStream_t s,
                           LaunchEvents ev, float *carry, int gmode, const StepSide &side)
{
    if (!G) return launch_any<kGNone, kOT2>(g, lam_in, lam_next, lam_out, w, nullptr, nullptr, nullptr, nullptr, 0.0,
                                            s, ev, side);
    if (gmode != kGAdd && (g.ndim != 3 || !carry)) return hipErrorInvalidValue;
    switch (gmode) {
    case kGAdd:
        return launch_any<kGAdd, kOT2>(g, lam_in, lam_next, lam_out, w, uk, nullptr, nullptr, G, gscale, s, ev, side);
    case kGCarryOut:
        return launch_any<kGCarryOut, kOT2>(g, lam_in, lam_next, lam_out, w, uk, nullptr, nullptr, G, gscale, s, ev,
                                            side, carry);
    case kGCarryIn:
        return launch_any<kGCarryIn, kOT2>(g, lam_in, lam_next, lam_out, w, uk, nullptr, nullptr, G, gscale, s, ev,
                                           side, carry);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_lapw(const Grid &g, const float *f, float *v_out, const float *w, hipStream_t s, LaunchEvents ev,
                       const StepSide &side)
{
    return launch_any<kGNone, kLapW>(g, f, nullptr, v_out, w, nullptr, nullptr, nullptr, nullptr, 0.0, s, ev, side);
}

hipError_t launch_ot4_update(const Grid &g, const float *v, const float *u_in, const float *u_prev, float *u_out,
                             const float *w, const float *uk, const float *vu, double *G, double gscale, hipStream_t s,
                             LaunchEvents ev, const StepSide &side)
{
    if (G) return launch_any<kGAdd, kOT4>(g, v, u_prev, u_out, w, uk, u_in, vu, G, gscale, s, ev, side);
    return launch_any<kGNone, kOT4>(g, v, u_prev, u_out, w, nullptr, u_in, nullptr, nullptr, 0.0, s, ev, side);
}

hipError_t launch_plane_setup(const Grid &g, const Sparse &sp, float *planes, int nsets, bool weights, hipStream_t s)
{
    const long long set = (long long)sp.np * g.px * g.ny;
    hipLaunchKernelGGL((fill_kernel<float>), dim3(grid_for(nsets * set, 256)), dim3(256), 0, s, planes, nsets * set,
                       0.0f);
    hipLaunchKernelGGL(plane_setup_kernel, dim3(grid_for(sp.npts, 256)), dim3(256), 0, s, sp, g.px * g.ny,
                       weights ? planes : nullptr);
    return hipGetLastError();
}

hipError_t launch_plane_sums(const Sparse &sp, const float *vals, float *plane, hipStream_t s)
{
    hipLaunchKernelGGL(plane_sums_kernel, dim3(grid_for(sp.npts, 256)), dim3(256), 0, s, sp, vals, plane);
    return hipGetLastError();
}

hipError_t launch_inject_src(const Grid &g, const Sparse &sp, const float *q, int n, const float *w,
                             float *u_out, hipStream_t s)
{
    if (sp.npts == 0) return hipSuccess;
    hipLaunchKernelGGL((inject_kernel<false>), dim3((sp.npts + 63) / 64), dim3(64), 0, s, g, sp, q + n, w, u_out,
                       nullptr, nullptr, 0.0);
    return hipGetLastError();
}

hipError_t launch_inject_res(const Grid &g, const Sparse &sp, const float *r_row, const float *w, float *lam_out,
                             const float *uk, double *G, double gscale, hipStream_t s)
{
    if (sp.npts == 0) return hipSuccess;
    if (G)
        hipLaunchKernelGGL((inject_kernel<true>), dim3((sp.npts + 255) / 256), dim3(256), 0, s, g, sp, r_row, w,
                           lam_out, uk, G, gscale);
    else
        hipLaunchKernelGGL((inject_kernel<false>), dim3((sp.npts + 255) / 256), dim3(256), 0, s, g, sp, r_row, w,
                           lam_out, nullptr, nullptr, 0.0);
    return hipGetLastError();
}

hipError_t launch_gather(const Sparse &sp, const float *f, float *out, hipStream_t s)
{
    if (sp.n == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_kernel, dim3((sp.n + 255) / 256), dim3(256), 0, s, sp, f, out);
    return hipGetLastError();
}

hipError_t launch_gather_sum(const Sparse &sp, const float *f, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(gather_sum_kernel, dim3(1), dim3(64), 0, s, sp, f, out);
    return hipGetLastError();
}

hipError_t launch_setup_w(const Grid &g, const float *vel, float *w, double dt, double vmax, unsigned *err,
                          hipStream_t s)
{
    hipLaunchKernelGGL(setup_w_kernel, dim3(grid_for(g.P, 256)), dim3(256), 0, s, vel, w, g.P, g.nx, g.px, dt,
                       vmax, err);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, long long n, float v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((fill_kernel<float>), dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_f64(double *p, long long n, double v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((fill_kernel<double>), dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t *p, long long n, uint64_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((fill_kernel<uint64_t>), dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_check_finite(const float *f, long long n, unsigned *err, hipStream_t s)
{
    hipLaunchKernelGGL(check_finite_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, f, n, err);
    return hipGetLastError();
}

hipError_t launch_residual_misfit(const float *dsim, const float *dobs, float *res, long long n, long long nrec,
                                  double *partials, int nparts, double *misfit, hipStream_t s)
{
    hipLaunchKernelGGL(residual_kernel, dim3(nparts), dim3(kRedThreads), 0, s, dsim, dobs, res, n, nrec, partials);
    hipLaunchKernelGGL(final_sum_kernel, dim3(1), dim3(kRedThreads), 0, s, partials, nparts, misfit);
    return hipGetLastError();
}

hipError_t launch_pad_velocity(int ndim, const int *n, int nbl, const float *vin, float *vout, hipStream_t s)
{
    Dims3 d{};
    d.nd = ndim;
    d.nbl = nbl;
    long long P = 1;
    for (int a = 0; a < 3; ++a) {
        d.n[a] = a < ndim ? n[a] : 1;
        d.N[a] = a < ndim ? n[a] + 2 * nbl : 1;
        P *= d.N[a];
    }
    hipLaunchKernelGGL(pad_kernel, dim3(grid_for(P, 256)), dim3(256), 0, s, d, vin, vout, P);
    return hipGetLastError();
}

hipError_t launch_velocity_gradient(int ndim, const int *n, int nbl, const float *vpad, const double *gm,
                                    double *gv, hipStream_t s)
{
    Dims3 d{};
    d.nd = ndim;
    d.nbl = nbl;
    long long Pint = 1;
    for (int a = 0; a < 3; ++a) {
        d.n[a] = a < ndim ? n[a] : 1;
        d.N[a] = a < ndim ? n[a] + 2 * nbl : 1;
        Pint *= d.n[a];
    }
    hipLaunchKernelGGL(velgrad_kernel, dim3(grid_for(Pint, 256)), dim3(256), 0, s, d, vpad, gm, gv, Pint);
    return hipGetLastError();
}

}  // namespace wv
