// Internal declarations of libwv (GPU path).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/wv.h"

namespace wv {

constexpr int kMaxK = 8;            // space order up to 16
constexpr int kBlocksPerChunk = 256; // codec: blocks per chunk (one workgroup)

// Geometry and coefficients of one padded grid, as the stencil kernels see it.
// Axes are named for the array layout: x contiguous, z slowest.  In 2-D, y is
// absent (ny = 1) and the model's second axis is z.
// The solver's field arrays (wavefields, w, checkpoint slots) are pitched: point
// (x, y, z) sits at x + px (y + ny z), with px = nx rounded up to 32 in 3-D, so that
// every row starts on a 128-byte line (the columns from nx to a multiple of four
// hold zeros, those after them nothing that is read).  In 2-D px = nx.  Arrays the caller owns (velocity,
// gradient, final state) are dense: x + nx (y + ny z).
struct Grid {
    int nx, ny, nz;          // padded extents
    int px;                  // row pitch of the solver's field arrays (elements)
    int ix0[3], ix1[3];      // interior index range [ix0, ix1] per array axis (x, y, z)
    float cx[kMaxK + 1];     // a_k / h^2 per axis, k = 1..K;
    float cy[kMaxK + 1];     // cy[0] = h_x^2/h_y^2 and cz[0] = h_x^2/h_z^2 (the 3-D kernel
    float cz[kMaxK + 1];     // applies cx[k] on every axis and scales y, z by these)
    float cf2[3];            // 2 sum_{k>=2} of the axis's weights (x from cx, y from cy, z from cz)
    float dampx, dampy, dampz; // 0.5 dt smax_axis / nbl^2; a = sum damp_axis * delta_axis^2
    int K;
    int ndim;
    int time_order;          // 2 (OT2) or 4 (OT4)
    long long P;             // elements of one field array: px * ny * nz
};

// A 3-D step injects in its own launch when the points lie in few grid planes (a surface
// survey: one plane on the nodes, two between them); more planes take a launch of their own.
constexpr int kInjPlanes = 4;
// Sparse point operators (sources / receivers), built on the host.
//   gather:  out[r] = sum_c wt[r*nc + c] * f[idx[r*nc + c]]
//   scatter: unique points pts[i], entries [start[i], start[i+1]) of (col, wt)
struct Sparse {
    int n;            // number of sources or receivers
    int nc;           // corners per point (4 or 8)
    const int *g_idx; const float *g_wt;          // gather tables [n*nc]
    int npts;         // unique grid points touched
    const int *s_pts; const int *s_start;        // [npts], [npts+1]
    const int *s_col; const float *s_wt;         // [nnz]
    // 3-D: the grid planes that hold scatter points, when they are at most kInjPlanes
    // (np = 0 otherwise), ascending; s_pos[npts]: each unique point's place in an array of
    // np pitched planes
    int np; int pz[kInjPlanes];
    int *s_pos;
};

// What a step's launch does beside the step.
struct StepSide {
    // injects into the level it writes at the points of inj.  3-D (np > 0): plane holds their
    // values in np pitched planes, each multiplied by *scale when scale is set; 2-D: the samples
    // are vals
    const Sparse *inj = nullptr;
    const float *plane = nullptr, *scale = nullptr;
    const float *vals = nullptr;
    // gathers the receivers of its input level into row
    const Sparse *gat = nullptr;
    float *row = nullptr;
    // 3-D: sums the samples next_vals at the points of next into the planes next_plane (the
    // values a later step injects; places of no point are not written)
    const Sparse *next = nullptr;
    const float *next_vals = nullptr;
    float *next_plane = nullptr;
};

// ---------------------------------------------------------------- stencil launches (wv_stencil.hip)
// Optional pair of events recorded by the kernel dispatch itself (start and end of the
// stencil kernel, nothing else), for per-launch timing.
struct LaunchEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};
// Forward step: u_out = u_in + ((1-a)(u_in - u_prev) + w lap u_in)/(1+a).
// u_out may equal u_prev (in place); it must differ from u_in.
hipError_t launch_fwd_step(const Grid &g, const float *u_in, const float *u_prev, float *u_out, const float *w,
                           hipStream_t s, LaunchEvents ev = {}, const StepSide &side = {});
// How an adjoint step's gradient term t = uk * (w lap lam_in) reaches G.  The carried
// forms are for 3-D grids: a step with kGCarryOut leaves t, rounded to binary32, in a
// field-sized array, and the next adjoint step (kGCarryIn) adds it with its own term,
// so that a pair of steps reads and writes G once.
constexpr int kGNone = 0, kGAdd = 1, kGCarryOut = 2, kGCarryIn = 3;
// Adjoint step (lam_in = lam^k, lam_next = lam^{k+1}, lam_out = lam^{k-1}, may equal
// lam_next): the same update, and (if G) G += gscale * uk * (w lap lam_in), or the
// carried form gmode selects with the array carry (pitched like a field).  An injection adds
// its gradient term too.
// 2-D OT2 steps go through launch_tile2d, which marches some grids with these two.
hipError_t launch_adj_step(const Grid &g, const float *lam_in, const float *lam_next, float *lam_out,
                           const float *w, const float *uk, double *G, double gscale, hipStream_t s,
                           LaunchEvents ev = {}, float *carry = nullptr, int gmode = kGAdd,
                           const StepSide &side = {});
// OT4, first pass: v_out = w lap f (side: gather only, in 3-D).
hipError_t launch_lapw(const Grid &g, const float *f, float *v_out, const float *w, hipStream_t s,
                       LaunchEvents ev = {}, const StepSide &side = {});
// OT4, second pass: u_out = u_in + ((1-a)(u_in - u_prev) + v + (w/12) lap v)/(1+a), v = w lap u_in
// from the first pass; with G, G += gscale * (uk * (v + (w/12) lap v) + v * vu / 12), vu = w lap uk.
// u_out may equal u_prev.  side: injection and next planes, in 3-D.
hipError_t launch_ot4_update(const Grid &g, const float *v, const float *u_in, const float *u_prev, float *u_out,
                             const float *w, const float *uk, const float *vu, double *G, double gscale,
                             hipStream_t s, LaunchEvents ev = {}, const StepSide &side = {});
// 3-D tables with np > 0: fills sp.s_pos and zeroes planes (nplanes sets of np pitched planes);
// with weights, the first set receives each point's weight (tables of one entry a point).
hipError_t launch_plane_setup(const Grid &g, const Sparse &sp, float *planes, int nsets, bool weights, hipStream_t s);
// The points' summed samples, at their places in one set of planes (as StepSide::next).
hipError_t launch_plane_sums(const Sparse &sp, const float *vals, float *plane, hipStream_t s);
// 2-D OT2 steps of one shot in one launch: forward steps from u^n, or adjoint steps from
// lam^k, ns of them (at most tile2d_steps).
constexpr int kTileSteps = 8, kTileRegion = 64;   // a workgroup holds 64 x 64 points
constexpr int tile2d_steps(int K) { return K <= 2 ? 8 : (K == 8 ? 2 : 16 / K); }
// rim of a region that ns steps make invalid, in whole lanes' blocks
constexpr int tile2d_halo(int K, int ns) { return (K * ns + 3) & ~3; }
// What a 2-D OT2 run works with (see Prog2d::rings): its groups, and the field arrays they take.
struct Rings2d {
    int steps;      // most steps of a group
    int jobs;       // most fields of one encode or decode
    int levels;     // arrays of the ring of forward levels
    int decoded;    // and of decoded checkpoints
    int lam;        // adjoint levels
    bool march;     // steps march one by one instead of running in tiles
};
// bounds of the same for an order
constexpr int tile2d_jobs(int K) { return tile2d_steps(K) > 4 ? tile2d_steps(K) : 4; }
constexpr int tile2d_ring(int K) { return 2 * tile2d_jobs(K) + 3; }
constexpr int tile2d_decoded(int K) { return tile2d_jobs(K) + 2; }
struct Tile2dArgs {
    const float *u, *up, *w;        // u^n, u^{n-1} (lam^k, lam^{k+1}); w
    float *out[kTileSteps];         // where step j's level goes (null: it is not kept)
    int ns;
    Sparse inj;                     // injection of step j: samples vals + j vstride
    const float *vals;
    long long vstride;
    Sparse gat;                     // bit j of gmask: the receivers of u^{n+j} go to rows + j gat.n
    float *rows;
    unsigned gmask;
    const float *uk[kTileSteps];    // with G: u^k of step j, and the gradient (dense)
    double *G;
    double gscale;
    bool march;                     // of ns = 1 with out[0] set: marched instead, with the same bits
    __host__ __device__ const float *level(int j) const { return uk[j]; }
    __host__ __device__ float *dest(int j) const { return out[j]; }
};
hipError_t launch_tile2d(const Grid &g, const Tile2dArgs &A, hipStream_t s, LaunchEvents ev = {});
int device_cus();
// whether the steps of a call for one shot march
enum { kRunForward, kRunGradient, kRunAdjointSrc };
bool tile2d_march(int K, int nx, int nz, int run);
// steps per group for a grid, nshots shots advancing together
int tile2d_choose(int K, int nx, int nz, int nshots);

// Source injection of sample q[n] (forward) at the unique source points of u_out.
hipError_t launch_inject_src(const Grid &g, const Sparse &sp, const float *q, int n, const float *w,
                             float *u_out, hipStream_t s);
// Residual injection of row r_row (adjoint) at the unique receiver points; gradient term.
hipError_t launch_inject_res(const Grid &g, const Sparse &sp, const float *r_row, const float *w, float *lam_out,
                             const float *uk, double *G, double gscale, hipStream_t s);
// Receiver gather out[r] = (R f)_r.
hipError_t launch_gather(const Sparse &sp, const float *f, float *out, hipStream_t s);
// Sum over sources of the gathered field: out[0] = sum_s (S f)_s.
hipError_t launch_gather_sum(const Sparse &sp, const float *f, float *out, hipStream_t s);
// w = dt^2 vel^2 (vel dense, w pitched, pad columns 0) and validation; err bit 1:
// non-finite or out of (0, vmax].
hipError_t launch_setup_w(const Grid &g, const float *vel, float *w, double dt, double vmax, unsigned *err,
                          hipStream_t s);
hipError_t launch_fill_f32(float *p, long long n, float v, hipStream_t s);
hipError_t launch_fill_f64(double *p, long long n, double v, hipStream_t s);
hipError_t launch_fill_u64(uint64_t *p, long long n, uint64_t v, hipStream_t s);
// r = (float)((double)dsim - (double)dobs) for rows 1..nt (row 0 = 0); partial sums of r^2 (binary64).
hipError_t launch_residual_misfit(const float *dsim, const float *dobs, float *res, long long nrow_elems,
                                  long long nrec, double *partials, int nparts, double *misfit, hipStream_t s);
hipError_t launch_pad_velocity(int ndim, const int *n, int nbl, const float *vin, float *vout, hipStream_t s);
hipError_t launch_velocity_gradient(int ndim, const int *n, int nbl, const float *vpad, const double *gm,
                                    double *gv, hipStream_t s);
hipError_t launch_check_finite(const float *f, long long n, unsigned *err, hipStream_t s);

// ---------------------------------------------------------------- codec (wv_codec.hip)
struct CodecDims {
    int ndim;
    int dims[3];       // axis 0 fastest; 2-D: dims[2] = 1
    int pitch;         // elements from one row (axis 0) of the field array to the next (>= dims[0])
    int nb[3];         // blocks per axis
    long long nblocks;
    long long nchunks;
    long long prefix_bytes;  // header + chunk table + block lengths
};
// pitch 0: dense rows (pitch = dims[0])
CodecDims codec_dims(int ndim, const int *dims, int pitch = 0);
size_t codec_max_bytes(const CodecDims &cd);
// Encode fields of one geometry, in two launches or (many chunks) three, job by job into out + *base (device
// offset), capacity cap bytes from `out`; *next = *base + stream bytes rounded up to 256.  A
// job whose base is the word the job before it writes as its next starts where that ends.
// work: encode_work_bytes(cd, staged, jobs) bytes, 256-byte aligned, any contents (chunk
// word counts, offsets and, when staged, block lengths and a kLdsWords-word slot per chunk;
// without staging every chunk is encoded twice, and there is one job).
// err: bit 2 = capacity overflow, bit 1 = non-finite input.
// stats[0] += stream bytes, stats[1] = max(stats[1], *next).
constexpr int kEncJobs = 8;
struct EncJob {
    const float *field;
    const float *sub;        // nullable: field - sub, in binary32
    const uint64_t *base;
    uint64_t *next;
    uint64_t *size_out;      // nullable: receives the stream's size in bytes
};
size_t encode_work_bytes(const CodecDims &cd, bool staged, int jobs = 1);
hipError_t launch_encode(const CodecDims &cd, const EncJob *jobs, int njobs, double tol, uint8_t *out, uint64_t cap,
                         uint8_t *work, bool staged, unsigned *err, unsigned long long *stats, hipStream_t s);
// Decode the streams at in + *base (base == nullptr: offset 0) into field, or, when sub
// is not null, store sub - decoded; cap bytes are readable from `in` (a stream that
// does not fit decodes to zeros).
struct DecJob {
    const uint64_t *base;
    float *field;
    const float *sub;
};
hipError_t launch_decode(const CodecDims &cd, const uint8_t *in, const DecJob *jobs, int njobs, uint64_t cap,
                         hipStream_t s);

// ---------------------------------------------------------------- batched 2-D solver (wv_batch.hip)
// Several 2-D shots of one grid, order, step count and schedule advanced together: every
// step of their program is for all of them.  Each shot keeps the buffers of a solo call
// (field arrays dense in 2-D).
struct BatchShot {
    float *U, *UB, *DB, *Lm, *Z, *W;   // rings of field arrays, BatchArgs::fstride elements apart
    const float *wavelet;     // [nt]
    const float *dobs;        // [nt+1][nrec]
    float *dsim, *res;        // [nt+1][nrec]
    double *G;                // gradient (caller's, dense [P])
    double *partials;         // residual partial sums [kParts]
    double *misfit;           // phi (device)
    uint8_t *arena;           // checkpoint memory of this shot
    uint64_t arena_bytes;
    uint64_t *offs;           // stream offsets (as the solo executor's)
    uint64_t *sizes;          // stream bytes of u^k per stored k
    uint32_t *chunk_words;    // [jobs][nchunks]: words per chunk of the fields of an encode
    unsigned *err;            // bit 1: velocity, 2: non-finite input to the codec, 4: arena overflow,
                              // 8: non-finite wavefield, 16: barrier timeout
    unsigned long long *stats;  // [0] stream bytes stored, [1] peak arena offset
    Sparse src, rec;
};

// Buffers of a program step, by id: the shot's own arrays (member i of a ring as its first
// id + i), or level l of checkpoint slot b (uncompressed) as kBufSlot + 2 b + l.
enum BatchBuf { kBufNone = -1, kBufZ = 0, kBufDB = 1, kBufL = 2, kBufU = 8, kBufUB = 32, kBufSlot = 48 };
static_assert(kBufU + tile2d_ring(1) <= kBufUB && kBufUB + tile2d_decoded(1) <= kBufSlot, "buffer ids");
// Steps of a 2-D OT2 program (built by Prog2d).
//   kOpStep:   ns forward steps from u^n in a and u^{n-1} in b; step j's level goes to c[j]
//              (kBufNone: not kept) with the source sample n + j injected; bit j of e: data row
//              n + j from the level u^{n+j}
//   kOpAdj:    ns adjoint steps from lam^k in a and lam^{k+1} in b, k = n; step j reads u^{k-j}
//              in c[j] and injects the residual row k - j; the last level goes to d[0], the one
//              before it to d[1]
//   kOpGather: data row n from field a
//   kOpEnc:    ns fields into their streams: field c[j], less d[j] (kBufNone: whole), at
//              offs[x[j]]; the end of the last goes to offs[n], of the others to the next one's
//              offs word; y[j]: k of the stored u^k (its size is recorded), -1 none
//   kOpDec:    ns streams, at offs[x[j]], into c[j] (d[j] != kBufNone: d[j] - decoded)
//   kOpCopy:   copy field a into b
//   kOpResid:  residual r = d_sim - d_obs, partial sums of r^2, finiteness of field a
//   kOpMisfit: phi = 1/2 sum of the partials
enum BatchOpKind { kOpNop = 0, kOpStep, kOpAdj, kOpGather, kOpEnc, kOpDec, kOpCopy, kOpResid, kOpMisfit };
struct BatchOp {
    int32_t kind, n, ns, a, b, e;
    int32_t c[kTileSteps], d[kTileSteps], x[kTileSteps], y[kTileSteps];
};
static_assert(kEncJobs >= kTileSteps, "an encode or decode step is one launch");

struct BatchArgs {
    Grid g;
    CodecDims cd;
    const BatchShot *shots;
    int nshots;
    const BatchOp *ops;       // the program's ops but for its steps
    int op0, nops;            // the ops (of those that are no steps) a launch of the persistent kernel executes
    double gscale;
    double tol;
    int minexp;
    int nrec;                 // receivers per shot (every shot of a batch has as many)
    int nt;
    long long fstride;        // elements from one array of a ring to the next
    long long slot_elems;     // elements of one uncompressed checkpoint slot (two fields)
    unsigned *bar;            // device-wide barrier words: group counters, top, generation, abort (zero at launch)
    int nwg;                  // workgroups of the launch (at most what the device holds at once)
    unsigned spin_limit;      // polls before a barrier gives up and the launch aborts
};
// Workgroups the persistent kernel can keep resident (0 on error).
int batch2d_resident_workgroups();
// Launch of the persistent kernel with A.nwg workgroups.
hipError_t launch_batch2d(const BatchArgs &A, hipStream_t s);
// Launch of a group of forward or adjoint steps of every shot.
hipError_t launch_batch_steps(const BatchArgs &A, const BatchOp &op, hipStream_t s);

}  // namespace wv
