// Batched 2-D solver: one persistent kernel advances several 2-D shots together.
//
// Shots are independent (the paper computes one gradient per shot and sums them,
// Sec. "Example adjoint problem: Seismic inversion"), and small 2-D shots cannot fill
// the GPU one launch at a time: a 512^2 step is a few microseconds of work behind a
// launch of about the same cost.  So shots of one grid, space order, step count and
// checkpoint schedule run as one batch: the host turns the schedule into a program of
// phases (stencil steps, source and residual injections, checkpoint encodes and
// decodes, the misfit), and a persistent kernel, launched once for the whole reversal,
// executes every phase for every shot of the batch, with a device-wide barrier between
// phases.  Each shot's arithmetic is the solo solver's (the same point update,
// injection, gather, codec block and reduction code, in the same order), so a shot
// gives the same bits alone, in a solo call and in any batch.
#include "wv_codec_dev.h"
#include "wv_tile2d_dev.h"

namespace wv {

namespace {

constexpr int kBatchParts = 1024;   // residual partial sums per shot (as the solo misfit)
constexpr int kCopyItem = 65536;    // elements per copy or finiteness work item
// Threads of a workgroup: a region of the steps takes all of them, one row of points a
// lane; the codec's chunks and the reductions, shared with the solo path, take 256 lanes, so
// the workgroup runs them as groups.
constexpr int kBatchRows = 1, kBatchThreads = tile2d_threads(kBatchRows), kGroups = kBatchThreads / 256;
static_assert(kBatchThreads % 256 == 0, "whole groups");

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

// Device-wide barrier of the persistent launch.  Two levels: workgroup b arrives at the
// counter of its group b % 8 (the XCD it runs on under round-robin dispatch), the last
// arrival of a group at the top counter, and the last of those resets it and advances the
// generation; everyone else waits for the generation to move.  Counters, top, generation
// and the abort word sit 1 KB apart so that arrivals of different groups and the polling
// do not meet on one line.  Memory order: a release fence before each arrival, acquire +
// release fences around the group's and the top's last arrival, relaxed polling (an
// acquire poll would invalidate the L2 on every spin) and one acquire fence after the
// wait, so every write of the phase is visible to every workgroup of the next.
// The barrier needs every workgroup resident.  The spin is bounded (spin_limit polls, 2^18
// by default: a fraction of a second, where a phase takes microseconds): past the bound, or when another
// workgroup has given up, it sets err bit 16 and the abort word and returns false, and the
// kernel ends at once; the host then runs the batch's shots one by one.
__device__ __forceinline__ bool grid_barrier(unsigned *bar, unsigned nwg, unsigned spin_limit, unsigned *err,
                                             unsigned *s_flag)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned ng = nwg < 8u ? nwg : 8u;
        const unsigned grp = blockIdx.x & 7u;
        const unsigned in_grp = (nwg - grp + 7u) / 8u;
        unsigned *sub = bar + 256u * grp, *top = bar + 2048, *gen = bar + 3072, *abort = bar + 3584;
        const unsigned g0 = __hip_atomic_load(gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        bool waiting = true, ok = true;
        if (__hip_atomic_fetch_add(sub, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == in_grp - 1u) {
            __hip_atomic_store(sub, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
            if (__hip_atomic_fetch_add(top, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ng - 1u) {
                __hip_atomic_store(top, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
                __hip_atomic_fetch_add(gen, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                waiting = false;
            }
        }
        if (waiting) {
            unsigned spins = 0;
            while (__hip_atomic_load(gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == g0) {
                if (++spins > spin_limit || __hip_atomic_load(abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    atomicOr(err, 16u);
                    __hip_atomic_store(abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *s_flag = ok ? 1u : 0u;
    }
    __syncthreads();
    return *s_flag != 0u;
}

// inclusive scan of v over the group (s_scan: scratch for its wave totals); the trailing
// barrier lets the caller reuse s_scan at once
__device__ __forceinline__ unsigned block_scan(unsigned *s_scan, unsigned v, unsigned &total)
{
    const unsigned r = wg_scan256(v, s_scan, total);
    __syncthreads();
    return r;
}

// sum of w[0..n) by the group (its first wave does the adding), broadcast through *out
__device__ __forceinline__ unsigned long long block_sum_words(const uint32_t *w, long long n,
                                                              unsigned long long *out)
{
    const int tid = threadIdx.x & 255;
    if (tid < 64) {
        unsigned long long s = 0;
        for (long long i = tid; i < n; i += 64) s += w[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (tid == 0) *out = s;
    }
    __syncthreads();
    const unsigned long long r = *out;
    __syncthreads();
    return r;
}

template <bool VEC>
__device__ __forceinline__ void load_block2(const float *f, const float *sub, const CodecDims &cd, long long b,
                                            float *v)
{
    const int bx = (int)(b % cd.nb[0]);
    const int by = (int)((b / cd.nb[0]) % cd.nb[1]);
    load_block<2, VEC>(f, sub, cd.dims, cd.pitch, bx, by, 0, v);
}

// Phase bodies.  A phase runs work items item = shot * per + j over all workgroups; every
// lane of a workgroup takes part in each of its items (items hold workgroup barriers).
struct BatchCtx {
    const BatchArgs &A;
    const Grid &g;
    const CodecDims &cd;
    long long P;
    bool vec;
    long long nch;
};

template <typename Body>
__device__ __forceinline__ void for_items(const BatchArgs &A, int per, Body body)
{
    const int items = per * A.nshots;
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        const int si = it / per;
        body(A.shots[si], it - si * per);
    }
}

// A step or adjoint phase of one shot, as tile2d takes it.
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

// Forward (GRAD false) or adjoint (GRAD true) steps of every shot: one item per tile.
template <int K, bool GRAD>
__device__ __forceinline__ void phase_step(const BatchCtx &C, const BatchOp &op, Tile2dShared &S,
                                           typename Tile2dShared::template Levels<K> &L)
{
    const int core = kTileRegion - 2 * tile2d_halo(K, op.ns);
    const int tx = (C.g.nx + core - 1) / core, tz = (C.g.nz + core - 1) / core;
    for_items(C.A, tx * tz, [&](const BatchShot &shot, int j) {
        const ShotTile<GRAD> T(C.A, shot, op, C.P);
        tile2d<K, GRAD, kBatchRows>(C.g, T, j % tx, j / tx, S, L);
        __syncthreads();   // the next tile reuses the arrays
    });
}

// As for_items, an item for each group of 256 lanes; every group makes as many passes (the
// items hold workgroup barriers), on is false in those it has no item for.
template <typename Body>
__device__ __forceinline__ void for_group_items(const BatchArgs &A, int per, Body body)
{
    const int items = per * A.nshots;
    for (int i0 = blockIdx.x * kGroups; i0 < items; i0 += gridDim.x * kGroups) {
        const int it = i0 + (int)(threadIdx.x >> 8);
        const bool on = it < items;
        const int si = on ? it / per : 0;
        body(A.shots[si], on ? it - si * per : 0, on);
    }
}

// One workgroup per shot: the receivers of `gin` into data row `grow`.
__device__ __forceinline__ void phase_gather(const BatchCtx &C, int gin, int grow)
{
    const BatchArgs &A = C.A;
    for_items(A, 1, [&](const BatchShot &S, int) {
        const float *f = batch_buf(A, S, gin, C.P);
        for (int r = threadIdx.x; r < A.nrec; r += kBatchThreads) S.dsim[(long long)grow * A.nrec + r] = gather_point(S.rec, r, f);
    });
}

// s_scan, s_words and s_one are the group's own.
__device__ __forceinline__ void phase_encode(const BatchCtx &C, const BatchOp &op, bool emit, unsigned *s_scan,
                             unsigned long long *s_words, unsigned long long *s_one)
{
    const BatchArgs &A = C.A;
    const CodecDims &cd = C.cd;
    const long long nch = C.nch;
    const int tid = threadIdx.x & 255;
    for_group_items(A, (int)(op.ns * nch), [&](const BatchShot &S, int j, bool on) {
        const int f = (int)(j / nch);
        const long long c = j - (long long)f * nch;
        const float *field = batch_buf(A, S, op.c[f], C.P);
        const float *sub = batch_buf(A, S, op.d[f], C.P);
        const long long b = c * kBlocksPerChunk + tid;
        const bool valid = on && b < cd.nblocks;
        float v[16];
        if (valid) {
            if (C.vec) load_block2<true>(field, sub, cd, b, v);
            else load_block2<false>(field, sub, cd, b, v);
        } else {
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = 0.0f;
        }
        BlockEnc<2> blk;
        uint32_t m_lo[32], m_hi[32];
        blk.prepare(v, valid, A.minexp, m_lo, m_hi);
        const unsigned nbits = blk.count(m_lo, m_hi);
        unsigned total_bits;
        const unsigned incl = block_scan(s_scan, nbits, total_bits);
        const uint32_t chunk_words = (total_bits + 63u) / 64u;
        if (!emit) {
            if (on && !blk.finite) atomicOr(S.err, 2u);
            if (on && tid == 0) S.chunk_words[(long long)f * nch + c] = chunk_words;
            return;
        }
        // the first field's stream starts at its offset word, each other one where the one
        // before it ends, rounded up to 256 bytes
        uint64_t base = S.offs[op.x[0]];
        unsigned long long fwords = 0;
        for (int q = 0; q < op.ns; ++q) {
            const unsigned long long words = block_sum_words(S.chunk_words + q * nch, nch, s_one);
            if (q < f) base += (cd.prefix_bytes + 8ull * words + 255ull) & ~255ull;
            if (q == f) fwords = words;
        }
        const unsigned long long excl = block_sum_words(S.chunk_words + (long long)f * nch, c, s_one);
        const uint64_t cap = S.arena_bytes;
        const bool prefix_fits = on && base + (uint64_t)cd.prefix_bytes <= cap;
        const bool fits = prefix_fits && base + (uint64_t)cd.prefix_bytes + (excl + chunk_words) * 8ull <= cap;
        uint8_t *hdr = S.arena + base;
        uint64_t *chunk_off = (uint64_t *)(hdr + 64);
        uint16_t *lens = (uint16_t *)(hdr + 64 + 8 * nch);
        if (valid && prefix_fits) lens[b] = (uint16_t)nbits;
        if (tid == 0 && prefix_fits) chunk_off[c] = excl;
        if (on && tid == 0 && !fits) atomicOr(S.err, 4u);
        unsigned long long *data = (unsigned long long *)(hdr + cd.prefix_bytes) + excl;
        const unsigned excl_bits = incl - nbits;
        const bool staged = fits && chunk_words <= (uint32_t)kLdsWords;
        unsigned long long *words = staged ? s_words : data;
        if (fits)
            for (uint32_t q = tid; q < chunk_words; q += 256) words[q] = 0ull;
        __syncthreads();
        if (valid && staged) {
            auto sink = [&](long long w, unsigned long long bits) { atomicOr(&s_words[w], bits); };
            blk.emit((long long)excl_bits, sink, m_lo, m_hi);
        } else if (valid && fits) {
            auto sink = [&](long long w, unsigned long long bits) { atomicOr(&data[w], bits); };
            blk.emit((long long)excl_bits, sink, m_lo, m_hi);
        }
        __syncthreads();
        if (staged)
            for (uint32_t q = tid; q < chunk_words; q += 256) data[q] = s_words[q];
        __syncthreads();
        if (on && c == nch - 1 && tid == 0) {
            const unsigned long long total = (unsigned long long)cd.prefix_bytes + 8ull * fwords;
            if (prefix_fits) {
                uint32_t *h32 = (uint32_t *)hdr;
                h32[0] = kMagic;
                h32[1] = kVersion;
                h32[2] = 2u;
                h32[3] = (uint32_t)cd.dims[0];
                h32[4] = (uint32_t)cd.dims[1];
                h32[5] = (uint32_t)cd.dims[2];
                *(double *)(hdr + 24) = A.tol;
                h32[8] = (uint32_t)cd.nblocks;
                h32[9] = (uint32_t)nch;
                h32[10] = kBlocksPerChunk;
                h32[11] = 0;
                *(unsigned long long *)(hdr + 48) = fwords;
                *(unsigned long long *)(hdr + 56) = total;
                const long long lb = 64 + 8 * nch + 2 * cd.nblocks;
                for (long long q = lb; q < cd.prefix_bytes; ++q) hdr[q] = 0;
            }
            const unsigned long long nxt = base + ((total + 255ull) & ~255ull);
            S.offs[f + 1 < op.ns ? op.x[f + 1] : op.n] = nxt;
            if (op.y[f] >= 0) S.sizes[op.y[f]] = total;
            atomicAdd(&S.stats[0], total);
            atomicMax(&S.stats[1], nxt);
        }
    });
}

__device__ __forceinline__ void phase_decode(const BatchCtx &C, const BatchOp &op, unsigned *s_scan, unsigned long long *s_words)
{
    const BatchArgs &A = C.A;
    const CodecDims &cd = C.cd;
    const long long nch = C.nch;
    const int tid = threadIdx.x & 255;
    for_group_items(A, (int)(op.ns * nch), [&](const BatchShot &S, int j, bool on) {
        const int f = (int)(j / nch);
        float *field = batch_buf(A, S, op.c[f], C.P);
        const float *sub = batch_buf(A, S, op.d[f], C.P);
        const long long c = j - (long long)f * nch;
        const long long b = c * kBlocksPerChunk + tid;
        const bool valid = on && b < cd.nblocks;
        const uint64_t boff = S.offs[op.x[f]];
        const uint64_t cap = S.arena_bytes;
        // a stream outside the arena (an overflowed store) decodes to zeros, as in the solo decoder
        const bool fits = boff + (uint64_t)cd.prefix_bytes <= cap;
        const uint8_t *hdr = S.arena + (fits ? boff : 0);
        const uint64_t *chunk_off = (const uint64_t *)(hdr + 64);
        const uint16_t *lens = (const uint16_t *)(hdr + 64 + 8 * nch);
        const unsigned long long *data = (const unsigned long long *)(hdr + cd.prefix_bytes);
        long long nwords = 0, cbase = 0;
        int minexp = 0;
        if (fits) {
            nwords = (long long)*(const unsigned long long *)(hdr + 48);
            const long long maxw = (long long)((cap - boff - (uint64_t)cd.prefix_bytes) / 8);
            nwords = nwords < maxw ? nwords : maxw;
            int te;
            frexp(*(const double *)(hdr + 24), &te);
            minexp = te - 1;
            cbase = (long long)chunk_off[c];
            cbase = cbase < 0 ? 0 : (cbase > nwords ? nwords : cbase);
        }
        const unsigned nbits = valid && fits ? lens[b] : 0u;
        unsigned total_bits;
        const unsigned incl = block_scan(s_scan, nbits, total_bits);
        const long long cw = ((long long)total_bits + 63) / 64 + 1;
        const bool staged = cw <= kDecLdsWords;
        if (staged) {
            for (long long q = tid; q < cw + kDecPad; q += 256) {
                const long long jw = cbase + q;
                s_words[q] = (q < cw && jw >= 0 && jw < nwords) ? data[jw] : 0ull;
            }
        }
        __syncthreads();
        if (valid) {
            float out[16];
            if (fits) {
                const long long rel = (long long)(incl - nbits);
                if (staged) {
                    LdsReader rd{reinterpret_cast<const uint32_t *>(s_words), 2 * (int)cw, (int)rel};
                    decode_block<2>(rd, minexp, out);
                } else {
                    GlobalReader rd{data, nwords, 0, 0ull, 0ull, 0};
                    rd.init(cbase * 64 + rel);
                    decode_block<2>(rd, minexp, out);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 16; ++q) out[q] = 0.0f;
            }
            if (C.vec) store_block<2, true>(field, sub, cd.dims, cd.pitch, cd.nb, b, out);
            else store_block<2, false>(field, sub, cd.dims, cd.pitch, cd.nb, b, out);
        }
        __syncthreads();
    });
}

// residual r = d_sim - d_obs and its partial sums of r^2 (the solo misfit's blocks and
// order), plus the finiteness check of the last forward state (field a)
// s_red is the group's own.
__device__ __forceinline__ void phase_residual(const BatchCtx &C, int ufield, double *s_red)
{
    const BatchArgs &A = C.A;
    const int tid = threadIdx.x & 255;
    const int nfin = (int)((C.P + kCopyItem - 1) / kCopyItem);
    for_group_items(A, kBatchParts + nfin, [&](const BatchShot &S, int j, bool on) {
        const bool part = on && j < kBatchParts;
        double acc = 0.0;
        if (part) {
            const long long n = (long long)(A.nt + 1) * A.nrec;
            for (long long e = (long long)j * 256 + tid; e < n; e += (long long)kBatchParts * 256) {
                if (e < A.nrec) {
                    S.res[e] = 0.0f;
                    continue;
                }
                const double r = (double)S.dsim[e] - (double)S.dobs[e];
                S.res[e] = (float)r;
                acc += r * r;
            }
        } else if (on) {
            const float *u = batch_buf(A, S, ufield, C.P);
            const long long e0 = (long long)(j - kBatchParts) * kCopyItem, e1 = min(e0 + kCopyItem, C.P);
            bool bad = false;
            for (long long e = e0 + tid; e < e1; e += 256) bad |= !isfinite(u[e]);
            if (bad) atomicOr(S.err, 8u);
        }
        s_red[tid] = acc;
        __syncthreads();
        for (int sft = 128; sft > 0; sft >>= 1) {
            if (tid < sft) s_red[tid] += s_red[tid + sft];
            __syncthreads();
        }
        if (part && tid == 0) S.partials[j] = s_red[0];
        __syncthreads();
    });
}

// phi = 1/2 sum of the partials (the solo final sum's order)
__device__ __forceinline__ void phase_misfit(const BatchCtx &C, double *s_red)
{
    const int tid = threadIdx.x & 255;
    for_group_items(C.A, 1, [&](const BatchShot &S, int, bool on) {
        double acc = 0.0;
        if (on)
            for (int q = tid; q < kBatchParts; q += 256) acc += S.partials[q];
        s_red[tid] = acc;
        __syncthreads();
        for (int sft = 128; sft > 0; sft >>= 1) {
            if (tid < sft) s_red[tid] += s_red[tid + sft];
            __syncthreads();
        }
        if (on && tid == 0) S.misfit[0] = 0.5 * s_red[0];
        __syncthreads();
    });
}

__device__ __forceinline__ void phase_copy(const BatchCtx &C, int src, int dst)
{
    const BatchArgs &A = C.A;
    for_items(A, (int)((C.P + kCopyItem - 1) / kCopyItem), [&](const BatchShot &S, int j) {
        const float *a = batch_buf(A, S, src, C.P);
        float *b = batch_buf(A, S, dst, C.P);
        const long long e0 = (long long)j * kCopyItem, e1 = min(e0 + kCopyItem, C.P);
        for (long long e = e0 + threadIdx.x; e < e1; e += kBatchThreads) b[e] = a[e];
    });
}

template <int K>
__global__ __launch_bounds__(kBatchThreads) void batch2d_kernel(BatchArgs A)
{
    // the tile's levels and the codec's words are never live together (a barrier lies between)
    using Levels = typename Tile2dShared::template Levels<K>;
    constexpr size_t kCodec = 8 * (kDecLdsWords + kDecPad) * kGroups;
    constexpr size_t kPool = sizeof(Levels) > kCodec ? sizeof(Levels) : kCodec;
    __shared__ __align__(16) unsigned char s_pool[kPool];
    __shared__ __align__(16) Tile2dShared s_tile;
    Levels &s_levels = *reinterpret_cast<Levels *>(s_pool);
    const int grp = threadIdx.x >> 8;
    unsigned long long *s_words = reinterpret_cast<unsigned long long *>(s_pool) + grp * (kDecLdsWords + kDecPad);
    __shared__ unsigned s_scan_[kGroups][4];
    __shared__ unsigned long long s_one[kGroups];
    __shared__ double s_red_[kGroups][256];
    unsigned *s_scan = s_scan_[grp];
    double *s_red = s_red_[grp];
    const BatchCtx C{A, A.g, A.cd, A.g.P, A.cd.dims[0] % 4 == 0 && A.cd.pitch % 4 == 0, A.cd.nchunks};
    __shared__ unsigned s_flag;
    unsigned *err0 = A.shots[0].err;
    auto barrier = [&]() { return grid_barrier(A.bar, (unsigned)A.nwg, A.spin_limit, err0, &s_flag); };

    for (int oi = 0; oi < A.nops; ++oi) {
        const BatchOp &op = A.ops[oi];
        switch (op.kind) {
        case kOpStep:
            phase_step<K, false>(C, op, s_tile, s_levels);
            if (!barrier()) return;
            break;
        case kOpAdj:
            phase_step<K, true>(C, op, s_tile, s_levels);
            if (!barrier()) return;
            break;
        case kOpGather:
            phase_gather(C, op.a, op.n);
            if (!barrier()) return;
            break;
        case kOpEnc:
            phase_encode(C, op, false, s_scan, s_words, &s_one[grp]);
            if (!barrier()) return;
            phase_encode(C, op, true, s_scan, s_words, &s_one[grp]);
            if (!barrier()) return;
            break;
        case kOpDec:
            phase_decode(C, op, s_scan, s_words);
            if (!barrier()) return;
            break;
        case kOpCopy:
            phase_copy(C, op.a, op.b);
            if (!barrier()) return;
            break;
        case kOpResid:
            phase_residual(C, op.a, s_red);
            if (!barrier()) return;
            break;
        case kOpMisfit:
            phase_misfit(C, s_red);
            if (!barrier()) return;
            break;
        default:
            break;
        }
    }
}

template <int K>
int resident_of()
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batch2d_kernel<K>, kBatchThreads, 0) != hipSuccess) return 0;
    return cus * per_cu;
}

// A plain launch: the grid is at most what the device holds at once, and a barrier that
// does not complete (workgroups kept out by other streams' kernels) aborts the launch.
template <int K>
hipError_t launch_of(const BatchArgs &A, hipStream_t s)
{
    hipLaunchKernelGGL(batch2d_kernel<K>, dim3(A.nwg), dim3(kBatchThreads), 0, s, A);
    return hipGetLastError();
}

}  // namespace

int batch2d_resident_workgroups(int K)
{
    switch (K) {
    case 1: return resident_of<1>();
    case 2: return resident_of<2>();
    case 3: return resident_of<3>();
    case 4: return resident_of<4>();
    case 5: return resident_of<5>();
    case 6: return resident_of<6>();
    case 7: return resident_of<7>();
    case 8: return resident_of<8>();
    default: return 0;
    }
}

hipError_t launch_batch2d(const BatchArgs &A, int K, hipStream_t s)
{
    switch (K) {
    case 1: return launch_of<1>(A, s);
    case 2: return launch_of<2>(A, s);
    case 3: return launch_of<3>(A, s);
    case 4: return launch_of<4>(A, s);
    case 5: return launch_of<5>(A, s);
    case 6: return launch_of<6>(A, s);
    case 7: return launch_of<7>(A, s);
    case 8: return launch_of<8>(A, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace wv
