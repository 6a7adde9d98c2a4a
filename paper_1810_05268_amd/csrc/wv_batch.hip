// Batched 2-D solver: several 2-D shots advanced together.
//
// Shots are independent (the paper computes one gradient per shot and sums them,
// Sec. "Example adjoint problem: Seismic inversion"), and small 2-D shots cannot fill
// the GPU one at a time.  So shots of one grid, space order, step count and checkpoint
// schedule run as one batch: the host turns the schedule into a program (see Prog2d), whose
// groups of forward or adjoint steps are one launch each, over the tiles of every shot, and
// whose runs of other steps between them (encodes, decodes, copies, gathers, the residual and
// the misfit) one launch of the persistent kernel below, which executes its phases for every
// shot with a device-wide barrier between them.  Each shot's arithmetic is the solo solver's
// (the same tile, gather, codec block and reduction code, in the same order), so a shot
// gives the same bits alone, in a solo call and in any batch.
//
// With the steps in the persistent kernel too, one launch for a whole reversal, eight shots
// of 552^2 points at order 8, 300 steps, took 24.4 ms, and take 16.6 this way: its barrier
// costs 6 us more than a launch, and the codec's registers leave the tiles 8 waves a CU.
#include "wv_codec_dev.h"
#include "wv_tile2d_dev.h"

namespace wv {

namespace {

constexpr int kBatchParts = 1024;   // residual partial sums per shot (as the solo misfit)
constexpr int kCopyItem = 65536;    // elements per copy or finiteness work item
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

// inclusive workgroup scan of v (s_scan: scratch for the wave totals); the trailing
// barrier lets the caller reuse s_scan at once
__device__ __forceinline__ unsigned block_scan(unsigned *s_scan, unsigned v, unsigned &total)
{
    const unsigned r = wg_scan256(v, s_scan, total);
    __syncthreads();
    return r;
}

// sum of w[0..n) by one workgroup (wave 0 does the adding), broadcast through *out
__device__ __forceinline__ unsigned long long block_sum_words(const uint32_t *w, long long n,
                                                              unsigned long long *out)
{
    if (threadIdx.x < 64) {
        unsigned long long s = 0;
        for (long long i = threadIdx.x; i < n; i += 64) s += w[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (threadIdx.x == 0) *out = s;
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

// One workgroup per shot: the receivers of `gin` into data row `grow`.
__device__ __forceinline__ void phase_gather(const BatchCtx &C, int gin, int grow)
{
    const BatchArgs &A = C.A;
    for_items(A, 1, [&](const BatchShot &S, int) {
        const float *f = batch_buf(A, S, gin, C.P);
        for (int r = threadIdx.x; r < A.nrec; r += 256) S.dsim[(long long)grow * A.nrec + r] = gather_point(S.rec, r, f);
    });
}

__device__ __forceinline__ void phase_encode(const BatchCtx &C, const BatchOp &op, bool emit, unsigned *s_scan,
                             unsigned long long *s_words, unsigned long long *s_one)
{
    const BatchArgs &A = C.A;
    const CodecDims &cd = C.cd;
    const long long nch = C.nch;
    const int tid = threadIdx.x;
    for_items(A, (int)(op.ns * nch), [&](const BatchShot &S, int j) {
        const int f = (int)(j / nch);
        const long long c = j - (long long)f * nch;
        const float *field = batch_buf(A, S, op.c[f], C.P);
        const float *sub = batch_buf(A, S, op.d[f], C.P);
        const long long b = c * kBlocksPerChunk + tid;
        const bool valid = b < cd.nblocks;
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
            if (!blk.finite) atomicOr(S.err, 2u);
            if (tid == 0) S.chunk_words[(long long)f * nch + c] = chunk_words;
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
        const bool prefix_fits = base + (uint64_t)cd.prefix_bytes <= cap;
        const bool fits = prefix_fits && base + (uint64_t)cd.prefix_bytes + (excl + chunk_words) * 8ull <= cap;
        uint8_t *hdr = S.arena + base;
        uint64_t *chunk_off = (uint64_t *)(hdr + 64);
        uint16_t *lens = (uint16_t *)(hdr + 64 + 8 * nch);
        if (valid && prefix_fits) lens[b] = (uint16_t)nbits;
        if (tid == 0 && prefix_fits) chunk_off[c] = excl;
        if (tid == 0 && !fits) atomicOr(S.err, 4u);
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
        if (c == nch - 1 && tid == 0) {
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
    const int tid = threadIdx.x;
    for_items(A, (int)(op.ns * nch), [&](const BatchShot &S, int j) {
        const int f = (int)(j / nch);
        float *field = batch_buf(A, S, op.c[f], C.P);
        const float *sub = batch_buf(A, S, op.d[f], C.P);
        const long long c = j - (long long)f * nch;
        const long long b = c * kBlocksPerChunk + tid;
        const bool valid = b < cd.nblocks;
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
__device__ __forceinline__ void phase_residual(const BatchCtx &C, int ufield, double *s_red)
{
    const BatchArgs &A = C.A;
    const int tid = threadIdx.x;
    const int nfin = (int)((C.P + kCopyItem - 1) / kCopyItem);
    for_items(A, kBatchParts + nfin, [&](const BatchShot &S, int j) {
        const bool part = j < kBatchParts;
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
        } else {
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
    const int tid = threadIdx.x;
    for_items(C.A, 1, [&](const BatchShot &S, int) {
        double acc = 0.0;
        for (int q = tid; q < kBatchParts; q += 256) acc += S.partials[q];
        s_red[tid] = acc;
        __syncthreads();
        for (int sft = 128; sft > 0; sft >>= 1) {
            if (tid < sft) s_red[tid] += s_red[tid + sft];
            __syncthreads();
        }
        if (tid == 0) S.misfit[0] = 0.5 * s_red[0];
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
        for (long long e = e0 + threadIdx.x; e < e1; e += 256) b[e] = a[e];
    });
}

// Ops A.op0 .. A.op0 + A.nops - 1 of those the persistent kernel runs (no forward or adjoint steps).  Once a
// barrier of an earlier launch has given up, the abort word keeps the later ones from running.
__global__ __launch_bounds__(256) void batch2d_kernel(BatchArgs A)
{
    __shared__ unsigned s_scan[4];
    __shared__ unsigned long long s_words[kDecLdsWords + kDecPad];
    __shared__ unsigned long long s_one;
    __shared__ double s_red[256];
    __shared__ unsigned s_flag;
    const BatchCtx C{A, A.g, A.cd, A.g.P, A.cd.dims[0] % 4 == 0 && A.cd.pitch % 4 == 0, A.cd.nchunks};
    unsigned *err0 = A.shots[0].err;
    auto barrier = [&]() { return grid_barrier(A.bar, (unsigned)A.nwg, A.spin_limit, err0, &s_flag); };
    if (threadIdx.x == 0) s_flag = __hip_atomic_load(A.bar + 3584, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_flag != 0u) return;
    __syncthreads();

    for (int oi = A.op0; oi < A.op0 + A.nops; ++oi) {
        if (oi > A.op0 && !barrier()) return;
        const BatchOp &op = A.ops[oi];
        switch (op.kind) {
        case kOpGather: phase_gather(C, op.a, op.n); break;
        case kOpEnc:
            phase_encode(C, op, false, s_scan, s_words, &s_one);
            if (!barrier()) return;
            phase_encode(C, op, true, s_scan, s_words, &s_one);
            break;
        case kOpDec: phase_decode(C, op, s_scan, s_words); break;
        case kOpCopy: phase_copy(C, op.a, op.b); break;
        case kOpResid: phase_residual(C, op.a, s_red); break;
        case kOpMisfit: phase_misfit(C, s_red); break;
        default: break;
        }
    }
}

}  // namespace

int batch2d_resident_workgroups()
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batch2d_kernel, 256, 0) != hipSuccess) return 0;
    return device_cus() * per_cu;
}

// A plain launch: the grid is at most what the device holds at once, and a barrier that
// does not complete (workgroups kept out by other streams' kernels) aborts the launch.
hipError_t launch_batch2d(const BatchArgs &A, hipStream_t s)
{
    hipLaunchKernelGGL(batch2d_kernel, dim3(A.nwg), dim3(256), 0, s, A);
    return hipGetLastError();
}

}  // namespace wv
