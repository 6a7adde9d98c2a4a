// ZFP-kind fixed-accuracy codec for binary32 checkpoints (gfx950).
//
// The paper stores every checkpoint through ZFP in its fixed-tolerance mode, i.e.
// with an absolute error bound (Sec. "Lossy Compression").  This codec follows the
// published ZFP block scheme (Lindstrom 2014): 4^d blocks, a common block exponent,
// block-floating-point integers, a separable decorrelating lifting transform, a
// sequency reordering, negabinary coefficients and embedded bit-plane coding with
// group tests, truncated at the plane that guarantees the tolerance.  The stream
// container is this library's own (documented in wv.h), designed for the GPU:
//   * one lane encodes one block, so a 256-lane workgroup encodes a chunk of 256
//     blocks; a block's bit length has a closed form per bit plane, so each lane
//     first counts its bits and the workgroup scans them;
//   * up to three launches place the chunks: every chunk counts its words and assembles
//     its bits at chunk-local positions in a staging slot; one workgroup scans the
//     word counts into offsets (in fields of few chunks each chunk sums the counts before
//     it instead); every chunk copies its slot to its offset (a chunk
//     longer than a slot, or every chunk without staging, is encoded again there).
//     No workgroup waits for another: a single pass with a look-back over the
//     preceding chunks spent most of its time in those waits, each a trip to memory;
//   * chunks start at 64-bit word boundaries and record their word offsets, so the
//     decoder needs only a per-chunk scan of the 16-bit block lengths and every
//     block decodes independently.
#include <algorithm>

#include "wv_codec_dev.h"

namespace wv {

namespace {

struct EncArgs {
    EncJob job[kEncJobs];    // the fields of the launch
    bool chain[kEncJobs];    // job e starts where job e - 1 ends
    int dims[3];
    int pitch;               // elements between rows of field and sub
    int nb[3];
    long long nblocks, nchunks, prefix_bytes;
    int ndim;
    int minexp;
    double tol;
    uint8_t *out;
    uint64_t cap;
    uint32_t *words;         // per job and chunk: its stream words
    uint64_t *offs;          // per job and chunk: its first word in the data area
    unsigned long long *staging;   // nullable: slot_words words per job and chunk
    uint16_t *lens;          // with staging: per job and block, its length (the stream's place for
                             // them is known after the scan)
    int slot_words;
    unsigned *err;
    unsigned long long *stats;
};

// The blocks of chunk c: values, exponent, transform, planes and bit counts, and the
// workgroup scan of the counts; returns whether the lane has a block.  The planes are
// the caller's local arrays (inside a struct they would be placed in scratch).  Every
// lane of the workgroup calls it.
template <int ND, bool VEC>
__device__ __forceinline__ bool chunk_prepare(const EncArgs &A, int job, long long c, BlockEnc<ND> &blk,
                                              uint32_t (&m_lo)[32], uint32_t (&m_hi)[32], unsigned &nbits,
                                              unsigned &excl_bits, unsigned &total_bits, unsigned *s_scan)
{
    constexpr int S = ND == 3 ? 64 : 16;
    const long long b = c * kBlocksPerChunk + threadIdx.x;
    const bool valid = b < A.nblocks;
    float v[S];
    if (valid) {
        const int bx = (int)(b % A.nb[0]);
        const int by = (int)((b / A.nb[0]) % A.nb[1]);
        const int bz = (int)(b / ((long long)A.nb[0] * A.nb[1]));
        load_block<ND, VEC>(A.job[job].field, A.job[job].sub, A.dims, A.pitch, bx, by, bz, v);
    } else {
#pragma unroll
        for (int i = 0; i < S; ++i) v[i] = 0.0f;
    }
    blk.prepare(v, valid, A.minexp, m_lo, m_hi);
    nbits = blk.count(m_lo, m_hi);
    excl_bits = wg_scan256(nbits, s_scan, total_bits) - nbits;
    return valid;
}

// Sum of w[0..n) over the workgroup's lanes.
__device__ __forceinline__ unsigned long long wg_total(const uint32_t *w, long long n, unsigned long long *s_scan)
{
    unsigned long long v = 0, total;
    for (long long i = threadIdx.x; i < n; i += 256) v += w[i];
    (void)wg_scan256(v, s_scan, total);
    __syncthreads();
    return total;
}

// Where job e's stream starts: its own offset word, or the end of the jobs it follows.
__device__ __forceinline__ uint64_t job_base(const EncArgs &A, int e, unsigned long long *s_scan)
{
    int f = e;
    while (f > 0 && A.chain[f]) --f;
    uint64_t base = *A.job[f].base;
    for (; f < e; ++f) {
        const unsigned long long words = wg_total(A.words + f * A.nchunks, A.nchunks, s_scan);
        base += ((uint64_t)A.prefix_bytes + 8ull * words + 255ull) & ~255ull;
    }
    return base;
}

// Job e's header, stream size and next free offset (one lane).
__device__ __forceinline__ void write_header(const EncArgs &A, int e, uint64_t base, unsigned long long data_words)
{
    const bool prefix_fits = base + (uint64_t)A.prefix_bytes <= A.cap;
    uint8_t *hdr = A.out + base;
    const unsigned long long total = (unsigned long long)A.prefix_bytes + 8ull * data_words;
    if (!prefix_fits || base + total > A.cap) atomicOr(A.err, 4u);
    if (prefix_fits) {
        uint32_t *h32 = (uint32_t *)hdr;
        h32[0] = kMagic;
        h32[1] = kVersion;
        h32[2] = (uint32_t)A.ndim;
        h32[3] = (uint32_t)A.dims[0];
        h32[4] = (uint32_t)A.dims[1];
        h32[5] = (uint32_t)A.dims[2];
        *(double *)(hdr + 24) = A.tol;
        h32[8] = (uint32_t)A.nblocks;
        h32[9] = (uint32_t)A.nchunks;
        h32[10] = kBlocksPerChunk;
        h32[11] = 0;
        *(unsigned long long *)(hdr + 48) = data_words;
        *(unsigned long long *)(hdr + 56) = total;
        // zero the padding after the block lengths
        const long long lb = kHdr + 8 * A.nchunks + 2 * A.nblocks;
        for (long long i = lb; i < A.prefix_bytes; ++i) hdr[i] = 0;
    }
    const unsigned long long nxt = base + ((total + 255ull) & ~255ull);
    *A.job[e].next = nxt;
    if (A.job[e].size_out) *A.job[e].size_out = total;
    atomicAdd(&A.stats[0], total);
    atomicMax(&A.stats[1], nxt);
}

// Exclusive scan of job e's chunk word counts into offs (and the stream's chunk offsets),
// then the header, the stream size and the next free offset; one workgroup.  Each lane
// sums a run of up to 16 counts held in registers.
__device__ __forceinline__ void scan_chunks(const EncArgs &A, int e, unsigned long long *s_scan)
{
    const int tid = threadIdx.x;
    const long long n = A.nchunks;
    const uint64_t base = job_base(A, e, s_scan);
    uint64_t *__restrict__ offs = A.offs + e * n;
    const long long per = (n + 1023) / 1024 * 4;   // a multiple of 4: whole uint4 loads
    const long long i0 = min((long long)tid * per, n), i1 = min(i0 + per, n);
    const uint32_t *__restrict__ words = A.words + e * n;
    constexpr int kReg = 16;
    uint32_t wr[kReg];
    const bool in_reg = per <= kReg && i1 - i0 == per && (e * n) % 4 == 0;
    unsigned long long part = 0;
    if (in_reg) {
        const uint4 *w4 = reinterpret_cast<const uint4 *>(words + i0);   // 16-byte aligned
#pragma unroll
        for (int q = 0; q < kReg / 4; ++q) {
            const uint4 t = q < per / 4 ? w4[q] : make_uint4(0u, 0u, 0u, 0u);
            wr[4 * q] = t.x;
            wr[4 * q + 1] = t.y;
            wr[4 * q + 2] = t.z;
            wr[4 * q + 3] = t.w;
        }
#pragma unroll
        for (int k = 0; k < kReg; ++k) part += wr[k];
    } else {
        for (long long i = i0; i < i1; ++i) part += words[i];
    }
    unsigned long long data_words;
    unsigned long long run = wg_scan256(part, s_scan, data_words) - part;
    const bool prefix_fits = base + (uint64_t)A.prefix_bytes <= A.cap;
    uint8_t *hdr = A.out + base;
    uint64_t *chunk_off = (uint64_t *)(hdr + kHdr);
    if (in_reg) {
#pragma unroll
        for (int k = 0; k < kReg; ++k)
            if (k < per) {
                offs[i0 + k] = run;
                if (prefix_fits) chunk_off[i0 + k] = run;
                run += wr[k];
            }
    } else {
        for (long long i = i0; i < i1; ++i) {
            offs[i] = run;
            if (prefix_fits) chunk_off[i] = run;
            run += words[i];
        }
    }
    if (tid != 0) return;
    write_header(A, e, base, data_words);
}

// A 400^3 field of 11.4 MB: 76 us (2270 vector instructions a wave; 97 us and 3090 before the
// exponents came from one maximum of the magnitudes, the transposes were bit inserts, and a
// plane's groups were put out in one piece).
// Pass 1, one workgroup per chunk (and field): the block lengths, the chunk's word count, and, when it fits a staging slot, the chunk's bits, assembled in
// LDS at chunk-local positions.  Chunks are independent: no workgroup waits for another.
template <int ND, bool VEC>
__global__ __launch_bounds__(256, 4) void encode_count_kernel(EncArgs A)
{
    __shared__ unsigned s_scan[4];
    __shared__ unsigned long long s_bits[kLdsWords];
    const int tid = threadIdx.x;
    const long long c = blockIdx.x;
    const int e = blockIdx.y;
    BlockEnc<ND> blk;
    uint32_t m_lo[32], m_hi[32];
    unsigned nbits, excl_bits, total_bits;
    const bool valid = chunk_prepare<ND, VEC>(A, e, c, blk, m_lo, m_hi, nbits, excl_bits, total_bits, s_scan);
    if (!blk.finite) atomicOr(A.err, 2u);
    const long long b = c * kBlocksPerChunk + tid;
    if (valid && A.staging) {
        A.lens[e * A.nblocks + b] = (uint16_t)nbits;
    } else if (valid) {   // a single field, whose place is known
        const uint64_t base = *A.job[0].base;
        if (base + (uint64_t)A.prefix_bytes <= A.cap)
            ((uint16_t *)(A.out + base + kHdr + 8 * A.nchunks))[b] = (uint16_t)nbits;
    }
    const uint32_t cw = (total_bits + 63u) / 64u;
    if (tid == 0) A.words[e * A.nchunks + c] = cw;
    if (A.staging && cw <= (uint32_t)A.slot_words) {   // else encoded again by pass 3
        for (uint32_t i = tid; i < cw; i += 256) s_bits[i] = 0ull;
        __syncthreads();
        if (valid) {
            auto sink = [&](long long w, unsigned long long bits) { atomicOr(&s_bits[w], bits); };
            blk.emit((long long)excl_bits, sink, m_lo, m_hi);
        }
        __syncthreads();
        unsigned long long *slot = A.staging + (e * A.nchunks + c) * (long long)A.slot_words;
        for (uint32_t i = tid; i < cw; i += 256) slot[i] = s_bits[i];
    }
}

// Pass 2, one workgroup per field: the offsets scan (a kernel of its own: finishing pass 1 with a
// last-workgroup scan needs an agent-scope release in every workgroup, each an L2
// write-back, which cost more than this launch).
__global__ __launch_bounds__(256) void encode_scan_kernel(EncArgs A)
{
    __shared__ unsigned long long s_scan64[4];
    scan_chunks(A, blockIdx.x, s_scan64);
}

// Pass 3, one workgroup per chunk: a staged chunk is copied to its offset; a chunk too
// long for its slot (or every chunk, without staging) is encoded again and emitted there.
// SCAN (fields of few chunks): there is no pass 2, every workgroup sums the counts before
// its chunk itself, and a field's last one writes the header.  For a field of 75 chunks the
// launch saved, 4.5 us and a gap, was a sixth of its encode; from about a thousand chunks on
// the sums cost as much.
template <int ND, bool VEC, bool SCAN>
__global__ __launch_bounds__(256) void encode_place_kernel(EncArgs A)
{
    __shared__ unsigned s_scan[4];
    const int tid = threadIdx.x;
    const long long c = blockIdx.x;
    const int e = blockIdx.y;
    const uint32_t cw = A.words[e * A.nchunks + c];
    uint64_t base;
    unsigned long long off;
    if constexpr (SCAN) {
        __shared__ unsigned long long s_scan64[4];
        base = job_base(A, e, s_scan64);
        off = wg_total(A.words + e * A.nchunks, c, s_scan64);
        if (tid == 0) {
            if (base + (uint64_t)A.prefix_bytes <= A.cap) ((uint64_t *)(A.out + base + kHdr))[c] = off;
            if (c == A.nchunks - 1) write_header(A, e, base, off + cw);
        }
    } else {
        base = *A.job[e].base;   // pass 2 has written the bases that follow another field
        off = A.offs[e * A.nchunks + c];
    }
    if (A.staging && base + (uint64_t)A.prefix_bytes <= A.cap) {
        const long long b = c * kBlocksPerChunk + tid;
        if (b < A.nblocks) ((uint16_t *)(A.out + base + kHdr + 8 * A.nchunks))[b] = A.lens[e * A.nblocks + b];
    }
    if (base + (uint64_t)A.prefix_bytes + (off + cw) * 8ull > A.cap) return;   // write_header flags it
    unsigned long long *data = (unsigned long long *)(A.out + base + A.prefix_bytes) + off;
    if (A.staging && cw <= (uint32_t)A.slot_words) {
        const unsigned long long *slot = A.staging + (e * A.nchunks + c) * (long long)A.slot_words;
        for (uint32_t i = tid; i < cw; i += 256) data[i] = slot[i];
        return;
    }
    BlockEnc<ND> blk;
    uint32_t m_lo[32], m_hi[32];
    unsigned nbits, excl_bits, total_bits;
    const bool valid = chunk_prepare<ND, VEC>(A, e, c, blk, m_lo, m_hi, nbits, excl_bits, total_bits, s_scan);
    for (uint32_t i = tid; i < cw; i += 256) data[i] = 0ull;
    __syncthreads();
    if (valid) {
        auto sink = [&](long long w, unsigned long long bits) { atomicOr(&data[w], bits); };
        blk.emit((long long)excl_bits, sink, m_lo, m_hi);
    }
}

struct DecArgs {
    DecJob job[kEncJobs];
    const uint8_t *in;
    uint64_t cap;        // bytes readable from `in`
    int dims[3];
    int pitch;           // elements between rows of the field
    int nb[3];
    long long nblocks, nchunks, prefix_bytes;
};

// One lane per block; bound by the instructions of the waves that hold coded blocks.  A 400^3
// field of 11.4 MB: 78 us (2000 vector instructions a wave on average, of which the two plane
// transposes 512, the inverse transform 576; 102 us and 2870 before the transposes were bit
// inserts, the lifting butterflies, the group tests read from one window and the bits from
// LDS words by funnel shifts).  Four waves a SIMD: at its natural 134 registers (three) 85 us.
template <int ND, bool VEC>
__global__ __launch_bounds__(256, 4) void decode_kernel(DecArgs A)
{
    constexpr int S = ND == 3 ? 64 : 16;
    __shared__ unsigned s_scan[4];
    __shared__ unsigned long long s_words[kDecLdsWords + kDecPad];
    const int tid = threadIdx.x;
    const long long c = blockIdx.x;
    const long long b = c * kBlocksPerChunk + tid;
    const bool valid = b < A.nblocks;
    const float *sub = A.job[blockIdx.y].sub;
    float *field = A.job[blockIdx.y].field;
    const uint64_t boff = A.job[blockIdx.y].base ? *A.job[blockIdx.y].base : 0ull;
    if (boff + (uint64_t)A.prefix_bytes > A.cap) {
        // stream outside the readable range (an overflowed store): decode zeros
        if (valid) {
            const int bx = (int)(b % A.nb[0]);
            const int by = (int)((b / A.nb[0]) % A.nb[1]);
            const int bz = (int)(b / ((long long)A.nb[0] * A.nb[1]));
            const int nzz = ND == 3 ? A.dims[2] : 1;
            for (int k = 0; k < (ND == 3 ? 4 : 1); ++k)
                for (int j = 0; j < 4; ++j)
                    for (int i = 0; i < 4; ++i) {
                        const int x = 4 * bx + i, y = 4 * by + j, z = 4 * bz + k;
                        if (x < A.dims[0] && y < A.dims[1] && z < nzz) {
                            const long long p = ((long long)z * A.dims[1] + y) * A.pitch + x;
                            field[p] = sub ? sub[p] : 0.0f;
                        }
                    }
        }
        return;
    }
    const uint8_t *hdr = A.in + boff;
    const uint64_t *chunk_off = (const uint64_t *)(hdr + kHdr);
    const uint16_t *lens = (const uint16_t *)(hdr + kHdr + 8 * A.nchunks);
    const unsigned long long *data = (const unsigned long long *)(hdr + A.prefix_bytes);
    long long nwords = (long long)*(const unsigned long long *)(hdr + 48);
    const long long maxw = (long long)((A.cap - boff - (uint64_t)A.prefix_bytes) / 8);
    nwords = nwords < maxw ? nwords : maxw;
    const double tol = *(const double *)(hdr + 24);
    int te;
    frexp(tol, &te);
    const int minexp = te - 1;

    const unsigned nbits = valid ? lens[b] : 0u;
    unsigned total_bits;
    const unsigned incl = wg_scan256(nbits, s_scan, total_bits);
    // The chunk's words are contiguous: stage them in LDS with one coalesced pass, so
    // that each lane's sequential bit reads are LDS reads instead of a chain of
    // dependent global loads.  Chunks too long for the buffer read global memory.
    // a chunk offset outside the data words (only a corrupt stream has one) is clamped,
    // so that every word read below stays inside the readable range
    long long cbase = (long long)chunk_off[c];
    cbase = cbase < 0 ? 0 : (cbase > nwords ? nwords : cbase);
    const long long cw = ((long long)total_bits + 63) / 64 + 1;   // + a word of look-ahead
    const bool staged = cw <= kDecLdsWords;
    if (staged) {
        for (long long i = tid; i < cw + kDecPad; i += 256) {
            const long long j = cbase + i;
            s_words[i] = (i < cw && j >= 0 && j < nwords) ? data[j] : 0ull;
        }
    }
    __syncthreads();
    if (!valid) return;
    const long long rel = (long long)(incl - nbits);
    float out[S];
    if (staged) {
        LdsReader rd{reinterpret_cast<const uint32_t *>(s_words), 2 * (int)cw, (int)rel};
        decode_block<ND>(rd, minexp, out);
    } else {
        GlobalReader rd{data, nwords, 0, 0ull, 0ull, 0};
        rd.init(cbase * 64 + rel);
        decode_block<ND>(rd, minexp, out);
    }
    store_block<ND, VEC>(field, sub, A.dims, A.pitch, A.nb, b, out);
}

}  // namespace

CodecDims codec_dims(int ndim, const int *dims, int pitch)
{
    CodecDims cd{};
    cd.ndim = ndim;
    cd.pitch = pitch > 0 ? pitch : dims[0];
    for (int a = 0; a < 3; ++a) {
        cd.dims[a] = (a < ndim) ? dims[a] : 1;
        cd.nb[a] = (a < ndim) ? (dims[a] + 3) / 4 : 1;
    }
    cd.nblocks = (long long)cd.nb[0] * cd.nb[1] * cd.nb[2];
    cd.nchunks = (cd.nblocks + kBlocksPerChunk - 1) / kBlocksPerChunk;
    cd.prefix_bytes = kHdr + 8 * cd.nchunks + ((2 * cd.nblocks + 7) / 8) * 8;
    return cd;
}

size_t codec_max_bytes(const CodecDims &cd)
{
    // worst case per block: 1 + 8 + 32 planes of (S verbatim + S group + 1) bits
    const long long S = cd.ndim == 3 ? 64 : 16;
    const long long per_block_bits = 9 + 32 * (2 * S + 1);
    const long long words = cd.nchunks + (cd.nblocks * per_block_bits + 63) / 64;
    return (size_t)(cd.prefix_bytes + 8 * words);
}

namespace {

constexpr long long kScanChunks = 1024;   // fields of up to so many chunks have no scan pass

size_t pad256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

size_t encode_work_bytes(const CodecDims &cd, bool staged, int jobs)
{
    const size_t n = (size_t)cd.nchunks * jobs;
    size_t b = pad256(n * 4) + pad256(n * 8);
    if (staged) b += n * (size_t)kLdsWords * 8 + pad256((size_t)cd.nblocks * jobs * 2);
    return b;
}

hipError_t launch_encode(const CodecDims &cd, const EncJob *jobs, int njobs, double tol, uint8_t *out, uint64_t cap,
                         uint8_t *work, bool staged, unsigned *err, unsigned long long *stats, hipStream_t s)
{
    if (njobs < 1 || njobs > kEncJobs || (!staged && njobs != 1)) return hipErrorInvalidValue;
    EncArgs A{};
    for (int e = 0; e < njobs; ++e) {
        A.job[e] = jobs[e];
        A.chain[e] = e > 0 && jobs[e].base == jobs[e - 1].next;
    }
    for (int a = 0; a < 3; ++a) {
        A.dims[a] = cd.dims[a];
        A.nb[a] = cd.nb[a];
    }
    A.pitch = cd.pitch;
    A.nblocks = cd.nblocks;
    A.nchunks = cd.nchunks;
    A.prefix_bytes = cd.prefix_bytes;
    A.ndim = cd.ndim;
    int te;
    frexp(tol, &te);
    A.minexp = te - 1;
    A.tol = tol;
    A.out = out;
    A.cap = cap;
    const size_t n = (size_t)cd.nchunks * njobs;
    A.words = reinterpret_cast<uint32_t *>(work);
    A.offs = reinterpret_cast<uint64_t *>(work + pad256(n * 4));
    if (staged) {
        uint8_t *slots = work + pad256(n * 4) + pad256(n * 8);
        A.staging = reinterpret_cast<unsigned long long *>(slots);
        A.lens = reinterpret_cast<uint16_t *>(slots + n * (size_t)kLdsWords * 8);
        A.slot_words = kLdsWords;
    }
    A.err = err;
    A.stats = stats;
    const bool vec = cd.dims[0] % 4 == 0 && cd.pitch % 4 == 0;
    const dim3 grid((unsigned)cd.nchunks, (unsigned)njobs);
    if (cd.ndim == 3) {
        if (vec) hipLaunchKernelGGL((encode_count_kernel<3, true>), grid, dim3(256), 0, s, A);
        else hipLaunchKernelGGL((encode_count_kernel<3, false>), grid, dim3(256), 0, s, A);
    } else {
        if (vec) hipLaunchKernelGGL((encode_count_kernel<2, true>), grid, dim3(256), 0, s, A);
        else hipLaunchKernelGGL((encode_count_kernel<2, false>), grid, dim3(256), 0, s, A);
    }
    const bool scan = cd.nchunks <= kScanChunks;
    if (!scan) hipLaunchKernelGGL(encode_scan_kernel, dim3((unsigned)njobs), dim3(256), 0, s, A);
    auto place = [&](auto with, auto without) {
        if (scan) hipLaunchKernelGGL(with, grid, dim3(256), 0, s, A);
        else hipLaunchKernelGGL(without, grid, dim3(256), 0, s, A);
    };
    if (cd.ndim == 3) {
        if (vec) place(encode_place_kernel<3, true, true>, encode_place_kernel<3, true, false>);
        else place(encode_place_kernel<3, false, true>, encode_place_kernel<3, false, false>);
    } else {
        if (vec) place(encode_place_kernel<2, true, true>, encode_place_kernel<2, true, false>);
        else place(encode_place_kernel<2, false, true>, encode_place_kernel<2, false, false>);
    }
    return hipGetLastError();
}

hipError_t launch_decode(const CodecDims &cd, const uint8_t *in, const DecJob *jobs, int njobs, uint64_t cap,
                         hipStream_t s)
{
    if (njobs < 1 || njobs > kEncJobs) return hipErrorInvalidValue;
    DecArgs A{};
    std::copy(jobs, jobs + njobs, A.job);
    A.in = in;
    A.cap = cap;
    for (int a = 0; a < 3; ++a) {
        A.dims[a] = cd.dims[a];
        A.nb[a] = cd.nb[a];
    }
    A.pitch = cd.pitch;
    A.nblocks = cd.nblocks;
    A.nchunks = cd.nchunks;
    A.prefix_bytes = cd.prefix_bytes;
    const bool vec = cd.dims[0] % 4 == 0 && cd.pitch % 4 == 0;
    const dim3 grid((unsigned)cd.nchunks, (unsigned)njobs);
    if (cd.ndim == 3) {
        if (vec) hipLaunchKernelGGL((decode_kernel<3, true>), grid, dim3(256), 0, s, A);
        else hipLaunchKernelGGL((decode_kernel<3, false>), grid, dim3(256), 0, s, A);
    } else {
        if (vec) hipLaunchKernelGGL((decode_kernel<2, true>), grid, dim3(256), 0, s, A);
        else hipLaunchKernelGGL((decode_kernel<2, false>), grid, dim3(256), 0, s, A);
    }
    return hipGetLastError();
}

}  // namespace wv
