// Device building blocks of the ZFP-kind fixed-accuracy codec, shared by the codec's
// own kernels and the batched solver (one definition, so every stream and every decoded
// value is the same whichever kernel produced it).  The method and the stream layout
// are described in wv_codec.hip and wv.h.
#pragma once

#include "wv_internal.h"

namespace wv {

namespace {

constexpr uint32_t kMagic = 0x4B50465Au;
constexpr uint32_t kVersion = 1u;
constexpr int kHdr = 64;

struct Perm { int v[64]; };

// Coefficient order: ascending total degree i+j+k, then i^2+j^2+k^2, then the
// slowest index first (k, j, i).  Built at compile time by insertion sort.
constexpr Perm make_perm(int nd)
{
    Perm p{};
    const int S = nd == 3 ? 64 : 16;
    int key[64][5]{};
    for (int v = 0; v < S; ++v) {
        const int i = v & 3, j = (v >> 2) & 3, k = (v >> 4) & 3;
        key[v][0] = i + j + k;
        key[v][1] = i * i + j * j + k * k;
        key[v][2] = k;
        key[v][3] = j;
        key[v][4] = i;
        p.v[v] = v;
    }
    for (int a = 1; a < S; ++a) {
        const int cur = p.v[a];
        int b = a - 1;
        while (b >= 0) {
            const int o = p.v[b];
            bool less = false;
            for (int t = 0; t < 5; ++t)
                if (key[cur][t] != key[o][t]) {
                    less = key[cur][t] < key[o][t];
                    break;
                }
            if (!less) break;
            p.v[b + 1] = o;
            --b;
        }
        p.v[b + 1] = cur;
    }
    return p;
}

constexpr Perm kPerm3 = make_perm(3);
constexpr Perm kPerm2 = make_perm(2);

// Forward lifting of four integers (stride s inside the block array):
// the exact-arithmetic map is (1/16)[[4,4,4,4],[5,1,-1,-5],[-4,4,4,-4],[-2,6,-6,2]].
__device__ __forceinline__ void fwd_lift(int32_t *p, const int S0, const int S)
{
    int32_t x = p[S0], y = p[S0 + S], z = p[S0 + 2 * S], w = p[S0 + 3 * S];
    x += w; x >>= 1; w -= x;
    z += y; z >>= 1; y -= z;
    x += z; x >>= 1; z -= x;
    w += y; w >>= 1; y -= w;
    w += y >> 1; y -= w >> 1;
    p[S0] = x; p[S0 + S] = y; p[S0 + 2 * S] = z; p[S0 + 3 * S] = w;
}

// Inverse: each real-valued forward step undone in reverse order (wrap-around arithmetic
// keeps any stream well defined).  Undoing x = (x + w) / 2, w -= x is w += x, x = 2x - w,
// which is the pair (w + x, x - w).
__device__ __forceinline__ void inv_lift(int32_t *p, const int S0, const int S)
{
    const uint32_t x = (uint32_t)p[S0], z = (uint32_t)p[S0 + 2 * S];
    uint32_t y = (uint32_t)p[S0 + S], w = (uint32_t)p[S0 + 3 * S];
    y += (uint32_t)((int32_t)w >> 1); w -= (uint32_t)((int32_t)y >> 1);
    const uint32_t y1 = y + w, w1 = w - y, z1 = z + x, x1 = x - z;
    p[S0] = (int32_t)(x1 - w1);
    p[S0 + S] = (int32_t)(y1 + z1);
    p[S0 + 2 * S] = (int32_t)(z1 - y1);
    p[S0 + 3 * S] = (int32_t)(w1 + x1);
}

template <int ND>
__device__ __forceinline__ void fwd_transform(int32_t *q)
{
    if constexpr (ND == 3) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            fwd_lift(q, 16 * k + 0, 1); fwd_lift(q, 16 * k + 4, 1);
            fwd_lift(q, 16 * k + 8, 1); fwd_lift(q, 16 * k + 12, 1);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            fwd_lift(q, 16 * k + 0, 4); fwd_lift(q, 16 * k + 1, 4);
            fwd_lift(q, 16 * k + 2, 4); fwd_lift(q, 16 * k + 3, 4);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            fwd_lift(q, 4 * j + 0, 16); fwd_lift(q, 4 * j + 1, 16);
            fwd_lift(q, 4 * j + 2, 16); fwd_lift(q, 4 * j + 3, 16);
        }
    } else {
        fwd_lift(q, 0, 1); fwd_lift(q, 4, 1); fwd_lift(q, 8, 1); fwd_lift(q, 12, 1);
        fwd_lift(q, 0, 4); fwd_lift(q, 1, 4); fwd_lift(q, 2, 4); fwd_lift(q, 3, 4);
    }
}

template <int ND>
__device__ __forceinline__ void inv_transform(int32_t *q)
{
    if constexpr (ND == 3) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            inv_lift(q, 4 * j + 0, 16); inv_lift(q, 4 * j + 1, 16);
            inv_lift(q, 4 * j + 2, 16); inv_lift(q, 4 * j + 3, 16);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            inv_lift(q, 16 * k + 0, 4); inv_lift(q, 16 * k + 1, 4);
            inv_lift(q, 16 * k + 2, 4); inv_lift(q, 16 * k + 3, 4);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            inv_lift(q, 16 * k + 0, 1); inv_lift(q, 16 * k + 4, 1);
            inv_lift(q, 16 * k + 8, 1); inv_lift(q, 16 * k + 12, 1);
        }
    } else {
        inv_lift(q, 0, 4); inv_lift(q, 1, 4); inv_lift(q, 2, 4); inv_lift(q, 3, 4);
        inv_lift(q, 0, 1); inv_lift(q, 4, 1); inv_lift(q, 8, 1); inv_lift(q, 12, 1);
    }
}

__device__ __forceinline__ uint64_t low_mask(int n) { return n >= 64 ? ~0ull : ((1ull << n) - 1ull); }

// In-place transpose of a 32 x 32 bit matrix: bit k of a[s] moves to bit s of a[k]
// (five stages of masked block swaps; an involution).  The swaps of half-words and bytes
// are byte permutes, the others a shift and a bit-field insert per word: 256 operations
// (480 as three exclusive ors each).
constexpr uint32_t kSwapMask[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};

__device__ __forceinline__ void transpose32(uint32_t *a)
{
#pragma unroll
    for (int st = 0; st < 5; ++st) {
        const int j = 16 >> st;
        const uint32_t m = kSwapMask[st];
#pragma unroll
        for (int s = 0; s < 32; ++s) {
            if (!(s & j)) {
                const uint32_t x = a[s], y = a[s + j];
                if (st == 0) {          // bytes: x = y1 y0 x1 x0, y = y3 y2 x3 x2
                    a[s] = __builtin_amdgcn_perm(y, x, 0x05040100u);
                    a[s + j] = __builtin_amdgcn_perm(y, x, 0x07060302u);
                } else if (st == 1) {
                    a[s] = __builtin_amdgcn_perm(y, x, 0x06020400u);
                    a[s + j] = __builtin_amdgcn_perm(y, x, 0x07030501u);
                } else {
                    a[s] = (x & ~(m << j)) | ((y << j) & (m << j));
                    a[s + j] = (y & ~m) | ((x >> j) & m);
                }
            }
        }
    }
}

// Bit emitter: bits accumulate in `acc` for the word that holds `pos`; each
// completed word, and the last partial one, goes to sink(word_index, bits), which
// ORs it into a zeroed word range (neighbouring lanes share edge words).
struct Emitter {
    long long pos;
    unsigned long long acc;
    template <typename Sink>
    __device__ __forceinline__ void put(unsigned long long v, int nb, Sink &sink)   // nb <= 64
    {
        const int off = (int)(pos & 63);
        acc |= v << off;
        if (off + nb >= 64) {
            sink(pos >> 6, acc);
            acc = off ? (v >> (64 - off)) : 0ull;
        }
        pos += nb;
    }
    template <typename Sink>
    __device__ __forceinline__ void flush(Sink &sink)
    {
        if (pos & 63) sink(pos >> 6, acc);
    }
};

// Bit readers: peek() gives the next 64 bits, skip() passes up to 64 of them.
// From LDS words, the stream's and two of zeros behind it (which a corrupt stream may read
// on and on): three word reads and two funnel shifts a peek.
struct LdsReader {
    const uint32_t *w;
    int last;                // the zero words' place
    int pos;
    __device__ __forceinline__ unsigned long long peek() const
    {
        const int i = min(pos >> 5, last);
        const uint32_t a = w[i], b = w[i + 1], c = w[i + 2];
        return (unsigned long long)__builtin_amdgcn_alignbit(c, b, (uint32_t)pos) << 32 |
               __builtin_amdgcn_alignbit(b, a, (uint32_t)pos);
    }
    __device__ __forceinline__ void skip(int nb) { pos += nb; }
};

// From global memory (a chunk too long for LDS); words outside [0, nw) read as zero.
struct GlobalReader {
    const unsigned long long *data;
    long long nw;
    long long widx;
    unsigned long long w0, w1;
    int off;
    __device__ __forceinline__ unsigned long long load(long long i) const
    {
        return (i >= 0 && i < nw) ? data[i] : 0ull;
    }
    __device__ __forceinline__ void init(long long pos)
    {
        widx = pos >> 6;
        off = (int)(pos & 63);
        w0 = load(widx);
        w1 = load(widx + 1);
    }
    __device__ __forceinline__ unsigned long long peek() const { return off ? (w0 >> off) | (w1 << (64 - off)) : w0; }
    __device__ __forceinline__ void skip(int nb)
    {
        off += nb;
        if (off >= 64) {
            off -= 64;
            ++widx;
            w0 = w1;
            w1 = load(widx + 1);
        }
    }
};

// Inclusive scan of v over 256 lanes (a workgroup, or one of its groups of 256, each with an
// s_w of its own): shuffles inside each wave, then one exchange of the four wave totals
// through s_w[0..3].  Returns the lane's inclusive sum and sets total to the group's sum.
// Every lane of the workgroup calls it; it holds one barrier, and s_w may be written again
// only after another barrier of the caller.
template <typename T>
__device__ __forceinline__ T wg_scan256(T v, T *s_w, T &total)
{
    const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    const T w0 = s_w[0], w1 = s_w[1], w2 = s_w[2], w3 = s_w[3];
    total = w0 + w1 + w2 + w3;
    return x + (wave > 0 ? w0 : T(0)) + (wave > 1 ? w1 : T(0)) + (wave > 2 ? w2 : T(0));
}

// Block values, axis 0 fastest; partial blocks repeat the last valid index.  With
// VEC (dims[0] % 4 == 0) every block is complete along x and each row is one
// float4 load with no branch, so all 16 row loads of a lane are in flight together.
template <int ND, bool VEC>
__device__ __forceinline__ void load_raw(const float *f, const int *dims, int pitch, int bx, int by, int bz,
                                         float *v)
{
    constexpr int KZ = ND == 3 ? 4 : 1;
    const int ny = dims[1];
    const int nzz = ND == 3 ? dims[2] : 1;
#pragma unroll
    for (int k = 0; k < KZ; ++k) {
        const int z = min(4 * bz + k, nzz - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int y = min(4 * by + j, ny - 1);
            const float *row = f + ((long long)z * ny + y) * pitch;
            if constexpr (VEC) {
                const float4 t = *reinterpret_cast<const float4 *>(row + 4 * bx);
                v[16 * k + 4 * j + 0] = t.x;
                v[16 * k + 4 * j + 1] = t.y;
                v[16 * k + 4 * j + 2] = t.z;
                v[16 * k + 4 * j + 3] = t.w;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[16 * k + 4 * j + i] = row[min(4 * bx + i, dims[0] - 1)];
            }
        }
    }
}

// The block of f, or of f - sub (one binary32 subtraction per value) when sub is set.
template <int ND, bool VEC>
__device__ __forceinline__ void load_block(const float *f, const float *sub, const int *dims, int pitch, int bx,
                                           int by, int bz, float *v)
{
    constexpr int S = ND == 3 ? 64 : 16;
    load_raw<ND, VEC>(f, dims, pitch, bx, by, bz, v);
    if (sub) {
        float t[S];
        load_raw<ND, VEC>(sub, dims, pitch, bx, by, bz, t);
#pragma unroll
        for (int i = 0; i < S; ++i) v[i] -= t[i];
    }
}


// One block of the fixed-accuracy code, one lane per block: exponent, block-floating-
// point integers, forward transform, sequency order, negabinary, and the bit planes
// m_lo[k] / m_hi[k] (bit k of coefficients 0..31 / 32..63).  The planes are the
// caller's own local arrays (a plain array stays in registers under the planes loops'
// wave-uniform indexing; inside a struct it would be placed in scratch).  prepare() is
// called by all lanes of a wave together (waves whose blocks are all uncoded skip the
// transform and the plane transposes; the planes loops run down to the wave's lowest
// kmin).
template <int ND>
struct BlockEnc {
    static constexpr int S = ND == 3 ? 64 : 16;
    bool valid = false, finite = true, coded = false;
    int emax = -126, kmin = 32, kmin_w = 32;

    __device__ __forceinline__ void prepare(const float *v, bool valid_, int minexp, uint32_t (&m_lo)[32],
                                            uint32_t (&m_hi)[32])
    {
        valid = valid_;
        // magnitudes order as their bits do: the largest gives the exponent, and whether any
        // value is not finite or not zero
        uint32_t most = 0u;
#pragma unroll
        for (int i = 0; i < S; ++i) most = max(most, __float_as_uint(v[i]) & 0x7FFFFFFFu);
        finite = most < 0x7F800000u;
        const bool nonzero = most != 0u;
        emax = most < 0x00800000u ? -126 : (int)(most >> 23) - 126;
        int prec = emax - minexp + 2 * (ND + 1);
        prec = prec > 32 ? 32 : prec;
        coded = valid && finite && nonzero && prec > 0;
        kmin = 32 - prec;
#pragma unroll
        for (int k = 0; k < 32; ++k) m_lo[k] = m_hi[k] = 0u;
        if (__ballot(coded) != 0ull) {
            // exact scaling, truncation; an uncoded block's integers are not used, but a value
            // that is not finite has none
            int32_t q[S];
            const int sh = 30 - emax;
            if (__any(!finite)) {
#pragma unroll
                for (int i = 0; i < S; ++i) q[i] = coded ? (int32_t)ldexpf(v[i], sh) : 0;
            } else {
#pragma unroll
                for (int i = 0; i < S; ++i) q[i] = (int32_t)ldexpf(v[i], sh);
            }
            fwd_transform<ND>(q);
#pragma unroll
            for (int s = 0; s < 32; ++s) {
                const int src = ND == 3 ? kPerm3.v[s] : kPerm2.v[s & 15];
                m_lo[s] = (s < S) ? (((uint32_t)q[src] + 0xAAAAAAAAu) ^ 0xAAAAAAAAu) : 0u;
                if constexpr (ND == 3) m_hi[s] = (((uint32_t)q[kPerm3.v[32 + s]] + 0xAAAAAAAAu) ^ 0xAAAAAAAAu);
                else m_hi[s] = 0u;
            }
            if constexpr (ND == 3) {
                // Two transposes of half-words: the upper halves of coefficients s and
                // 32+s packed into one word (low and high 16 bits) transpose into planes
                // 16..31, the lower halves into planes 0..15.  A wave none of whose blocks
                // codes a plane below 16 (kmin >= 16) needs only the first.
#pragma unroll
                for (int s = 0; s < 32; ++s) {
                    const uint32_t a = m_lo[s], b = m_hi[s];
                    m_lo[s] = __builtin_amdgcn_perm(b, a, 0x07060302u);   // upper halves
                    m_hi[s] = __builtin_amdgcn_perm(b, a, 0x05040100u);   // lower halves
                }
                transpose32(m_lo);   // word k < 16: plane k+16 of 0..31; k >= 16: plane k of 32..63
                if (__ballot(coded && kmin < 16) != 0ull) transpose32(m_hi);   // planes 0..15 likewise
                else {
#pragma unroll
                    for (int k = 0; k < 32; ++k) m_hi[k] = 0u;
                }
                uint32_t U[32], L[32];
#pragma unroll
                for (int k = 0; k < 32; ++k) {
                    U[k] = m_lo[k];
                    L[k] = m_hi[k];
                }
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    m_lo[k] = L[k];
                    m_lo[k + 16] = U[k];
                    m_hi[k] = L[k + 16];
                    m_hi[k + 16] = U[k + 16];
                }
            } else {
                transpose32(m_lo);
            }
        }
        // Planes run from 31 down to the lowest kmin of the wave in a plain (rolled)
        // loop: the plane index is wave-uniform, so m_lo[k] / m_hi[k] stay in registers
        // (indexed moves), and each lane skips the planes below its own kmin.
        kmin_w = coded ? kmin : 32;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) kmin_w = min(kmin_w, __shfl_xor(kmin_w, o));
        kmin_w = __builtin_amdgcn_readfirstlane(kmin_w);
    }

    // closed-form bit count of the block (0 for a lane without a block)
    __device__ __forceinline__ unsigned count(const uint32_t (&m_lo)[32], const uint32_t (&m_hi)[32]) const
    {
        unsigned nbits = valid ? 1u : 0u;
        if (coded) nbits += 8;
        int n = 0;
#pragma unroll 1
        for (int k = 31; k >= kmin_w; --k) {
            if (coded && k >= kmin) {
                nbits += n;
                if (n < S) {
                    const unsigned long long r = ((unsigned long long)m_hi[k] << 32 | m_lo[k]) >> n;
                    if (r == 0ull) nbits += 1;
                    else {
                        const int pt = 63 - __clzll((long long)r);
                        nbits += pt + 1 + __popcll(r);
                        n += pt + 1;
                        if (n < S) nbits += 1;
                    }
                }
            }
        }
        return nbits;
    }

    // the block's bits at bit position pos of the sink's word space
    template <typename Sink>
    __device__ __forceinline__ void emit(long long pos, Sink &sink, const uint32_t (&m_lo)[32],
                                         const uint32_t (&m_hi)[32]) const
    {
        Emitter em{pos, 0ull};
        em.put(coded ? 1ull : 0ull, 1, sink);
        if (coded) em.put((unsigned long long)(emax + 127), 8, sink);
        int n = 0;
#pragma unroll 1
        for (int k = 31; k >= kmin_w; --k) {
            if (coded && k >= kmin) {
                const unsigned long long mk = (unsigned long long)m_hi[k] << 32 | m_lo[k];
                // the plane's verbatim bits, then its groups (1, the zeros before the next
                // one bit, that bit) and the 0 that ends them, collected in up to 64 bits
                unsigned long long out = mk & low_mask(n);
                int used = n;
                if (n < S) {
                    unsigned long long r = mk >> n;
                    while (r != 0ull) {
                        const int z = __ffsll((long long)r) - 1;
                        if (used + z + 2 > 64) {
                            em.put(out, used, sink);
                            out = 0ull;
                            used = 0;
                        }
                        if (z == 63) {          // 65 bits: the group test by itself (S = 64, n = 0)
                            em.put(1ull, 1, sink);
                            out = 1ull << 63;
                            used = 64;
                        } else {
                            out |= (1ull | (2ull << z)) << used;
                            used += z + 2;
                        }
                        n += z + 1;
                        r = z == 63 ? 0ull : r >> (z + 1);
                    }
                    if (n < S) {
                        if (used == 64) {
                            em.put(out, 64, sink);
                            out = 0ull;
                            used = 0;
                        }
                        ++used;
                    }
                }
                em.put(out, used, sink);
            }
        }
        em.flush(sink);
    }
};

// Decode one block from rd (positioned at its first bit) into out[S] (C order of the
// block, axis 0 fastest).
template <int ND, typename Reader>
__device__ __forceinline__ void decode_block(Reader &rd, int minexp, float *out)
{
    constexpr int S = ND == 3 ? 64 : 16;
    const bool coded = rd.peek() & 1ull;
    rd.skip(1);
    if (!coded) {
#pragma unroll
        for (int i = 0; i < S; ++i) out[i] = 0.0f;
        return;
    }
    const int emax = (int)(rd.peek() & 0xFFull) - 127;
    rd.skip(8);
    int prec = emax - minexp + 2 * (ND + 1);
    prec = prec > 32 ? 32 : prec;
    const int kmin = 32 - prec;
    // planes 16..31 and 0..15 in half-words: word k < 16 of hi (lo) is plane 16 + k (k) of
    // coefficients 0..31, word 16 + k that of 32..63; a wave none of whose blocks codes a
    // plane below 16 has no lo
    uint32_t hi[32], lo[32];
    const bool low = __any(kmin < 16);
    int n = 0;
    auto plane = [&](int k) -> unsigned long long {
        unsigned long long mk = 0ull;
        if (k >= kmin) {
            if (n > 0) {
                mk = rd.peek() & low_mask(n);
                rd.skip(n);
            }
            if (n < S) {
                // group tests out of one 64-bit window, read again where a run of zeros (or
                // the groups) reach its end
                unsigned long long w = rd.peek();
                int used = 0;
                for (;;) {
                    const bool g = w & 1ull;
                    ++used;
                    if (!g) break;
                    w >>= 1;
                    const int rem = S - n;
                    if (ND == 3 && w == 0ull && used + rem > 64) {
                        rd.skip(used);
                        used = 0;
                        w = rd.peek();
                    }
                    const unsigned z = (unsigned)__ffsll((long long)w) - 1u;   // no bit: larger than any rem
                    if (z >= (unsigned)rem) {
                        used += rem;
                        n = S;
                        break;
                    }
                    mk |= 1ull << (n + z);
                    n += z + 1;
                    used += z + 1;
                    if (n >= S) break;
                    w >>= z + 1;            // z < 63: n would be S
                    if (ND == 3 && used >= 64) {
                        rd.skip(used);
                        used = 0;
                        w = rd.peek();
                    }
                }
                rd.skip(used);
            }
        }
        return mk;
    };
#pragma unroll
    for (int k = 31; k >= 16; --k) {
        const unsigned long long mk = plane(k);
        hi[k - 16] = (uint32_t)mk;
        hi[k] = (uint32_t)(mk >> 32);
    }
    transpose32(hi);
#pragma unroll
    for (int s = 0; s < 32; ++s) lo[s] = 0u;
    if (low) {
#pragma unroll
        for (int k = 15; k >= 0; --k) {
            const unsigned long long mk = plane(k);
            lo[k] = (uint32_t)mk;
            lo[k + 16] = (uint32_t)(mk >> 32);
        }
        transpose32(lo);
    }
    int32_t q[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const uint32_t u = s < 32 ? __builtin_amdgcn_perm(hi[s & 31], lo[s & 31], 0x05040100u)
                                  : __builtin_amdgcn_perm(hi[s & 31], lo[s & 31], 0x07060302u);
        const int dst = ND == 3 ? kPerm3.v[s] : kPerm2.v[s];
        q[dst] = (int32_t)((u ^ 0xAAAAAAAAu) - 0xAAAAAAAAu);
    }
    inv_transform<ND>(q);
    // one rounding: to binary32 by the conversion, unless a value could be subnormal
    if (__all(emax >= -96)) {
#pragma unroll
        for (int i = 0; i < S; ++i) out[i] = ldexpf((float)q[i], emax - 30);
    } else {
#pragma unroll
        for (int i = 0; i < S; ++i) out[i] = (float)ldexp((double)q[i], emax - 30);
    }
}

// Write decoded block b (values out, C order) into field, or sub - decoded when sub is
// set; only the grid's own points are written, streamed out past the caches with VEC.
template <int ND, bool VEC>
__device__ __forceinline__ void store_block(float *field, const float *sub, const int *dims, int pitch,
                                            const int *nb, long long b, const float *out)
{
    const int bx = (int)(b % nb[0]);
    const int by = (int)((b / nb[0]) % nb[1]);
    const int bz = (int)(b / ((long long)nb[0] * nb[1]));
    constexpr int KZ = ND == 3 ? 4 : 1;
    const int nzz = ND == 3 ? dims[2] : 1;
#pragma unroll
    for (int k = 0; k < KZ; ++k) {
        const int z = 4 * bz + k;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int y = 4 * by + j;
            if (y >= dims[1] || z >= nzz) continue;
            const long long r0 = ((long long)z * dims[1] + y) * pitch;
            float *row = field + r0;
            if (VEC) {
                float4 o = make_float4(out[16 * k + 4 * j + 0], out[16 * k + 4 * j + 1], out[16 * k + 4 * j + 2],
                                       out[16 * k + 4 * j + 3]);
                if (sub) {
                    const float4 t = *reinterpret_cast<const float4 *>(sub + r0 + 4 * bx);
                    o = make_float4(t.x - o.x, t.y - o.y, t.z - o.z, t.w - o.w);
                }
                // streamed out: the next kernel reads it once, so it need not stay in the
                // caches (and its write-back is paid here, not during that kernel)
                typedef float f4v __attribute__((ext_vector_type(4)));
                const f4v t = {o.x, o.y, o.z, o.w};
                __builtin_nontemporal_store(t, reinterpret_cast<f4v *>(row + 4 * bx));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * bx + i < dims[0]) {
                        const float o = out[16 * k + 4 * j + i];
                        row[4 * bx + i] = sub ? sub[r0 + 4 * bx + i] - o : o;
                    }
            }
        }
    }
}

constexpr int kLdsWords = 2048;      // chunk bitstreams up to 16 KB are assembled in LDS
constexpr int kDecLdsWords = 2048;   // and chunks up to 16 KB are staged in LDS for decoding
constexpr int kDecPad = 2;           // zero words behind them

}  // namespace

}  // namespace wv
