// HIP kernels for gfx950: Philox4x32-10, initial spins, checkerboard
// Metropolis half-sweeps, per-replica energy reduction and the replica
// exchange step of the Exchange Monte Carlo method (arXiv:1508.06268,
// Sec. 3.1-3.3, Eq. 1-3).
//
// Compiled with -ffp-contract=off: every FP64 expression that feeds an
// exchange decision is evaluated exactly as written.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <cmath>

#include "rfim_internal.h"

namespace rfim_dev {

namespace {

constexpr uint32_t kTagInit = 1u, kTagSweep = 2u, kTagExch = 3u;

// Pointers read from a descriptor table in memory are generic; typing them
// as global (address space 1) all the way to the access keeps loads and
// stores global_* rather than flat_* instructions.
#define GAS __attribute__((address_space(1)))

template <class T>
__device__ __forceinline__ GAS T *gptr(T *p) {
    return (GAS T *)p;
}

// Pointer to U in the address space (and constness) of pointer type P.
template <class P, class U> struct rebind_ptr;
template <class U> struct rebind_ptr<uint8_t *, U> { using type = U *; };
template <class U> struct rebind_ptr<const uint8_t *, U> { using type = const U *; };
template <class U> struct rebind_ptr<GAS uint8_t *, U> { using type = GAS U *; };
template <class U> struct rebind_ptr<GAS const uint8_t *, U> { using type = GAS const U *; };
template <class U> struct rebind_ptr<const float *, U> { using type = const U *; };
template <class U> struct rebind_ptr<GAS const float *, U> { using type = GAS const U *; };

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each two
// 32x32->64 products by fixed odd multipliers whose high halves are mixed
// with the other two words and the round key; the key follows a Weyl
// sequence.  Written from the published definition.
struct Words { uint32_t w0, w1, w2, w3; };

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;

// Philox4x32-10 with the first round's product M0 * c0 given: a caller
// whose counters step by a constant can form it with one multiply-add.
__device__ __forceinline__ Words philox10_p(uint64_t a0, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                            uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t a = round == 0 ? a0 : (uint64_t)kPhiloxM0 * c0;
        const uint64_t b = (uint64_t)0xCD9E8D57u * c2;
        uint32_t n0, n2;
        if (round < 2) {
            // the first rounds still hold wave-uniform words: leave them to
            // the scalar unit
            n0 = (uint32_t)(b >> 32) ^ (c1 ^ k0);
            n2 = (uint32_t)(a >> 32) ^ (c3 ^ k1);
        } else if (round == 2) {
            // with a wave-uniform c0 and c2 at round 0 (one site block per
            // lane), c3 is still uniform here: one scalar XOR, one VALU XOR
            // (a three-input VALU XOR can read only one scalar operand)
            n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(b >> 32), c1, k0, 0x96);
            n2 = (uint32_t)(a >> 32) ^ (c3 ^ k1);
        } else {
            // three-input XOR in one VALU instruction (truth table 0x96)
            n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(b >> 32), c1, k0, 0x96);
            n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), c3, k1, 0x96);
        }
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return Words{c0, c1, c2, c3};
}

__device__ __forceinline__ Words philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t k0, uint32_t k1) {
    return philox10_p((uint64_t)kPhiloxM0 * c0, c0, c1, c2, c3, k0, k1);
}

// M0 x + c in one v_mad_u64_u32 (c a wave-uniform 64-bit addend; M0 from
// a VGPR, since one instruction reads one scalar operand).  Written out
// because the compiler folds M0 x + M0 b back into M0 (x + b), which costs
// the addition of b on top of the product.  The carry-out register is not
// read.
__device__ __forceinline__ uint64_t mad_m0(uint32_t x, uint32_t m0, uint64_t c) {
    uint64_t r, carry;
    asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(r), "=s"(carry) : "v"(x), "v"(m0), "s"(c));
    return r;
}

__device__ __forceinline__ uint32_t word_at(const Words &w, int q) {
    return q == 0 ? w.w0 : q == 1 ? w.w1 : q == 2 ? w.w2 : w.w3;
}

// Continuous fields, one site, in FP32.  With up = number of +1 neighbours,
// J n + h h_i = 2J up + (h h_i - 6J) = y (the second term precomputed per
// site), and the flip costs dE = 2 s y.  With a = -2 beta log2(e),
// exp(-beta dE) = 2^(s a y): accept iff s a y >= 0 (dE <= 0) or
// u32 2^-32 < 2^(s a y).
__device__ __forceinline__ bool cont_accept(float up, float hfs, float twoJ, float a, bool up_spin,
                                            uint32_t u) {
    const float y = fmaf(twoJ, up, hfs);
    const float ta = a * y;
    const float t = up_spin ? ta : -ta;
    const float p = __builtin_amdgcn_exp2f(t);
    return t >= 0.0f || (float)u * 0x1p-32f < p;
}

// ---------------------------------------------------------------------
// Initial spins (method step 3): replica r, natural sites 4g..4g+3 take
// the four words of block (g, 0, r) of the INIT stream.
// ---------------------------------------------------------------------
__global__ __launch_bounds__(256) void init_kernel(Lattice lat, int r0) {
    const int G = lat.N >> 2;
    const int g = blockIdx.x * 256 + threadIdx.x;
    const int r = r0 + blockIdx.y;
    if (g >= G) return;
    const Words w = philox10((uint32_t)g, 0u, (uint32_t)r, (kTagInit << 28) | lat.rho, lat.key0,
                             lat.key1);
    uint8_t *base = lat.spins + (size_t)r * lat.N;
    const int L = lat.L;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = 4 * g + q;
        const int x = i % L, y = (i / L) % L, z = i / (L * L);
        const int c = (x + y + z) & 1;
        base[(size_t)c * lat.half + (i >> 1)] = word_at(w, q) >= 0x80000000u ? 1 : 0;
    }
}

// ---------------------------------------------------------------------
// Half-sweep, L = 2^l >= 8, on one chunk of NW x 4 consecutive sublattice
// sites of one row (NW Philox blocks): the spin bytes, the six neighbour
// words and the field bytes are NW-dword loads, and the neighbour counts of
// four sites are one packed byte-wise sum per dword (each byte <= 6, so no
// carries).
//
// Colour-c site of pair m in row (y, z) sits at x = 2m + p, p = (c+y+z)&1;
// its x-neighbours of the other colour are pair m and pair m-1+2p of the
// same row, so the row's other-colour bytes shifted by one (with one byte
// from the adjacent dword, wrapping in the row) supply the second x
// neighbour.
// ---------------------------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int NW> struct Vec;
template <> struct Vec<1> { using T = uint32_t; };
template <> struct Vec<2> { using T = u32x2; };
template <> struct Vec<4> { using T = u32x4; };

template <int NW, class P>
__device__ __forceinline__ void load_words(P base, uint32_t off, uint32_t (&w)[NW]) {
    if constexpr (NW == 8) {
        // two 16-byte loads
        uint32_t lo[4], hi[4];
        load_words<4>(base, off, lo);
        load_words<4>(base, off + 16u, hi);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w[q] = lo[q];
            w[q + 4] = hi[q];
        }
        return;
    } else {
    const typename Vec<NW>::T v = *(typename rebind_ptr<P, const typename Vec<NW>::T>::type)(base + off);
    if constexpr (NW == 1) {
        w[0] = v;
    } else if constexpr (NW == 2) {
        w[0] = v.x; w[1] = v.y;
    } else {
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    }
    }
}

template <int NW, class P>
__device__ __forceinline__ void store_words(P base, uint32_t off, const uint32_t (&w)[NW]) {
    if constexpr (NW == 8) {
        const uint32_t lo[4] = {w[0], w[1], w[2], w[3]}, hi[4] = {w[4], w[5], w[6], w[7]};
        store_words<4>(base, off, lo);
        store_words<4>(base, off + 16u, hi);
        return;
    } else {
    typename Vec<NW>::T v;
    if constexpr (NW == 1) {
        v = w[0];
    } else if constexpr (NW == 2) {
        v.x = w[0]; v.y = w[1];
    } else {
        v.x = w[0]; v.y = w[1]; v.z = w[2]; v.w = w[3];
    }
    *(typename rebind_ptr<P, typename Vec<NW>::T>::type)(base + off) = v;
    }
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The same in a workgroup whose last wave may be partly empty: what a shuffle
// gives for a lane that is not there counts as 0.
__device__ __forceinline__ double part_wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const double o = __shfl_xor(v, off, 64);
        v += (threadIdx.x ^ (uint32_t)off) < blockDim.x ? o : 0.0;
    }
    return v;
}

// Offsets (in sublattice bytes) of the other-colour words around a chunk.
struct Chunk {
    uint32_t p, jxw, jyp, jym, jzp, jzm;
};

template <int NW>
__device__ __forceinline__ Chunk chunk_geometry(uint32_t j0, uint32_t colour, uint32_t L, uint32_t l,
                                                uint32_t half) {
    Chunk c;
    const uint32_t hm = (L >> 1) - 1u;          // m bits of j
    const uint32_t ystep = L >> 1;
    const uint32_t ymask = (L - 1u) << (l - 1u);
    const uint32_t zstep = (L * L) >> 1;
    const uint32_t jmask = half - 1u;
    const uint32_t m0 = j0 & hm;
    const uint32_t row = j0 >> (l - 1u);
    c.p = (colour + row + (row >> l)) & 1u;     // (c + y + z) & 1
    // the one dword of the adjacent chunk that the x-shift needs
    c.jxw = (j0 - m0) | ((m0 + (c.p ? 4u * NW : 0u - 4u)) & hm);
    c.jyp = (j0 & ~ymask) | ((j0 + ystep) & ymask);
    c.jym = (j0 & ~ymask) | ((j0 - ystep) & ymask);
    c.jzp = (j0 + zstep) & jmask;
    c.jzm = (j0 - zstep) & jmask;
    return c;
}

// x / d for x < 2^31 by a multiplication (d >= 2): with 2^s < d <= 2^(s+1)
// and mul = floor(2^(32+s) / d) + 1, mul d exceeds 2^(32+s) by at most d, so
// the quotient is exact while x d < 2^(32+s), that is x < 2^31.
struct FastDiv {
    uint32_t mul, shift, d;
};

FastDiv fast_div(uint32_t d) {
    uint32_t s = 0;
    while ((2u << s) < d) ++s;
    return FastDiv{d < 2 ? 0u : (uint32_t)((1ull << (32 + s)) / d) + 1u, s, d};
}

__device__ __forceinline__ uint32_t div_by(uint32_t x, const FastDiv &f) {
    return f.d == 1u ? x : __umulhi(x, f.mul) >> f.shift;
}

// The geometry of a chunk when L is any multiple of 8 NW.
template <int NW>
__device__ __forceinline__ Chunk row_chunk(uint32_t j0, uint32_t colour, uint32_t L, const FastDiv &by_row,
                                           const FastDiv &by_l) {
    const uint32_t Lh = L >> 1, plane = L * Lh, half = L * plane;
    const uint32_t row = div_by(j0, by_row), m0 = j0 - row * Lh;
    const uint32_t z = div_by(row, by_l), y = row - z * L;
    Chunk c;
    c.p = (colour + y + z) & 1u;
    c.jxw = j0 - m0 + (c.p ? (m0 + 4u * NW == Lh ? 0u : m0 + 4u * NW) : (m0 == 0u ? Lh : m0) - 4u);
    c.jyp = y + 1u == L ? j0 + Lh - plane : j0 + Lh;
    c.jym = y == 0u ? j0 - Lh + plane : j0 - Lh;
    c.jzp = z + 1u == L ? j0 + plane - half : j0 + plane;
    c.jzm = z == 0u ? j0 - plane + half : j0 - plane;
    return c;
}

// Up counts of four consecutive pairs of any even L, which may lie in two
// rows, one per byte; W = the other colour's sites of the same pairs.
template <class P>
__device__ __forceinline__ uint32_t site_counts(P oth, uint32_t j0, uint32_t W, uint32_t colour, uint32_t L,
                                                const FastDiv &by_row, const FastDiv &by_l) {
    const uint32_t Lh = L >> 1, plane = L * Lh, half = L * plane;
    const uint32_t row = div_by(j0, by_row);
    uint32_t m = j0 - row * Lh, z = div_by(row, by_l), y = row - z * L, U = W;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t j = j0 + q;
        const uint32_t jx =
            ((colour + y + z) & 1u) ? (m + 1u == Lh ? j + 1u - Lh : j + 1u) : (m == 0u ? j + Lh - 1u : j - 1u);
        const uint32_t up = (uint32_t)oth[jx] + oth[y + 1u == L ? j + Lh - plane : j + Lh] +
                            oth[y == 0u ? j - Lh + plane : j - Lh] + oth[z + 1u == L ? j + plane - half : j + plane] +
                            oth[z == 0u ? j - plane + half : j - plane];
        U += up << (8u * q);
        if (++m == Lh) {
            m = 0;
            if (++y == L) {
                y = 0;
                ++z;
            }
        }
    }
    return U;
}

// The other-colour words around a chunk: the chunk's own pair words W, the
// one dword of the adjacent chunk the x-shift needs, and the y+-1, z+-1 rows.
template <int NW> struct Around {
    uint32_t W[NW], Wx, Wyp[NW], Wym[NW], Wzp[NW], Wzm[NW];
};

template <int NW, class P>
__device__ __forceinline__ void load_around(P oth, uint32_t j0, const Chunk &c, Around<NW> &a) {
    load_words<NW>(oth, j0, a.W);
    a.Wx = *(typename rebind_ptr<P, const uint32_t>::type)(oth + c.jxw);
    load_words<NW>(oth, c.jyp, a.Wyp);
    load_words<NW>(oth, c.jym, a.Wym);
    load_words<NW>(oth, c.jzp, a.Wzp);
    load_words<NW>(oth, c.jzm, a.Wzm);
}

// Up-neighbour counts (per byte) of the NW words of a chunk.
template <int NW>
__device__ __forceinline__ void neighbour_sums(const Chunk &c, const Around<NW> &a, uint32_t (&U)[NW]) {
    // p = 1: bytes of pairs m+1..m+4 (bytes 1-3 of W[w], byte 0 of the next
    // word); p = 0: bytes of pairs m-1..m+2 (byte 3 of the previous word,
    // bytes 0-2 of W[w]).  One byte permute of {other word, W[w]}.
    const uint32_t sel = c.p ? 0x04030201u : 0x02010007u;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint32_t nxt = (w + 1 < NW) ? a.W[w + 1 < NW ? w + 1 : 0] : a.Wx;
        const uint32_t prv = (w > 0) ? a.W[w > 0 ? w - 1 : 0] : a.Wx;
        const uint32_t Xs = __builtin_amdgcn_perm(c.p ? nxt : prv, a.W[w], sel);
        U[w] = a.W[w] + Xs + a.Wyp[w] + a.Wym[w] + a.Wzp[w] + a.Wzm[w];
    }
}

template <int NW, class P>
__device__ __forceinline__ void neighbour_counts(P oth, uint32_t j0, const Chunk &c, uint32_t (&W)[NW],
                                                 uint32_t (&U)[NW]) {
    Around<NW> a;
    load_around<NW>(oth, j0, c, a);
    neighbour_sums<NW>(c, a, U);
#pragma unroll
    for (int w = 0; w < NW; ++w) W[w] = a.W[w];
}

// Bit q set iff u_q <= t_q, for four sites.  The compares write four lane
// masks that an add-with-carry chain folds into one register (acc = 2 acc +
// mask), so each site costs two VALU instructions and no select.  gfx950
// wants two wait states between a VALU write of a lane mask and a VALU read
// of it: every mask is read three instructions after it is written, and the
// trailing nop covers reads after the block.
__device__ __forceinline__ uint32_t accept_bits(uint32_t u0, uint32_t u1, uint32_t u2, uint32_t u3,
                                                uint32_t t0, uint32_t t1, uint32_t t2, uint32_t t3) {
    uint32_t acc;
    uint64_t c3, c2, c1, c0, cx;
    asm("v_cmp_le_u32_e64 %1, %9, %13\n\t"
        "v_cmp_le_u32_e64 %2, %8, %12\n\t"
        "v_cmp_le_u32_e64 %3, %7, %11\n\t"
        "v_cmp_le_u32_e64 %4, %6, %10\n\t"
        "v_cndmask_b32_e64 %0, 0, 1, %1\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %4\n\t"
        "s_nop 1"
        : "=&v"(acc), "=&s"(c3), "=&s"(c2), "=&s"(c1), "=&s"(c0), "=&s"(cx)
        : "v"(u0), "v"(u1), "v"(u2), "v"(u3), "v"(t0), "v"(t1), "v"(t2), "v"(t3));
    return acc;
}

// The bit sweep's form: the four decisions of one Philox block shifted
// into four accumulators, f_q = 2 f_q + [u_q <= t_q].  Run over blocks 7
// down to 0, bit b of f_q ends as the flip of block b's site q, which is
// bit 8q + b of the word: byte q of the flips is f_q, with no per-block
// spreading.  Four compares and four add-with-carry per block; each mask
// is read four instructions after it is written (gfx950's VALU-mask
// hazard), and the trailing nop covers reads after the block.
__device__ __forceinline__ void accept_shift(uint32_t u0, uint32_t u1, uint32_t u2, uint32_t u3,
                                             uint32_t t0, uint32_t t1, uint32_t t2, uint32_t t3,
                                             uint32_t &f0, uint32_t &f1, uint32_t &f2, uint32_t &f3) {
    uint64_t c0, c1, c2, c3, cx;
    asm("v_cmp_le_u32_e64 %4, %9, %13\n\t"
        "v_cmp_le_u32_e64 %5, %10, %14\n\t"
        "v_cmp_le_u32_e64 %6, %11, %15\n\t"
        "v_cmp_le_u32_e64 %7, %12, %16\n\t"
        "v_addc_co_u32_e64 %0, %8, %0, %0, %4\n\t"
        "v_addc_co_u32_e64 %1, %8, %1, %1, %5\n\t"
        "v_addc_co_u32_e64 %2, %8, %2, %2, %6\n\t"
        "v_addc_co_u32_e64 %3, %8, %3, %3, %7\n\t"
        "s_nop 1"
        : "+v"(f0), "+v"(f1), "+v"(f2), "+v"(f3), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3), "=&s"(cx)
        : "v"(u0), "v"(u1), "v"(u2), "v"(u3), "v"(t0), "v"(t1), "v"(t2), "v"(t3));
}

// Metropolis decisions of one Philox block's four sites (+-1 fields): the
// table entry sits at LDS byte address ((up << 2) | (s << 1) | f) * 4 and a
// site flips iff u <= entry.  `never` marks classes whose bound is 0 at this
// temperature: there u = 0 would pass, so with NEV those sites are
// corrected when some u is 0 (about one block in 2^30).  Returns the flips
// as one bit per byte.
template <bool NEV>
__device__ __forceinline__ uint32_t bimodal_flips(const uint32_t *sthr, uint32_t U, uint32_t Wown,
                                                  uint32_t F4, const Words &rw, uint32_t never) {
    const uint32_t A = (U << 4) | (Wown << 3) | F4;
    const uint8_t *tb = (const uint8_t *)sthr;
    const uint32_t a0 = A & 0xFFu, a1 = (A >> 8) & 0xFFu, a2 = (A >> 16) & 0xFFu, a3 = A >> 24;
    const uint32_t th0 = *(const uint32_t *)(tb + a0), th1 = *(const uint32_t *)(tb + a1);
    const uint32_t th2 = *(const uint32_t *)(tb + a2), th3 = *(const uint32_t *)(tb + a3);
    const uint32_t acc = accept_bits(rw.w0, rw.w1, rw.w2, rw.w3, th0, th1, th2, th3);
    // bit q of a 4-bit value to bit 8q: the shifted copies 0, 7, 14, 21
    // do not overlap, so the product has no carries
    uint32_t fl = __umul24(acc, 0x204081u) & 0x01010101u;
    if (NEV) {
        const uint32_t umin = min(min(rw.w0, rw.w1), min(rw.w2, rw.w3));
        if (umin == 0u) {
            if (rw.w0 == 0u && ((never >> (a0 >> 2)) & 1u)) fl &= ~0x1u;
            if (rw.w1 == 0u && ((never >> (a1 >> 2)) & 1u)) fl &= ~0x100u;
            if (rw.w2 == 0u && ((never >> (a2 >> 2)) & 1u)) fl &= ~0x10000u;
            if (rw.w3 == 0u && ((never >> (a3 >> 2)) & 1u)) fl &= ~0x1000000u;
        }
    }
    return fl;
}

// Float to unsigned integer with the hardware's saturation (values at or
// above 2^32, infinity included, give 0xFFFFFFFF; negative values give 0).
__device__ __forceinline__ uint32_t cvt_u32_sat(float x) {
    uint32_t r;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// Continuous fields.  With up = number of +1 neighbours of a site and s
// its spin bit, J n + h h_i = 2J up + (h h_i - 6J) = 2J up + hfs (the
// second term precomputed per site), the flip costs dE = 2 (2s - 1) y with
// y = 2J up + hfs, and e^(-beta dE) = 2^x with
//   x = a (2s - 1) y = a (2s - 1) 2J up + a (2s - 1) hfs,  a = -2 beta log2(e).
// The two site-independent factors depend only on (up, s) at a given
// temperature: a per-slot LDS table holds them, entry (up << 1) | s =
// {a (2s - 1) 2J up, a (2s - 1)}, so x costs one FMA per site.  The integer
// bound is floor(2^x 2^32), saturated; dE <= 0 gives x >= 0 and the bound
// 0xFFFFFFFF, which every u32 meets: one integer test u <= bound covers
// both cases of the Metropolis rule.
__device__ __forceinline__ void cont_table_fill(uint32_t *sthr, float beta, float Jf) {
    const uint32_t q = threadIdx.x;
    if (q < 14u) {
        const float a = -2.0f * 1.44269504088896341f * beta;
        const float sa = (q & 1u) ? a : -a;
        const float two_j_up = 2.0f * Jf * (float)(q >> 1);
        sthr[2 * q] = __float_as_uint(sa * two_j_up);
        sthr[2 * q + 1] = __float_as_uint(sa);
    }
}

// The bound of one site from its table entry (at LDS byte offset e) and hfs.
__device__ __forceinline__ uint32_t cont_bound(const uint8_t *tb, uint32_t e, float hfs) {
    const float2 c = *(const float2 *)(tb + e);
    const float x = fmaf(c.y, hfs, c.x);
    return cvt_u32_sat(__builtin_amdgcn_exp2f(x) * 0x1p32f);
}

// Continuous fields: four sites of one Philox block, byte q of A the table
// entry offset (up << 4) | (s << 3) of site q; bit q set iff site q flips.
__device__ __forceinline__ uint32_t continuous_acc_at(const uint32_t *sthr, uint32_t A, const f32x4 hf,
                                                      const Words &rw) {
    const uint8_t *tb = (const uint8_t *)sthr;
    const uint32_t b0 = cont_bound(tb, A & 0xFFu, hf.x), b1 = cont_bound(tb, __builtin_amdgcn_ubfe(A, 8u, 8u), hf.y);
    const uint32_t b2 = cont_bound(tb, (A >> 16) & 0xFFu, hf.z), b3 = cont_bound(tb, A >> 24, hf.w);
    return accept_bits(rw.w0, rw.w1, rw.w2, rw.w3, b0, b1, b2, b3);
}

// The same from up counts U and spins Wown one per byte.
__device__ __forceinline__ uint32_t continuous_acc(const uint32_t *sthr, uint32_t U, uint32_t Wown, const f32x4 hf,
                                                   const Words &rw) {
    return continuous_acc_at(sthr, (U << 4) | (Wown << 3), hf, rw);
}

// Continuous fields: four sites of one Philox block, the flips one bit
// per byte.
__device__ __forceinline__ uint32_t continuous_flips(const uint32_t *sthr, uint32_t U, uint32_t Wown,
                                                     const f32x4 hf, const Words &rw) {
    return __umul24(continuous_acc(sthr, U, Wown, hf, rw), 0x204081u) & 0x01010101u;
}

// The words a chunk's half-sweep update reads: its own words, the
// other-colour words around it and its fields.
template <int KIND, int NW> struct ChunkIn {
    Chunk c;
    uint32_t Wown[NW];
    Around<NW> a;
    f32x4 HF[NW];   // continuous fields (KIND 1)
};

// Issue every load of a chunk (F4: the +-1 field bits, KIND 0).  Callers put
// a scheduling barrier after it so the compiler does not sink a load next to
// its use: with many realizations in a launch the fields and rows miss in
// L2, and a load issued per Philox block would expose the memory latency
// each time.
template <int KIND, int NW, class PO, class PC, class PB, class PF>
__device__ __forceinline__ void chunk_load(const Lattice &lat, PO own, PC oth, PB fb_own, PF hf_own, uint32_t j0,
                                           uint32_t colour, ChunkIn<KIND, NW> &in, uint32_t (&F4)[NW]) {
    in.c = chunk_geometry<NW>(j0, colour, (uint32_t)lat.L, (uint32_t)lat.log2L, (uint32_t)lat.half);
    load_words<NW>(own, j0, in.Wown);
    load_around<NW>(oth, j0, in.c, in.a);
    if (KIND == 0) {
        load_words<NW>(fb_own, j0, F4);
    } else {
#pragma unroll
        for (int w = 0; w < NW; ++w)
            in.HF[w] = *(typename rebind_ptr<PF, const f32x4>::type)(hf_own + j0 + 4u * w);
    }
}

// The flip decisions of a loaded chunk; returns nonzero if any site flips,
// with the new own words in Wnew (and the other-colour words and neighbour
// sums the energy pass reuses in W and U).
template <int KIND, int NW, bool NEV>
__device__ __forceinline__ uint32_t chunk_flip(const Lattice &lat, const uint32_t *sthr, uint32_t never,
                                               const ChunkIn<KIND, NW> &in, const uint32_t (&F4)[NW],
                                               uint32_t g0, uint32_t c1, uint32_t r, float beta,
                                               uint32_t (&W)[NW], uint32_t (&U)[NW], uint32_t (&Wnew)[NW]) {
    neighbour_sums<NW>(in.c, in.a, U);
#pragma unroll
    for (int w = 0; w < NW; ++w) W[w] = in.a.W[w];
    const uint32_t c3 = (kTagSweep << 28) | lat.rho;
    uint32_t any = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const Words rw = philox10(g0 + (uint32_t)w, c1, r, c3, lat.key0, lat.key1);
        uint32_t fl;
        if (KIND == 0) {
            fl = bimodal_flips<NEV>(sthr, U[w], in.Wown[w], F4[w], rw, never);
        } else {
            fl = continuous_flips(sthr, U[w], in.Wown[w], in.HF[w], rw);
        }
        any |= fl;
        Wnew[w] = in.Wown[w] ^ fl;
    }
    return any;
}

// chunk_flip with the never-class correction only where this slot has such
// classes (a wave-uniform branch between two copies).
template <int KIND, int NW>
__device__ __forceinline__ uint32_t chunk_flip_any(const Lattice &lat, const uint32_t *sthr, uint32_t never,
                                                   const ChunkIn<KIND, NW> &in, const uint32_t (&F4)[NW],
                                                   uint32_t g0, uint32_t c1, uint32_t r, float beta,
                                                   uint32_t (&W)[NW], uint32_t (&U)[NW], uint32_t (&Wnew)[NW]) {
    if (KIND == 0 && never != 0u) return chunk_flip<KIND, NW, true>(lat, sthr, never, in, F4, g0, c1, r, beta, W, U, Wnew);
    return chunk_flip<KIND, NW, false>(lat, sthr, never, in, F4, g0, c1, r, beta, W, U, Wnew);
}

// One chunk's half-sweep update: load, then flip.
template <int KIND, int NW, class PO, class PC, class PB, class PF>
__device__ __forceinline__ uint32_t chunk_update_any(const Lattice &lat, const uint32_t *sthr, uint32_t never,
                                                     PO own, PC oth, PB fb_own, PF hf_own, uint32_t j0,
                                                     uint32_t g0, uint32_t colour, uint32_t c1, uint32_t r,
                                                     float beta, uint32_t (&W)[NW], uint32_t (&U)[NW],
                                                     uint32_t (&Wnew)[NW], uint32_t (&F4)[NW]) {
    ChunkIn<KIND, NW> in;
    chunk_load<KIND, NW>(lat, own, oth, fb_own, hf_own, j0, colour, in, F4);
    __builtin_amdgcn_sched_barrier(0);
    return chunk_flip_any<KIND, NW>(lat, sthr, never, in, F4, g0, c1, r, beta, W, U, Wnew);
}

// f, negated where bit `bit` of `down` is set (the sign goes onto the FP32
// value, so it costs a shift and one three-input operation).
__device__ __forceinline__ double signed_field(float f, uint32_t down, int bit) {
    return (double)__uint_as_float(__float_as_uint(f) ^ ((down << (31 - bit)) & 0x80000000u));
}

// Energy pieces of a chunk of colour-1 sites and the colour-0 sites of the
// same pairs, from the final spins: every bond joins a colour-0 and a
// colour-1 site, so B = sum over colour-1 sites of s_i n_i counts each bond
// once; F and M take both colours.
template <int KIND, int NW, class PB, class PF>
__device__ __forceinline__ void chunk_energy(const Lattice &lat, const uint32_t (&S1)[NW],
                                             const uint32_t (&S0)[NW], const uint32_t (&U)[NW],
                                             const uint32_t (&F1)[NW], PB fb0, PF fr1, PF fr0, uint32_t j0,
                                             int &ksum, int &upsum, int &eqsum, double &fsum) {
    uint32_t F0[NW];
    if (KIND == 0) load_words<NW>(fb0, j0, F0);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint32_t Mb = S1[w] * 0xFFu;                                // 0x00 / 0xFF per byte
        const uint32_t K = (Mb & U[w]) | (~Mb & (0x06060606u - U[w]));  // aligned neighbours
        ksum = (int)__builtin_amdgcn_sad_u8(K, 0u, (uint32_t)ksum);
        upsum = (int)__builtin_amdgcn_sad_u8(S1[w] + S0[w], 0u, (uint32_t)upsum);
        if (KIND == 0) {
            const uint32_t e1 = ~(S1[w] ^ (F1[w] >> 2)) & 0x01010101u;
            const uint32_t e0 = ~(S0[w] ^ (F0[w] >> 2)) & 0x01010101u;
            eqsum = (int)__builtin_amdgcn_sad_u8(e1 + e0, 0u, (uint32_t)eqsum);
        } else {
            const f32x4 f1 = *(typename rebind_ptr<PF, const f32x4>::type)(fr1 + j0 + 4u * w);
            const f32x4 f0 = *(typename rebind_ptr<PF, const f32x4>::type)(fr0 + j0 + 4u * w);
            const float a1[4] = {f1.x, f1.y, f1.z, f1.w}, a0[4] = {f0.x, f0.y, f0.z, f0.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                fsum += signed_field(a1[q], ~S1[w], 8 * q);
                fsum += signed_field(a0[q], ~S0[w], 8 * q);
            }
        }
    }
}

// Block-wide (B, F, M) partial in a fixed order; thread 0..2 write it.  WAVES:
// the workgroup is whole waves.
template <int KIND, bool WAVES = true, class PD>
__device__ __forceinline__ void block_partial(PD dst, int nsite, int ksum, int upsum, int eqsum,
                                              double fsum) {
    __shared__ double red[3][16];
    const int bpart = 2 * ksum - 6 * nsite;
    const int mpart = 2 * upsum - 2 * nsite;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // integer sums over the wave's active lanes (DPP reduction in the
    // device library; exact, so the order does not matter)
    const int vb = __ockl_wfred_add_i32(bpart), vm = __ockl_wfred_add_i32(mpart);
    const double vf = KIND == 0 ? (double)__ockl_wfred_add_i32(2 * eqsum - 2 * nsite)
                                : (WAVES ? wave_sum(fsum) : part_wave_sum(fsum));
    if (lane == 0) {
        red[0][wave] = (double)vb;
        red[1][wave] = vf;
        red[2][wave] = (double)vm;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int nw = (int)((blockDim.x + 63) >> 6);
        double v = red[threadIdx.x][0];
        for (int q = 1; q < nw; ++q) v += red[threadIdx.x][q];
        dst[threadIdx.x] = v;
    }
}

__device__ __forceinline__ double energy_of(const Lattice &lat, double B, double F) {
    return -(lat.J * B) - (lat.h * F);
}

// The decision for pair (p, p+1) of exchange step k: Philox word pair ->
// a uniform double in [0, 1) with 53 random bits, accepted if Delta >= 0 or
// u < e^Delta.
__device__ __forceinline__ bool exchange_accept(const Lattice &lat, int p, uint64_t k, double delta) {
    const Words w = philox10((uint32_t)p, (uint32_t)k, 0u, (kTagExch << 28) | lat.rho, lat.key0, lat.key1);
    const double u53 = ((double)(w.w0 >> 11) * 4294967296.0 + (double)w.w1) * 0x1p-53;
    return delta >= 0.0 || u53 < exp(delta);
}

// Energy and magnetisation of replica r from its partials, added in the order
// of replica_totals.
__device__ __forceinline__ void partial_totals(const Lattice &lat, const StepIn &in, uint32_t r, double &E, double &M) {
    GAS const double *pp = (GAS const double *)in.part + 3 * (size_t)r;
    const size_t stride = 3 * (size_t)lat.pstride;
    double v[kMaxStepPartials][3];
#pragma unroll
    for (int q = 0; q < kMaxStepPartials; ++q)
        if (q < in.nblk)
#pragma unroll
            for (int i = 0; i < 3; ++i) v[q][i] = pp[(size_t)q * stride + i];
    double T[3] = {0.0, 0.0, 0.0}, g[3] = {0.0, 0.0, 0.0};
    int left = in.per;
#pragma unroll
    for (int q = 0; q < kMaxStepPartials; ++q) {
        if (q >= in.nblk) break;
#pragma unroll
        for (int i = 0; i < 3; ++i) g[i] += v[q][i];
        if (--left > 0 && q + 1 < in.nblk) continue;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            T[i] = q < in.per ? g[i] : T[i] + g[i];
            g[i] = 0.0;
        }
        left = in.per;
    }
    E = energy_of(lat, T[0], T[1]);
    M = T[2];
}

// The slot replica r sweeps at (first wave of a workgroup).  With a pending
// step, its pair's exchange first; `lead` (one workgroup per replica) records
// it: the permutation, the pair's counters if the replica was the colder one,
// and the sample of the slot the replica ends at.
// STEP is a template parameter of the kernels: the step's FP64 code costs
// scalar registers, and with them a wave per SIMD, that launches without one
// should not pay.
template <bool STEP>
__device__ __forceinline__ int take_slot(const Lattice &lat, const StepIn &in, uint32_t r, bool lead) {
    const int p = ((GAS const int32_t *)(in.r2t ? in.r2t : lat.r2t))[r];
    if (!STEP) return p;
    // the pairs of step k are (q, q + 1) with q = k mod 2
    const int lo = ((p ^ (int)in.k) & 1) == 0 ? p : p - 1;
    const bool pair = lo >= 0 && lo + 1 < lat.R;
    double E, M;
    partial_totals(lat, in, r, E, M);
    int slot = p;
    bool yes = false;
    if (pair) {
        const int other = p == lo ? lo + 1 : lo;
        const int b = ((GAS const int32_t *)in.t2r)[other];
        const double db = gptr(lat.beta)[lo + 1] - gptr(lat.beta)[lo];
        double Eb, Mb;
        partial_totals(lat, in, (uint32_t)b, Eb, Mb);
        const double delta = p == lo ? db * (Eb - E) : db * (E - Eb);
        yes = exchange_accept(lat, lo, in.k, delta);
        if (yes) slot = other;
    }
    if (lead) {
        if (threadIdx.x == 0) {
            in.r2t_out[r] = slot;
            in.t2r_out[slot] = (int32_t)r;
            if (pair && p == lo) {
                gptr(lat.att)[p] += 1;
                if (yes) gptr(lat.acc)[p] += 1;
            }
        }
        if (threadIdx.x < 6u) {
            const double m2 = M * M;
            const double add[6] = {1.0, E, E * E, fabs(M), m2, m2 * m2};
            double a = add[0];
#pragma unroll
            for (int q = 1; q < 6; ++q) a = threadIdx.x == (uint32_t)q ? add[q] : a;
            gptr(lat.obs)[6 * (size_t)slot + threadIdx.x] += a;
        }
    }
    return slot;
}

// The slot's table into LDS: thresholds (+-1 fields) or the continuous
// factors; by the first wave.
template <int KIND, bool STEP>
__device__ __forceinline__ void stage_table(const Lattice &lat, const StepIn &in, uint32_t r, bool lead, uint32_t *sthr) {
    if (threadIdx.x >= 64u) return;
    const int slot = take_slot<STEP>(lat, in, r, lead);
    if (KIND == 0) {
        if (threadIdx.x < 32u) sthr[threadIdx.x] = gptr(lat.thr)[slot * 32 + threadIdx.x];
    } else {
        cont_table_fill(sthr, gptr(lat.betaf)[slot], lat.Jf);
    }
}

// The same for the sizes whose decisions take the exponent's factor a.
template <int KIND, bool STEP>
__device__ __forceinline__ void stage_factor(const Lattice &lat, const StepIn &in, uint32_t r, bool lead, uint32_t *sthr) {
    if (threadIdx.x >= 64u) return;
    const int slot = take_slot<STEP>(lat, in, r, lead);
    if (KIND == 0) {
        if (threadIdx.x < 32u) sthr[threadIdx.x] = gptr(lat.thr)[slot * 32 + threadIdx.x];
    } else if (threadIdx.x == 0) {
        sthr[0] = __float_as_uint(-2.0f * 1.44269504088896341f * gptr(lat.betaf)[slot]);
    }
}

// Streaming half-sweep: one chunk per thread; one launch covers every
// replica of every realization listed in the block map (entry: realization,
// (replica << 16) | block within the replica), or, for one realization,
// replicas r0, r0 + 1, ... in block order.  ENERGY (colour 1 of the last
// sweep before an exchange) also writes one energy partial per workgroup.
template <int KIND, int NW, int ENERGY, bool BATCH>
__global__ __launch_bounds__(256) void sweep_pow2(Lattice lat0, const Lattice *__restrict__ lats,
                                                   const uint2 *__restrict__ map, int colour, int toff,
                                                   int remap, int lwpr, int r0) {
    __shared__ __align__(16) uint32_t sthr[32];   // +-1 thresholds or the continuous-field table
    uint32_t blk = blockIdx.x;
    if (remap) {
        // consecutive block ids go round-robin to the 8 XCDs; give each XCD a
        // contiguous range of tiles so that halo rows stay in its L2
        const uint32_t per = gridDim.x >> 3;
        blk = (blk & 7u) * per + (blk >> 3);
    }
    uint32_t r, gb;
    if (BATCH) {
        const uint2 e = map[blk];
        r = e.x & 0xFFFFu;
        gb = e.y;
    } else {
        r = (uint32_t)r0 + (blk >> lwpr);
        gb = blk & ((1u << lwpr) - 1u);
    }
    const Lattice &lat = BATCH ? lats[map[blk].x >> 16] : lat0;
    const uint32_t g0 = (gb * blockDim.x + threadIdx.x) * NW;   // first Philox block
    const uint32_t j0 = 4u * g0;
    const uint32_t col = (uint32_t)colour;
    GAS uint8_t *spins = gptr(lat.spins);
    GAS uint8_t *own = spins + (size_t)r * lat.N + (size_t)col * lat.half;
    GAS const uint8_t *oth = spins + (size_t)r * lat.N + (size_t)(1 - col) * lat.half;
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fhf = gptr(lat.fhf), *fraw = gptr(lat.fraw);
    // The chunk's loads go out first; the slot's table (r2t, then thr) is
    // fetched while they are in flight, so the workgroup's barrier on the
    // table costs the longer of the two chains rather than their sum.
    ChunkIn<KIND, NW> in;
    uint32_t F4[NW];
    chunk_load<KIND, NW>(lat, own, oth, fbits + (size_t)col * lat.half, fhf + (size_t)col * lat.half, j0, col, in,
                         F4);
    __builtin_amdgcn_sched_barrier(0);
    const int slot = gptr(lat.r2t)[r];
    const uint32_t t = (uint32_t)(gptr(lat.ctrs)[0] + (uint64_t)toff);
    uint32_t never = 0;
    const float beta = KIND == 1 ? gptr(lat.betaf)[slot] : 0.0f;
    if (KIND == 0) {
        if (threadIdx.x < 32u) sthr[threadIdx.x] = gptr(lat.thr)[slot * 32 + threadIdx.x];
        __syncthreads();
        never = __builtin_amdgcn_readfirstlane(sthr[31]);
    } else {
        cont_table_fill(sthr, beta, lat.Jf);
        __syncthreads();
    }
    uint32_t W[NW], U[NW], Wnew[NW];
    const uint32_t any = chunk_flip_any<KIND, NW>(lat, sthr, never, in, F4, g0, 2u * t + col, r, beta, W, U, Wnew);
    if (any) store_words<NW>(own, j0, Wnew);
    if (ENERGY) {
        int ksum = 0, upsum = 0, eqsum = 0;
        double fsum = 0.0;
        chunk_energy<KIND, NW>(lat, Wnew, W, U, F4, fbits, fraw + lat.half, fraw, j0, ksum, upsum, eqsum,
                               fsum);
        block_partial<KIND>(gptr(lat.part) + ((size_t)gb * lat.pstride + r) * 3, 4 * NW, ksum, upsum, eqsum,
                            fsum);
    }
}

// ---------------------------------------------------------------------
// Other even L (not a power of two, or below 8): four consecutive sublattice
// sites j0..j0+3 (one Philox block) of colour c, their spins one dword.  With
// ROWS (L a multiple of 8) they lie in one row and the neighbours are dwords,
// as in the chunks above; otherwise the neighbours are gathered as bytes.
// ---------------------------------------------------------------------

// What a site's field contributes: the +-1 field bits of the block, or its
// four continuous fields.
template <int KIND> struct BlockField {
    uint32_t F4 = 0u;
    f32x4 hf = {0.0f, 0.0f, 0.0f, 0.0f};
};

template <int KIND, class PB, class PF>
__device__ __forceinline__ BlockField<KIND> block_field(PB fb_own, PF hf_own, uint32_t j0) {
    BlockField<KIND> f;
    if (KIND == 0)
        f.F4 = *(typename rebind_ptr<PB, const uint32_t>::type)(fb_own + j0);
    else
        f.hf = *(typename rebind_ptr<PF, const f32x4>::type)(hf_own + j0);
    return f;
}

// The flips of a block, one bit per byte, from its up counts.
template <int KIND>
__device__ __forceinline__ uint32_t block_flips(const Lattice &lat, const uint32_t *sthr, uint32_t never, float a,
                                                const BlockField<KIND> &f, uint32_t U, uint32_t Wown, uint32_t g,
                                                uint32_t c1, uint32_t r) {
    const Words rw = philox10(g, c1, r, (kTagSweep << 28) | lat.rho, lat.key0, lat.key1);
    if (KIND == 0)
        return never != 0u ? bimodal_flips<true>(sthr, U, Wown, f.F4, rw, never)
                           : bimodal_flips<false>(sthr, U, Wown, f.F4, rw, never);
    const float h[4] = {f.hf.x, f.hf.y, f.hf.z, f.hf.w};
    uint32_t fl = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float up = (float)((U >> (8 * q)) & 0xFFu);
        if (cont_accept(up, h[q], 2.0f * lat.Jf, a, ((Wown >> (8 * q)) & 1u) != 0, word_at(rw, q))) fl |= 1u << (8 * q);
    }
    return fl;
}

// The same for a block of a whole replica in LDS, its neighbours gathered.
template <int KIND, class P, class PB, class PF>
__device__ __forceinline__ uint32_t any_flips(const Lattice &lat, const FastDiv &by_row, const FastDiv &by_l,
                                              const uint32_t *sthr, uint32_t never, float a, P oth, PB fb_own,
                                              PF hf_own, uint32_t j0, uint32_t Wown, uint32_t colour, uint32_t c1,
                                              uint32_t r) {
    const BlockField<KIND> f = block_field<KIND>(fb_own, hf_own, j0);
    uint32_t W[1];
    load_words<1>(oth, j0, W);
    const uint32_t U = site_counts(oth, j0, W[0], colour, (uint32_t)lat.L, by_row, by_l);
    return block_flips<KIND>(lat, sthr, never, a, f, U, Wown, j0 >> 2, c1, r);
}

// Half-sweep, one thread per block of four sites, the workgroups of replicas
// r0.. in one row.
// L = 48, R = 32, +-1 fields: 4.5 us a launch against 12.3 with a division
// per coordinate and site, byte neighbours and the table read from memory;
// about 3.5 us of it are the launch.  L = 80, R = 32: 11 us (12.2 without the
// XCD ranges; several replicas per thread were no faster).
template <int KIND, bool ROWS>
__global__ __launch_bounds__(256) void sweep_generic(Lattice lat, FastDiv by_row, FastDiv by_l, FastDiv by_blocks, int r0,
                                                     int colour, int toff) {
    __shared__ __align__(16) uint32_t sthr[32];
    // a contiguous range of blocks for each of the 8 XCDs (ids go round-robin
    // to them), so that the planes above and below are in its L2
    const uint32_t per = gridDim.x >> 3;
    const uint32_t blk = blockIdx.x < 8u * per ? (blockIdx.x & 7u) * per + (blockIdx.x >> 3) : blockIdx.x;
    const uint32_t rb = div_by(blk, by_blocks), r = (uint32_t)r0 + rb, half = (uint32_t)lat.half, col = (uint32_t)colour;
    const uint32_t j0 = 4u * ((blk - rb * by_blocks.d) * 256u + threadIdx.x);
    GAS uint8_t *own = gptr(lat.spins) + (size_t)r * lat.N + (size_t)col * half;
    GAS const uint8_t *oth = gptr((const uint8_t *)lat.spins) + (size_t)r * lat.N + (size_t)(1u - col) * half;
    // the block's loads go out first, the slot's table behind them (its two
    // round trips overlap theirs)
    const bool in = j0 < half;
    const uint32_t j = in ? j0 : 0u;
    const BlockField<KIND> f = block_field<KIND>(gptr(lat.fbits) + (size_t)col * half, gptr(lat.fhf) + (size_t)col * half, j);
    const uint32_t Wown = *(GAS const uint32_t *)(own + j);
    Around<1> ar;
    Chunk c;
    uint32_t U[1];
    if (ROWS) {
        c = row_chunk<1>(j, col, (uint32_t)lat.L, by_row, by_l);
        load_around<1>(oth, j, c, ar);
    } else {
        U[0] = site_counts(oth, j, *(GAS const uint32_t *)(oth + j), col, (uint32_t)lat.L, by_row, by_l);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int slot = gptr(lat.r2t)[r];
    const uint32_t t = (uint32_t)(gptr(lat.ctrs)[0] + (uint64_t)toff);
    uint32_t never = 0;
    float a = 0.0f;
    if (KIND == 0) {
        if (threadIdx.x < 32u) sthr[threadIdx.x] = gptr(lat.thr)[slot * 32 + threadIdx.x];
        __syncthreads();
        never = __builtin_amdgcn_readfirstlane(sthr[31]);
    } else {
        a = -2.0f * 1.44269504088896341f * gptr(lat.betaf)[slot];
    }
    if (ROWS) neighbour_sums<1>(c, ar, U);
    const uint32_t fl = block_flips<KIND>(lat, sthr, never, a, f, U[0], Wown, j >> 2, 2u * t + col, r);
    if (in && fl) *(GAS uint32_t *)(own + j0) = Wown ^ fl;
}

// Resident form (small L whose colour-planes do not hold whole blocks): one
// workgroup holds one replica's spins in LDS for `nsweep` whole sweeps and
// writes the energy partial of the final state, as sweep_resident does for
// powers of two.
template <int KIND, bool STEP>
__global__ __launch_bounds__(1024) void sweep_generic_resident(Lattice lat, StepIn in, FastDiv by_row, FastDiv by_l, int nsweep,
                                                                int energy) {
    extern __shared__ uint4 lds_raw[];
    __shared__ __align__(16) uint32_t sthr[32];
    uint8_t *sp = (uint8_t *)lds_raw;                  // [2][half]
    uint32_t *lds1 = (uint32_t *)lds_raw;
    const uint32_t r = blockIdx.x, half = (uint32_t)lat.half, words = (uint32_t)lat.N >> 2;
    // N is a multiple of 8: whole dwords
    GAS uint32_t *home = (GAS uint32_t *)(gptr(lat.spins) + (size_t)r * lat.N);
    for (uint32_t q = threadIdx.x; q < words; q += blockDim.x) lds1[q] = home[q];
    stage_factor<KIND, STEP>(lat, in, r, true, sthr);
    const uint32_t t0 = in.r2t ? in.t0 : (uint32_t)gptr(lat.ctrs)[0];
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fhf = gptr(lat.fhf), *fraw = gptr(lat.fraw);
    __syncthreads();
    const float a = KIND == 1 ? __uint_as_float(sthr[0]) : 0.0f;
    const uint32_t never = KIND == 0 ? __builtin_amdgcn_readfirstlane(sthr[31]) : 0u;
    for (int sw = 0; sw < nsweep; ++sw) {
        for (uint32_t col = 0; col < 2; ++col) {
            uint8_t *own = sp + col * half;
            const uint8_t *oth = sp + (1u - col) * half;
            const uint32_t c1 = 2u * (t0 + (uint32_t)sw) + col;
            for (uint32_t j0 = 4u * threadIdx.x; j0 < half; j0 += 4u * blockDim.x) {
                uint32_t Wown[1];
                load_words<1>((const uint8_t *)own, j0, Wown);
                const uint32_t fl =
                    any_flips<KIND>(lat, by_row, by_l, sthr, never, a, oth, fbits + (size_t)col * half,
                                          fhf + (size_t)col * half, j0, Wown[0], col, c1, r);
                if (fl) *(uint32_t *)(own + j0) = Wown[0] ^ fl;
            }
            __syncthreads();
        }
    }
    if (energy) {
        int ksum = 0, upsum = 0, eqsum = 0, n = 0;
        double fsum = 0.0;
        const uint8_t *s0 = sp, *s1 = sp + half;
        for (uint32_t j0 = 4u * threadIdx.x; j0 < half; j0 += 4u * blockDim.x, ++n) {
            uint32_t S1[1], W[1], U[1], F1[1];
            load_words<1>(s1, j0, S1);
            if (KIND == 0) load_words<1>(fbits + half, j0, F1);
            load_words<1>(s0, j0, W);
            U[0] = site_counts(s0, j0, W[0], 1u, (uint32_t)lat.L, by_row, by_l);
            chunk_energy<KIND, 1>(lat, S1, W, U, F1, fbits, fraw + half, fraw, j0, ksum, upsum, eqsum, fsum);
        }
        block_partial<KIND>(gptr(in.r2t ? in.part_out : lat.part) + (size_t)r * 3, 4 * n, ksum, upsum, eqsum, fsum);
    }
    for (uint32_t q = threadIdx.x; q < words; q += blockDim.x) home[q] = lds1[q];
}

// The place of a block in its colour-plane (byte d of it, its four sites in
// one row with ROWS, else in up to two) and the bytes of its neighbours there:
// computed once per thread, which keeps the place for a whole launch.
template <bool ROWS> struct Place {
    static constexpr int S = ROWS ? 1 : 4;      // sites with offsets of their own
    uint32_t d, y[S], xl[S], xr[S], yp[S], ym[S];
};

template <bool ROWS>
__device__ __forceinline__ Place<ROWS> place_of(uint32_t d, uint32_t L, const FastDiv &by_row) {
    const uint32_t Lh = L >> 1, plane = L * Lh, n = ROWS ? 4u : 1u;
    Place<ROWS> p;
    p.d = d;
    uint32_t y = div_by(d, by_row), m = d - y * Lh;
#pragma unroll
    for (int q = 0; q < Place<ROWS>::S; ++q) {
        const uint32_t j = d + (uint32_t)q;
        p.y[q] = y;
        p.xl[q] = m == 0u ? j + Lh - n : j - n;
        p.xr[q] = m + n == Lh ? j + n - Lh : j + n;
        p.yp[q] = y + 1u == L ? j + Lh - plane : j + Lh;
        p.ym[q] = y == 0u ? j + plane - Lh : j - Lh;
        if (!ROWS && ++m == Lh) {
            m = 0;
            ++y;                        // a plane holds whole blocks: y stays below L
        }
    }
    return p;
}

// Up counts of a block from the other colour's plane in LDS and its two
// neighbour planes; par = (colour + z) mod 2, W the block's other-colour sites.
template <bool ROWS>
__device__ __forceinline__ uint32_t plane_counts(const uint8_t *oth, const uint8_t *zp, const uint8_t *zm,
                                                 const Place<ROWS> &p, uint32_t par, uint32_t &W) {
    W = *(const uint32_t *)(oth + p.d);
    const uint32_t Wz = *(const uint32_t *)(zp + p.d) + *(const uint32_t *)(zm + p.d);
    if (ROWS) {
        const uint32_t right = (par + p.y[0]) & 1u;
        const uint32_t Wx = *(const uint32_t *)(oth + (right ? p.xr[0] : p.xl[0]));
        // as in neighbour_sums: the row shifted by one site
        const uint32_t Xs = __builtin_amdgcn_perm(Wx, W, right ? 0x04030201u : 0x02010007u);
        return W + Xs + Wz + *(const uint32_t *)(oth + p.yp[0]) + *(const uint32_t *)(oth + p.ym[0]);
    } else {
        uint32_t U = W + Wz;
#pragma unroll
        for (int q = 0; q < Place<ROWS>::S; ++q)
            U += ((uint32_t)oth[((par + p.y[q]) & 1u) ? p.xr[q] : p.xl[q]] + oth[p.yp[q]] + oth[p.ym[q]]) << (8 * q);
        return U;
    }
}

// Boxes (L a multiple of 4, so that a colour-plane holds whole blocks): a
// replica is cut along z into slabs of `np` planes (the last may be thinner),
// one workgroup each, and a launch runs `nsweep` whole sweeps in LDS on the
// slab and 2 nsweep halo planes on each side, which it recomputes instead of
// waiting for its neighbours, as sweep_slabs does; half-sweep s updates the
// planes [s + 1, P - 1 - s) of the box.  Reads `src`, writes `dst`.  A plane
// may appear twice in a box thicker than L - 1: both copies take the same
// updates from the same inputs as far as their halo reaches.  WHOLE: the box
// is the whole replica, periodic in z, without halo planes (any nsweep).
//
// A thread keeps one place of the plane and takes every G-th of the active
// planes (blockDim = G blocks-per-plane; the last wave may be partly empty,
// and filling it up cost 1 % at L = 48, R = 32).  Bound by instruction issue (104
// VALU instructions per block of four sites with whole-dword rows; 160 with
// the place worked out for every block) and, for thin slabs, by the launch
// and the staging: box_plan weighs them.  us a sweep, boxes against
// half-sweep launches (resident form at L = 24): L = 24, R = 32 3.3 and 3.9;
// L = 40, R = 32 6.0 and 8.4, R = 256 13.2 and 23.8; L = 48, R = 32 8.6 and
// 9.2; L = 52, R = 64 15.6 and 35.
template <int KIND, bool ROWS, bool WHOLE, bool STEP>
__global__ __launch_bounds__(1024) void sweep_box(Lattice lat, StepIn in, FastDiv by_row, FastDiv by_plane, FastDiv by_slab,
                                                   const uint8_t *__restrict__ src, uint8_t *__restrict__ dst, int np_,
                                                   int nsweep, int toff, int energy) {
    extern __shared__ uint4 lds_raw[];
    __shared__ __align__(16) uint32_t sthr[32];
    uint8_t *box = (uint8_t *)lds_raw;                       // [P][2][plane]
    const uint32_t L = (uint32_t)lat.L, half = (uint32_t)lat.half;
    const uint32_t plane = L * (L >> 1), bpp = plane >> 2;   // bytes and blocks per colour-plane
    const uint32_t r = div_by(blockIdx.x, by_slab), sl = blockIdx.x - r * by_slab.d;
    const uint32_t z0 = sl * (uint32_t)np_;
    const uint32_t np = min((uint32_t)np_, L - z0);
    const uint32_t H = WHOLE ? 0u : 2u * (uint32_t)nsweep, P = np + 2u * H;
    GAS const uint8_t *rsrc = gptr(src) + (size_t)r * lat.N;
    const uint32_t t0 = (in.r2t ? in.t0 : (uint32_t)gptr(lat.ctrs)[0]) + (uint32_t)toff;
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fhf = gptr(lat.fhf), *fraw = gptr(lat.fraw);
    // plane b of the box is plane z0 - H + b of the lattice (H <= L)
    auto z_of = [&](uint32_t b) {
        if (WHOLE) return b;
        uint32_t z = z0 + L - H + b;
        z -= z >= L ? L : 0u;
        return z - (z >= L ? L : 0u);
    };
    const uint32_t pg = div_by(threadIdx.x, by_plane), G = blockDim.x / bpp;   // this thread's first plane, planes per step
    const Place<ROWS> place = place_of<ROWS>(4u * (threadIdx.x - pg * bpp), L, by_row);
    // stage the box: the thread's block of its planes, both colours
    for (uint32_t b = pg; b < P; b += G) {
        const uint32_t at = z_of(b) * plane + place.d;
#pragma unroll
        for (uint32_t c = 0; c < 2; ++c)
            *(uint32_t *)(box + (2u * b + c) * plane + place.d) = *(GAS const uint32_t *)(rsrc + c * half + at);
    }
    stage_factor<KIND, STEP>(lat, in, r, sl == 0u, sthr);
    __syncthreads();
    const float a = KIND == 1 ? __uint_as_float(sthr[0]) : 0.0f;
    const uint32_t never = KIND == 0 ? __builtin_amdgcn_readfirstlane(sthr[31]) : 0u;
    for (uint32_t st = 0; st < 2u * (uint32_t)nsweep; ++st) {
        const uint32_t c = st & 1u, c1 = 2u * (t0 + (st >> 1)) + c;
        const uint32_t b0 = WHOLE ? 0u : st + 1u, b1 = WHOLE ? P : P - 1u - st;
        // (two or three planes of a thread at a time, their Philox chains
        // interleaved, were slower: the loop is bound by instruction issue)
        for (uint32_t b = b0 + pg; b < b1; b += G) {
            const uint32_t z = z_of(b), j0 = z * plane + place.d;
            const BlockField<KIND> f = block_field<KIND>(fbits + (size_t)c * half, fhf + (size_t)c * half, j0);
            uint8_t *own = box + (2u * b + c) * plane + place.d;
            const uint8_t *oth = box + (2u * b + 1u - c) * plane;
            const uint8_t *zp = WHOLE && b + 1u == P ? oth - 2u * (P - 1u) * plane : oth + 2u * plane;
            const uint8_t *zm = WHOLE && b == 0u ? oth + 2u * (P - 1u) * plane : oth - 2u * plane;
            const uint32_t Wown = *(const uint32_t *)own;
            uint32_t W;
            const uint32_t U = plane_counts<ROWS>(oth, zp, zm, place, c + z, W);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t fl = block_flips<KIND>(lat, sthr, never, a, f, U, Wown, j0 >> 2, c1, r);
            *(uint32_t *)own = Wown ^ fl;
        }
        __syncthreads();
    }
    if (energy) {
        int ksum = 0, upsum = 0, eqsum = 0, cnt = 0;
        double fsum = 0.0;
        for (uint32_t k = pg; k < np; k += G, ++cnt) {
            const uint32_t b = H + k, j0 = (z0 + k) * plane + place.d;
            const uint8_t *oth = box + 2u * b * plane;
            const uint8_t *zp = WHOLE && b + 1u == P ? box : oth + 2u * plane;
            const uint8_t *zm = WHOLE && b == 0u ? oth + 2u * (P - 1u) * plane : oth - 2u * plane;
            uint32_t S1[1], W[1], U[1], F1[1] = {0u};
            S1[0] = *(const uint32_t *)(oth + plane + place.d);
            U[0] = plane_counts<ROWS>(oth, zp, zm, place, 1u + z0 + k, W[0]);
            if (KIND == 0) load_words<1>(fbits + half, j0, F1);
            chunk_energy<KIND, 1>(lat, S1, W, U, F1, fbits, fraw + half, fraw, j0, ksum, upsum, eqsum, fsum);
        }
        block_partial<KIND, false>(gptr(in.r2t ? in.part_out : lat.part) + ((size_t)sl * lat.pstride + r) * 3, 4 * cnt, ksum,
                                   upsum, eqsum, fsum);
    }
    GAS uint8_t *rdst = gptr(dst) + (size_t)r * lat.N;
    for (uint32_t k = pg; k < np; k += G) {
#pragma unroll
        for (uint32_t c = 0; c < 2; ++c)
            *(GAS uint32_t *)(rdst + c * half + (z0 + k) * plane + place.d) =
                *(const uint32_t *)(box + (2u * (H + k) + c) * plane + place.d);
    }
}

// Resident sweeps (L = 2^l <= 32; few replicas at L = 8 run
// sweep_resident_ahead below): one workgroup holds one replica's spins
// in LDS and runs `nsweep` whole sweeps (colour 0 then colour 1, a barrier
// between half-sweeps), then, if asked, the energy partial of the final
// state, and writes the spins back.  Fields stay in global memory (shared
// by every replica, so they live in L2).
template <int KIND, int NW, bool BATCH, bool ONE, bool STEP>
__global__ __launch_bounds__(1024) void sweep_resident(Lattice lat0, const Lattice *__restrict__ lats,
                                                        const uint2 *__restrict__ map, StepIn in, int nsweep,
                                                        int energy) {
    extern __shared__ uint4 lds_raw[];
    __shared__ __align__(16) uint32_t sthr[32];   // +-1 thresholds or the continuous-field table
    uint8_t *sp = (uint8_t *)lds_raw;                  // [2][half]
    // batch: map entry (realization << 16 | replica, 0)
    const Lattice &lat = BATCH ? lats[map[blockIdx.x].x >> 16] : lat0;
    const uint32_t r = BATCH ? (map[blockIdx.x].x & 0xFFFFu) : blockIdx.x;
    const uint32_t N = (uint32_t)lat.N, half = (uint32_t)lat.half;
    GAS const u32x4 *src = (GAS const u32x4 *)(gptr(lat.spins) + (size_t)r * N);
    u32x4 *lds4 = (u32x4 *)lds_raw;
    for (uint32_t q = threadIdx.x; q < N / 16u; q += blockDim.x) lds4[q] = src[q];
    stage_table<KIND, STEP>(lat, in, r, true, sthr);
    const float beta = 0.0f;                           // the table holds what depends on it
    const uint32_t t0 = in.r2t ? in.t0 : (uint32_t)gptr(lat.ctrs)[0];
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fhf = gptr(lat.fhf), *fraw = gptr(lat.fraw);
    const uint32_t nchunk = half / (4u * NW);
    __syncthreads();
    const uint32_t never = KIND == 0 ? __builtin_amdgcn_readfirstlane(sthr[31]) : 0u;
    if constexpr (ONE) {
        // every thread owns chunk threadIdx.x of both colours: its fields
        // are read once per launch and kept in registers
        const uint32_t g0 = threadIdx.x * NW, j0 = 4u * g0;
        uint32_t F4c[2][NW];
        f32x4 HFc[2][NW];
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            if (KIND == 0) {
                load_words<NW>(fbits + (size_t)col * half, j0, F4c[col]);
            } else {
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    HFc[col][w] = *(GAS const f32x4 *)(fhf + (size_t)col * half + j0 + 4u * w);
            }
        }
        for (int sw = 0; sw < nsweep; ++sw) {
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                uint8_t *own = sp + col * half;
                const uint8_t *oth = sp + (1u - col) * half;
                const uint32_t c1 = 2u * (t0 + (uint32_t)sw) + col;
                ChunkIn<KIND, NW> in;
                in.c = chunk_geometry<NW>(j0, (uint32_t)col, (uint32_t)lat.L, (uint32_t)lat.log2L, half);
                load_words<NW>(own, j0, in.Wown);
                load_around<NW>(oth, j0, in.c, in.a);
                if (KIND == 1) {
#pragma unroll
                    for (int w = 0; w < NW; ++w) in.HF[w] = HFc[col][w];
                }
                uint32_t W[NW], U[NW], Wnew[NW];
                const uint32_t any = chunk_flip_any<KIND, NW>(lat, sthr, never, in, F4c[col], g0, c1, r, beta, W,
                                                              U, Wnew);
                if (any) store_words<NW>(own, j0, Wnew);
                __syncthreads();
            }
        }
    } else {
    for (int sw = 0; sw < nsweep; ++sw) {
        for (uint32_t col = 0; col < 2; ++col) {
            uint8_t *own = sp + col * half;
            const uint8_t *oth = sp + (1u - col) * half;
            const uint32_t c1 = 2u * (t0 + (uint32_t)sw) + col;
            for (uint32_t ch = threadIdx.x; ch < nchunk; ch += blockDim.x) {
                const uint32_t g0 = ch * NW, j0 = 4u * g0;
                uint32_t W[NW], U[NW], Wnew[NW], F4[NW];
                const uint32_t any = chunk_update_any<KIND, NW>(lat, sthr, never, own, oth, fbits + (size_t)col * half,
                                                            fhf + (size_t)col * half, j0, g0, col, c1, r, beta,
                                                            W, U, Wnew, F4);
                if (any) store_words<NW>(own, j0, Wnew);
            }
            __syncthreads();
        }
    }
    }
    if (energy) {
        int ksum = 0, upsum = 0, eqsum = 0;
        double fsum = 0.0;
        const uint8_t *s1 = sp + half, *s0 = sp;
        for (uint32_t ch = threadIdx.x; ch < nchunk; ch += blockDim.x) {
            const uint32_t j0 = 4u * NW * ch;
            const Chunk c = chunk_geometry<NW>(j0, 1u, (uint32_t)lat.L, (uint32_t)lat.log2L, half);
            uint32_t S1[NW], W[NW], U[NW], F1[NW];
            load_words<NW>(s1, j0, S1);
            neighbour_counts<NW>(s0, j0, c, W, U);
            if (KIND == 0) load_words<NW>(fbits + half, j0, F1);
            chunk_energy<KIND, NW>(lat, S1, W, U, F1, fbits, fraw + half, fraw, j0, ksum, upsum, eqsum, fsum);
        }
        // every thread covered 4*NW sites per chunk it took; nsite per thread
        // differs, so fold the affine offsets into the total instead
        const int nch = (int)((nchunk > threadIdx.x) ? (nchunk - 1 - threadIdx.x) / blockDim.x + 1 : 0);
        block_partial<KIND>(gptr(in.r2t ? in.part_out : lat.part) + (size_t)r * 3, 4 * NW * nch, ksum, upsum, eqsum, fsum);
    }
    GAS u32x4 *dst = (GAS u32x4 *)(gptr(lat.spins) + (size_t)r * N);
    for (uint32_t q = threadIdx.x; q < N / 16u; q += blockDim.x) dst[q] = lds4[q];
}

// L = 8, few replicas: a replica is one wave's worth of work, and the wave
// spends more than half of a half-sweep's instructions on the random words.
// Here its spins stay in the first wave's registers (lane: word of the row (y,
// z) = lane, both colours; the rows around it come from the other lanes) and
// three more waves, on the CU's other SIMDs, compute the words kWordsAhead
// half-sweeps at a time into LDS while the first one uses the batch before
// them (the first batch while it finds its slot).
// Bound by the first wave's own chain: an exchange, a table read and about 40
// instructions per half-sweep, 0.16 us (+-1; 0.25 in sweep_resident, where one
// wave does everything), and by the launch.  R = 16, ten sweeps and a step:
// +-1 9.99 -> 8.19 us, continuous 10.7 -> 8.87.
constexpr int kWordsAhead = 24;                 // half-sweeps per batch (even)
// While a CU has SIMDs for the extra waves: R = 512 12.8 -> 11.9 us, R = 768
// (continuous) 14.4 and 14.0, R = 1024 15.1 and 17.5.
constexpr int kAheadMaxReplicas = 512;

template <int KIND, bool STEP>
__global__ __launch_bounds__(256) void sweep_resident_ahead(Lattice lat, StepIn in, int nsweep, int energy) {
    __shared__ u32x4 words[2][kWordsAhead][64];
    __shared__ __align__(16) uint32_t sthr[32];   // +-1 thresholds or the continuous-field table
    const uint32_t r = blockIdx.x, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t t0 = in.r2t ? in.t0 : (uint32_t)gptr(lat.ctrs)[0], c3 = (kTagSweep << 28) | lat.rho;
    const int steps = 2 * nsweep;
    auto produce = [&](int h0) {
        const int n = min(kWordsAhead, steps - h0), buf = (h0 / kWordsAhead) & 1;
        for (int k = (int)wave - 1; k < n; k += 3) {
            const Words w = philox10(lane, 2u * t0 + (uint32_t)(h0 + k), r, c3, lat.key0, lat.key1);
            words[buf][k][lane] = u32x4{w.w0, w.w1, w.w2, w.w3};
        }
    };
    GAS uint32_t *home = (GAS uint32_t *)(gptr(lat.spins) + (size_t)r * 512u) + lane;
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fraw = gptr(lat.fraw);
    uint32_t S[2] = {0u, 0u}, F4[2] = {0u, 0u};
    f32x4 HF[2];
    if (wave == 0u) {
#pragma unroll
        for (uint32_t c = 0; c < 2; ++c) {
            S[c] = home[64u * c];
            if (KIND == 0)
                F4[c] = ((GAS const uint32_t *)fbits)[64u * c + lane];
            else
                HF[c] = ((GAS const f32x4 *)gptr(lat.fhf))[64u * c + lane];
        }
        stage_table<KIND, STEP>(lat, in, r, true, sthr);
    } else {
        produce(0);
    }
    __syncthreads();
    const uint32_t never = KIND == 0 ? __builtin_amdgcn_readfirstlane(sthr[31]) : 0u;
    // lanes of the rows around (byte addresses), and the byte order that puts
    // the x neighbours of colour 0 below its sites (colour 1: the other one)
    const int yp = (int)(4u * ((lane & 56u) | ((lane + 1u) & 7u))), ym = (int)(4u * ((lane & 56u) | ((lane - 1u) & 7u)));
    const int zp = (int)(4u * ((lane + 8u) & 63u)), zm = (int)(4u * ((lane - 8u) & 63u));
    const bool odd = ((lane ^ (lane >> 3)) & 1u) != 0u;
    const uint32_t sel0 = odd ? 0x00030201u : 0x02010003u, sel1 = odd ? 0x02010003u : 0x00030201u;
    auto counts = [&](uint32_t w, uint32_t sel) {
        return w + __builtin_amdgcn_perm(w, w, sel) + (uint32_t)__builtin_amdgcn_ds_bpermute(yp, (int)w) +
               (uint32_t)__builtin_amdgcn_ds_bpermute(ym, (int)w) + (uint32_t)__builtin_amdgcn_ds_bpermute(zp, (int)w) +
               (uint32_t)__builtin_amdgcn_ds_bpermute(zm, (int)w);
    };
    for (int h0 = 0; h0 < steps; h0 += kWordsAhead) {
        if (wave == 0u) {
            const u32x4 *wd = &words[(h0 / kWordsAhead) & 1][0][lane];
            const int n = min(kWordsAhead, steps - h0);
            u32x4 next = wd[0];
            for (int k = 0; k < n; k += 2) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const Words rw = {next.x, next.y, next.z, next.w};
                    next = wd[64 * min(k + c + 1, n - 1)];
                    const uint32_t U = counts(S[1 - c], c ? sel1 : sel0);
                    if (KIND == 1)
                        S[c] ^= continuous_flips(sthr, U, S[c], HF[c], rw);
                    else if (never != 0u)
                        S[c] ^= bimodal_flips<true>(sthr, U, S[c], F4[c], rw, never);
                    else
                        S[c] ^= bimodal_flips<false>(sthr, U, S[c], F4[c], rw, 0u);
                }
            }
        } else if (h0 + kWordsAhead < steps) {
            produce(h0 + kWordsAhead);
        }
        __syncthreads();
    }
    if (energy) {
        int ksum = 0, upsum = 0, eqsum = 0, n = 0;
        double fsum = 0.0;
        if (wave == 0u) {
            const uint32_t S1[1] = {S[1]}, W[1] = {S[0]}, U[1] = {counts(S[0], sel1)}, F1[1] = {F4[1]};
            chunk_energy<KIND, 1>(lat, S1, W, U, F1, fbits, fraw + 256, fraw, 4u * lane, ksum, upsum, eqsum, fsum);
            n = 4;
        }
        block_partial<KIND>(gptr(in.r2t ? in.part_out : lat.part) + (size_t)r * 3, n, ksum, upsum, eqsum, fsum);
    }
    if (wave == 0u) {
        home[0] = S[0];
        home[64] = S[1];
    }
}

// ---------------------------------------------------------------------
// Slab sweeps (L = 16 or 32): each replica is cut along z into S slabs of
// L/S planes, one workgroup per (replica, slab), so that a few replicas
// still fill every CU.  A launch runs `nsweep` whole sweeps of the plain
// order: the workgroup stages its slab and 2 nsweep halo planes on each
// side (both colours) in LDS and runs the 2 nsweep half-sweeps there,
// half-sweep s updating the planes [s + 1, P - 1 - s) of the box; the
// outer planes it updates are other slabs', recomputed here from the same
// inputs and the same random words, so the slab's own planes end exactly
// as in the plain sweep and no workgroup waits for another.  The slab goes
// to `dst` (reading from `src`: a workgroup must not see a neighbour's new
// planes), and with `energy` the workgroup writes the energy partial of
// its slab.
//
// Work item: SW dwords (4 SW sites) of one row of one colour.  Thread t
// owns the box positions t, t + blockDim, ... (NP of them) for the whole
// launch and keeps their fields, both colours, in registers; a position is
// updated at the half-steps whose plane range holds it.  A plane has
// L * L / (8 SW) items: at L = 32 a wave's positions share one plane, so
// the test is uniform per wave.  Every size is a power of two: no divisions.
//
// Bound by its fixed part: of 9.2 us a launch (L = 32, R = 64, two sweeps) the
// four half-sweeps' instructions are about 3 us; the rest is the launch,
// staging, barriers and write-back.  An interval of ten sweeps 46.7 -> 45.9 us
// without the divisions.  The first half-sweep peeled, its random words made
// while the box is being staged: 47.4.
// ---------------------------------------------------------------------
template <int KIND, int NP, bool STEP>
__global__ __launch_bounds__(1024) void sweep_slabs(Lattice lat, StepIn in, const uint8_t *__restrict__ src,
                                                     uint8_t *__restrict__ dst, int S, int nsweep, int toff,
                                                     int energy) {
    constexpr int SW = 2;
    extern __shared__ uint4 lds_raw[];
    __shared__ __align__(16) uint32_t sthr[32];   // +-1 thresholds or the continuous-field table
    uint8_t *box = (uint8_t *)lds_raw;                     // [P][2][plane]
    const uint32_t L = (uint32_t)lat.L, half = (uint32_t)lat.half;
    const uint32_t rowb = L >> 1;                          // bytes per row of one colour
    const uint32_t nwr = L >> 3;                           // dwords per row of one colour
    const uint32_t lipr = (uint32_t)lat.log2L - 4u;        // log2 of items per row (nwr / SW)
    const uint32_t ipr = 1u << lipr;
    const uint32_t plane = L * rowb;                       // bytes per plane of one colour
    const uint32_t ipp = L << lipr;                        // items per plane
    const uint32_t ls = (uint32_t)__builtin_ctz((uint32_t)S);
    const uint32_t slab = L >> ls;
    const uint32_t H = 2u * (uint32_t)nsweep;
    const uint32_t P = slab + 2u * H;
    const uint32_t r = blockIdx.x >> ls, sl = blockIdx.x & ((uint32_t)S - 1u);
    const uint32_t z0 = sl * slab;
    GAS const uint8_t *rsrc = gptr(src) + (size_t)r * lat.N;
    const float beta = 0.0f;                               // the table holds what depends on it
    const uint32_t t0 = (in.r2t ? in.t0 : (uint32_t)gptr(lat.ctrs)[0]) + (uint32_t)toff;
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fhf = gptr(lat.fhf), *fraw = gptr(lat.fraw);
    // the positions of this thread and their fields (issued first, so the
    // field loads overlap the staging loads)
    uint32_t pb[NP], py[NP], pz[NP], pw[NP];
    uint32_t F4c[2][NP][SW];
    f32x4 HFc[2][NP][SW];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const uint32_t pos = threadIdx.x + (uint32_t)k * blockDim.x;
        const uint32_t rem = pos & (ipp - 1u);
        pb[k] = pos >> ((uint32_t)lat.log2L + lipr);       // P or more when the position is past the box
        py[k] = rem >> lipr;
        pw[k] = SW * (rem & (ipr - 1u));
        pz[k] = (z0 + L - H + pb[k]) & (L - 1u);
        const uint32_t j0 = (pz[k] * L + py[k]) * rowb + 4u * pw[k];
        if (pb[k] < P) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (KIND == 0) {
                    load_words<SW>(fbits + (size_t)c * half, j0, F4c[c][k]);
                } else {
#pragma unroll
                    for (int w = 0; w < SW; ++w)
                        HFc[c][k][w] = *(GAS const f32x4 *)(fhf + (size_t)c * half + j0 + 4u * w);
                }
            }
        }
    }
    // stage the box, 16 bytes at a time: plane b of the box is z0 - H + b
    const uint32_t lp16 = 2u * (uint32_t)lat.log2L - 5u, per_plane16 = 1u << lp16;
    const uint32_t n16 = P * 2u * per_plane16;
    for (uint32_t e = threadIdx.x; e < n16; e += blockDim.x) {
        const uint32_t q = e & (per_plane16 - 1u), bc = e >> lp16;   // bc = 2 b + c
        const uint32_t b = bc >> 1, c = bc & 1u;
        const uint32_t zg = (z0 + L - H + b) & (L - 1u);
        ((u32x4 *)box)[e] = *(GAS const u32x4 *)(rsrc + (size_t)c * half + (size_t)zg * plane + 16u * q);
    }
    stage_table<KIND, STEP>(lat, in, r, sl == 0u, sthr);
    const uint32_t *bw = (const uint32_t *)box;
    const uint32_t ppw = plane >> 2;                       // dwords per colour-plane
    __syncthreads();
    const uint32_t never = KIND == 0 ? __builtin_amdgcn_readfirstlane(sthr[31]) : 0u;
    for (int sw = 0; sw < nsweep; ++sw) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t st = 2u * (uint32_t)sw + (uint32_t)c;
            const uint32_t c1 = 2u * (t0 + (uint32_t)sw) + (uint32_t)c;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                if (pb[k] >= st + 1u && pb[k] + 1u + st < P) {
                    const uint32_t b = pb[k], y = py[k], w0 = pw[k], zg = pz[k];
                    const uint32_t rown = (2u * b + (uint32_t)c) * ppw + y * nwr;
                    const uint32_t oth = (2u * b + 1u - (uint32_t)c) * ppw;
                    ChunkIn<KIND, SW> in;
                    in.c.p = ((uint32_t)c + y + zg) & 1u;
#pragma unroll
                    for (int w = 0; w < SW; ++w) {
                        in.Wown[w] = bw[rown + w0 + w];
                        in.a.W[w] = bw[oth + y * nwr + w0 + w];
                        in.a.Wyp[w] = bw[oth + ((y + 1u) & (L - 1u)) * nwr + w0 + w];
                        in.a.Wym[w] = bw[oth + ((y - 1u) & (L - 1u)) * nwr + w0 + w];
                        in.a.Wzp[w] = bw[oth + 2u * ppw + y * nwr + w0 + w];
                        in.a.Wzm[w] = bw[oth - 2u * ppw + y * nwr + w0 + w];
                        if (KIND == 1) in.HF[w] = HFc[c][k][w];
                    }
                    in.a.Wx = bw[oth + y * nwr + ((w0 + (in.c.p ? (uint32_t)SW : nwr - 1u)) & (nwr - 1u))];
                    const uint32_t g0 = ((pz[k] * L + y) * rowb >> 2) + w0;
                    uint32_t W[SW], U[SW], Wnew[SW];
                    const uint32_t any = chunk_flip_any<KIND, SW>(lat, sthr, never, in, F4c[c][k], g0, c1, r, beta,
                                                                  W, U, Wnew);
                    if (any) {
#pragma unroll
                        for (int w = 0; w < SW; ++w) ((uint32_t *)box)[rown + w0 + w] = Wnew[w];
                    }
                }
            }
            __syncthreads();
        }
    }
    if (energy) {
        // the slab's colour-1 items against the final colour-0 planes (the
        // last colour-0 half-sweep covered the slab and one plane each side)
        int ksum = 0, upsum = 0, eqsum = 0, nch = 0;
        double fsum = 0.0;
        for (uint32_t it = threadIdx.x; it < slab * ipp; it += blockDim.x, ++nch) {
            const uint32_t bs = it >> ((uint32_t)lat.log2L + lipr), rem = it & (ipp - 1u);
            const uint32_t b = H + bs, y = rem >> lipr, w0 = SW * (rem & (ipr - 1u));
            const uint32_t zg = z0 + bs;
            const uint32_t j0 = (zg * L + y) * rowb + 4u * w0;
            const uint32_t o0 = (2u * b) * ppw;
            Around<SW> a;
            Chunk cg;
            cg.p = (1u + y + zg) & 1u;
            uint32_t S1[SW], U[SW], F1[SW];
#pragma unroll
            for (int w = 0; w < SW; ++w) {
                a.W[w] = bw[o0 + y * nwr + w0 + w];
                a.Wyp[w] = bw[o0 + ((y + 1u) & (L - 1u)) * nwr + w0 + w];
                a.Wym[w] = bw[o0 + ((y - 1u) & (L - 1u)) * nwr + w0 + w];
                a.Wzp[w] = bw[o0 + 2u * ppw + y * nwr + w0 + w];
                a.Wzm[w] = bw[o0 - 2u * ppw + y * nwr + w0 + w];
                S1[w] = bw[(2u * b + 1u) * ppw + y * nwr + w0 + w];
                F1[w] = 0u;
            }
            a.Wx = bw[o0 + y * nwr + ((w0 + (cg.p ? (uint32_t)SW : nwr - 1u)) & (nwr - 1u))];
            neighbour_sums<SW>(cg, a, U);
            if (KIND == 0) load_words<SW>(fbits + half, j0, F1);
            chunk_energy<KIND, SW>(lat, S1, a.W, U, F1, fbits, fraw + half, fraw, j0, ksum, upsum, eqsum, fsum);
        }
        block_partial<KIND>(gptr(in.r2t ? in.part_out : lat.part) + ((size_t)sl * lat.pstride + r) * 3, 4 * SW * nch, ksum,
                            upsum, eqsum, fsum);
    }
    // the slab's planes, both colours
    GAS uint8_t *rdst = gptr(dst) + (size_t)r * lat.N;
    const uint32_t m16 = slab * 2u * per_plane16;
    for (uint32_t e = threadIdx.x; e < m16; e += blockDim.x) {
        const uint32_t q = e & (per_plane16 - 1u), bc = e >> lp16;
        const uint32_t bs = bc >> 1, c = bc & 1u;
        *(GAS u32x4 *)(rdst + (size_t)c * half + (size_t)(z0 + bs) * plane + 16u * q) =
            ((const u32x4 *)box)[(2u * (H + bs) + c) * per_plane16 + q];
    }
}

// ---------------------------------------------------------------------
// Double checkerboard with multi-hit updates (Sec. 3.2, Sec. 5.2): one
// workgroup per (replica, tile of the coarse colour), tile of tx * ty * tz
// sites (tx a multiple of 8).  The tile and a one-site halo around it are
// staged in LDS in the colour-split row layout of global memory: per colour
// and per row (y, z) of the box (the tile's rows and one halo row on each
// side in y and z), tx/2 bytes of the tile's sites with one dword before
// (the left neighbour tile's last four sites of that colour) and one after
// (the right neighbour's first four).  Every thread owns one dword (four
// consecutive sites of a colour in a row) of each colour and runs `hits`
// local sweeps -- its colour-0 dword, a barrier, its colour-1 dword, a
// barrier -- with the same neighbour sums and decisions as the streaming
// sweep; the halo is never written, so the neighbouring tiles stay frozen.
// Hit m of sweep t draws the tag-2 block (j >> 2, 2 (t hits + m) + c, r).
// Then the tile goes back to global memory.
// ---------------------------------------------------------------------
template <int KIND>
__global__ __launch_bounds__(1024) void sweep_tiles(Lattice lat, TileShape ts, int coarse, int toff) {
    extern __shared__ uint4 lds_raw[];
    __shared__ __align__(16) uint32_t sthr[32];   // +-1 thresholds or the continuous-field table
    uint8_t *box = (uint8_t *)lds_raw;
    const uint32_t L = (uint32_t)lat.L, half = (uint32_t)lat.half;
    const uint32_t tx = (uint32_t)ts.tx, ty = (uint32_t)ts.ty, tz = (uint32_t)ts.tz;
    const uint32_t dwr = tx >> 3;                   // tile dwords per row and colour
    const uint32_t rowb = 4u * (dwr + 2u);          // bytes per box row (with the halo dwords)
    const uint32_t by = ty + 2u;
    const uint32_t plane = rowb * by * (tz + 2u);   // bytes per colour
    // block -> (replica, tile of the coarse colour)
    const uint32_t dxh = L / tx / 2u, Dy = L / ty;
    const uint32_t ntile = dxh * Dy * (L / tz);
    const uint32_t r = blockIdx.x / ntile, q = blockIdx.x % ntile;
    const uint32_t Y = (q / dxh) % Dy, Z = q / (dxh * Dy);
    const uint32_t X = 2u * (q % dxh) + (((uint32_t)coarse + Y + Z) & 1u);
    const uint32_t x0 = X * tx, y0 = Y * ty, z0 = Z * tz;
    GAS uint8_t *spins = gptr(lat.spins) + (size_t)r * lat.N;
    const int slot = gptr(lat.r2t)[r];
    if (KIND == 0 && threadIdx.x < 32u) sthr[threadIdx.x] = gptr(lat.thr)[slot * 32 + threadIdx.x];
    const float beta = KIND == 1 ? gptr(lat.betaf)[slot] : 0.0f;
    if (KIND == 1) cont_table_fill(sthr, beta, lat.Jf);
    const uint32_t t = (uint32_t)(gptr(lat.ctrs)[0] + (uint64_t)toff);
    // stage the box: both colours, every row of the box, the tile's dwords
    // and the two halo dwords (x, y, z wrap around the periodic lattice)
    const uint32_t nbox = 2u * (dwr + 2u) * by * (tz + 2u);
    for (uint32_t e = threadIdx.x; e < nbox; e += blockDim.x) {
        const uint32_t d = e % (dwr + 2u), row = (e / (dwr + 2u)) % (by * (tz + 2u));
        const uint32_t c = e / ((dwr + 2u) * by * (tz + 2u));
        const uint32_t yy = row % by, zz = row / by;
        const uint32_t x = (x0 + L + 8u * d - 8u) & (L - 1u);
        const uint32_t y = (y0 + L + yy - 1u) & (L - 1u), z = (z0 + L + zz - 1u) & (L - 1u);
        const uint32_t j = (x + L * (y + L * z)) >> 1;
        *(uint32_t *)(box + c * plane + row * rowb + 4u * d) =
            *(GAS const uint32_t *)(spins + (size_t)c * half + j);
    }
    // this thread's dword: four sites of row (y0 + yy, z0 + zz) from
    // x0 + 8w, in each colour
    const uint32_t w = threadIdx.x % dwr, yy = (threadIdx.x / dwr) % ty, zz = threadIdx.x / (dwr * ty);
    const uint32_t j0 = (x0 + 8u * w + L * ((y0 + yy) + L * (z0 + zz))) >> 1;
    const uint32_t g0 = j0 >> 2;
    const uint32_t mid = ((zz + 1u) * by + (yy + 1u)) * rowb + 4u * (w + 1u);
    uint32_t F4[2][1] = {{0u}, {0u}};
    f32x4 HF[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        if (KIND == 0) {
            F4[c][0] = *(GAS const uint32_t *)(gptr(lat.fbits) + (size_t)c * half + j0);
        } else {
            HF[c] = *(GAS const f32x4 *)(gptr(lat.fhf) + (size_t)c * half + j0);
        }
    }
    __syncthreads();
    const uint32_t never = KIND == 0 ? __builtin_amdgcn_readfirstlane(sthr[31]) : 0u;
    const uint32_t p0 = (y0 + yy + z0 + zz) & 1u;   // (c + y + z) & 1 for colour 0
    for (int m = 0; m < ts.hits; ++m) {
        const uint32_t step = t * (uint32_t)ts.hits + (uint32_t)m;
#pragma unroll
        for (uint32_t c = 0; c < 2; ++c) {
            const uint8_t *oth = box + (1u - c) * plane;
            ChunkIn<KIND, 1> in;
            in.c.p = p0 ^ c;
            in.Wown[0] = *(const uint32_t *)(box + c * plane + mid);
            in.a.W[0] = *(const uint32_t *)(oth + mid);
            in.a.Wx = *(const uint32_t *)(oth + mid + (in.c.p ? 4u : 0u - 4u));
            in.a.Wyp[0] = *(const uint32_t *)(oth + mid + rowb);
            in.a.Wym[0] = *(const uint32_t *)(oth + mid - rowb);
            in.a.Wzp[0] = *(const uint32_t *)(oth + mid + rowb * by);
            in.a.Wzm[0] = *(const uint32_t *)(oth + mid - rowb * by);
            if (KIND == 1) in.HF[0] = HF[c];
            uint32_t Wn[1], Un[1], Wnew[1];
            const uint32_t any = chunk_flip_any<KIND, 1>(lat, sthr, never, in, F4[c], g0, 2u * step + c, r, beta,
                                                         Wn, Un, Wnew);
            if (any) *(uint32_t *)(box + c * plane + mid) = Wnew[0];
            __syncthreads();
        }
    }
#pragma unroll
    for (uint32_t c = 0; c < 2; ++c)
        *(GAS uint32_t *)(spins + (size_t)c * half + j0) = *(const uint32_t *)(box + c * plane + mid);
}

// ---------------------------------------------------------------------
// One bit per spin (multi-spin coding), L = 2^l in [64, 256].  Colour c of
// replica r is N/64 words; word w holds sublattice indices 32w..32w+31,
// index 32w + 4b + q at bit 8q + b, so that the four sites of Philox block
// 8w + b sit at bit b of the four bytes.  A row (y, z) of one colour is
// L/64 consecutive words.  One thread per word of the updated colour: the
// other colour's words around it are the pair word W (the same indices), W
// shifted by one index along the row with the neighbouring word's end bit
// (index m-1 when (c+y+z) is even, m+1 when odd, as in the byte layout),
// and the words of rows y+-1 and z+-1.  A bit-sliced full-adder tree turns
// the six into three planes of the up count; a bit transpose of the class
// planes gives every Philox block's byte-per-site table offsets, the
// operands of the byte sweep's decision, which runs on the same random
// words, so the chain is the same.  (Two words per thread, tried, ran the
// two-stream half-sweep 8 % slower: fewer waves to hide latency.)
// ---------------------------------------------------------------------
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
// position of sublattice index i (0..31) within its word
__host__ __device__ constexpr uint32_t bit_of_index(uint32_t i) { return 8u * (i & 3u) + (i >> 2); }

// Exchange the bits of a at positions i + sh with the bits of b at
// positions i, for the positions i that mask m selects: two shifts and two
// bit selects (table 0xD8: the third operand chooses the second over the
// first); the three-XOR swap takes one more.
__device__ __forceinline__ void swap_bit_groups(uint32_t &a, uint32_t &b, uint32_t sh, uint32_t m) {
    const uint32_t x = a >> sh, y = b << sh;
    a = __builtin_amdgcn_bitop3_b32(a, y, m << sh, 0xD8);
    b = __builtin_amdgcn_bitop3_b32(b, x, m, 0xD8);
}

// Table offsets of all eight Philox blocks of a word at once.  Byte q of
// plane k holds bit b for block b; the table offset of site (b, q) wants
// those five bits side by side, at bits 2 (f), 3 (s), 4..6 (up count).  With
// planes 0, 1 and 7 zero that is an 8x8 bit transpose inside every byte:
// three rounds of swapping bit groups of 4, 2 and 1 between planes, after
// which plane b is byte-per-site offset word A[b] = (U << 4) | (S << 3) | (F << 2)
// of block b.
__device__ __forceinline__ void class_offsets(uint32_t u0, uint32_t u1, uint32_t u2, uint32_t s, uint32_t f,
                                              uint32_t (&A)[8]) {
    uint32_t x[8] = {0u, 0u, f, s, u0, u1, u2, 0u};
#pragma unroll
    for (int k = 0; k < 4; ++k) swap_bit_groups(x[k], x[k + 4], 4u, 0x0F0F0F0Fu);
    swap_bit_groups(x[0], x[2], 2u, 0x33333333u);
    swap_bit_groups(x[1], x[3], 2u, 0x33333333u);
    swap_bit_groups(x[4], x[6], 2u, 0x33333333u);
    swap_bit_groups(x[5], x[7], 2u, 0x33333333u);
#pragma unroll
    for (int k = 0; k < 8; k += 2) swap_bit_groups(x[k], x[k + 1], 1u, 0x55555555u);
#pragma unroll
    for (int b = 0; b < 8; ++b) A[b] = x[b];
}

// sum of f_i s_i over the 32 sites of each of a wave's 64 consecutive words
// (bits S, words w0..w0+63 of one colour whose fields start at f), added up
// per lane in another order of the sites: float4 number 64k + lane of the
// wave's 2048 fields belongs to word 8k + lane / 8, block lane % 8, whose bits
// come from that word's lane.  Every load is one 1 KiB run; a thread reading
// its own word's fields (128 B apart in the wave) made the energy half-sweep
// of L = 64, R = 128 take 12.5 us against 7.3 without energies, 10.7 so.
__device__ __forceinline__ double bits_field_sum(GAS const float *f, uint32_t w0, uint32_t S) {
    const uint32_t lane = threadIdx.x & 63u;
    GAS const f32x4 *f4 = (GAS const f32x4 *)f + (size_t)w0 * 8u + lane;
    double sum = 0.0;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
        const f32x4 v = f4[64u * k];
        const uint32_t down =
            ~((uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * (8u * k + (lane >> 3))), (int)S) >> (lane & 7u));
        sum += signed_field(v.x, down, 0);
        sum += signed_field(v.y, down, 8);
        sum += signed_field(v.z, down, 16);
        sum += signed_field(v.w, down, 24);
    }
    return sum;
}

// Aligned neighbours of a word's 32 sites (up if s = +1, 6 - up if s = -1)
// from the three planes of the up count.
__device__ __forceinline__ int bits_aligned(uint32_t U0, uint32_t U1, uint32_t U2, uint32_t S) {
    const uint32_t nS = ~S;
    const int up_on = __popc(U0 & S) + 2 * __popc(U1 & S) + 4 * __popc(U2 & S);
    const int up_off = __popc(U0 & nS) + 2 * __popc(U1 & nS) + 4 * __popc(U2 & nS);
    return up_on + 6 * (32 - __popc(S)) - up_off;
}

constexpr int kBitsThreads = 256;

// A word of a colour's bit array, addressed as a wave-uniform base plus a
// 32-bit byte offset (one vector register per load instead of a 64-bit
// address).
__device__ __forceinline__ uint32_t bits_word(GAS const uint32_t *base, uint32_t byte) {
    return *(GAS const uint32_t *)((GAS const char *)base + byte);
}

// The words around word w of colour c's index space, as byte offsets.  The
// offset 4 w = 4 ((z L + y) words-per-row + wr) has the bit fields of wr, y and
// z side by side, so a neighbour's is a step inside one field, put back (the
// step's carry or borrow out of the field masked off: periodic wrap).  x: the
// word that holds index m - 1 (p = 0) or m + 1 (p = 1).
struct BitsAround {
    uint32_t own, x, yp, ym, zp, zm, p;
};

__device__ __forceinline__ BitsAround bits_around(const Lattice &lat, uint32_t w, uint32_t c) {
    const uint32_t L = (uint32_t)lat.L, l = (uint32_t)lat.log2L, lrw = l - 6u;
    const uint32_t y1 = 4u << lrw, z1 = y1 << l;
    const uint32_t xf = y1 - 4u, yf = (L - 1u) << (lrw + 2u), zf = yf << l;
    BitsAround a;
    a.own = 4u * w;
    a.p = (c + (w >> lrw) + (w >> (lrw + l))) & 1u;                   // (c + y + z) mod 2
    a.x = ((a.own + 8u * a.p - 4u) & xf) | (a.own & ~xf);
    a.yp = ((a.own + y1) & yf) | (a.own & ~yf);
    a.ym = ((a.own - y1) & yf) | (a.own & ~yf);
    a.zp = ((a.own + z1) & zf) | (a.own & ~zf);
    a.zm = ((a.own - z1) & zf) | (a.own & ~zf);
    return a;
}

// Up counts of a word's 32 sites in three bit planes.  The x neighbour, index
// m - 1 or m + 1, in the interleaved order: a step of one index is a step of
// one byte, with the carry between byte 3 and byte 0 one bit along, and the
// end bit from the neighbouring word of the row (around the row).
__device__ __forceinline__ void bits_planes(uint32_t p, uint32_t W, uint32_t Wn, uint32_t Wyp, uint32_t Wym, uint32_t Wzp,
                                            uint32_t Wzm, uint32_t &U0, uint32_t &U1, uint32_t &U2) {
    const uint32_t Wx = p ? ((W >> 8) | ((W << 23) & 0x7F000000u) | (Wn << 31))
                          : ((W << 8) | ((W >> 23) & 0x000000FEu) | (Wn >> 31));
    const uint32_t s1 = xor3(W, Wx, Wyp), c1 = maj3(W, Wx, Wyp);
    const uint32_t s2 = xor3(Wym, Wzp, Wzm), c2 = maj3(Wym, Wzp, Wzm);
    const uint32_t c3 = s1 & s2;
    U0 = s1 ^ s2;
    U1 = xor3(c1, c2, c3);
    U2 = maj3(c1, c2, c3);
}

// Flip bits of one word of the bit sweep (its 32 sites, eight Philox
// blocks), in the word's bit order.  NEV: the slot has classes that can
// never flip (+-1 fields), checked per block; the common case runs
// without that check.  (Interleaving the blocks' Philox chains by hand,
// two, four or eight at a time, was no faster: the sweep is bound by
// instruction issue, not by the chains' latency.  Nor was a loop of one, two
// or four blocks a turn, less code to fetch: L = 64, R = 192 21.6 us a sweep
// unrolled, 22.2 to 22.5 so.)
template <int KIND, bool NEV>
__device__ __forceinline__ uint32_t word_flips(const uint32_t *sthr, uint32_t never, const uint32_t (&Acls)[8],
                                               const f32x4 (&HF)[8], uint32_t w, uint32_t m0v, uint32_t c1w,
                                               uint32_t r, uint32_t c3w, uint32_t key0, uint32_t key1) {
    const uint8_t *tb = (const uint8_t *)sthr;
    uint32_t f0 = 0, f1 = 0, f2 = 0, f3 = 0;
#pragma unroll
    for (int b = 7; b >= 0; --b) {
        // block counters 8w + b: the first product M0 (8w + b) is one
        // multiply-add of 8w with the constant M0 b
        const Words rw = philox10_p(mad_m0(8u * w, m0v, (uint64_t)kPhiloxM0 * (uint32_t)b), 8u * w + b, c1w, r,
                                    c3w, key0, key1);
        const uint32_t A = Acls[b];
        const uint32_t a0 = A & 0xFFu, a1 = __builtin_amdgcn_ubfe(A, 8u, 8u), a2 = (A >> 16) & 0xFFu, a3 = A >> 24;
        if (KIND == 0) {
            const uint32_t th0 = *(const uint32_t *)(tb + a0), th1 = *(const uint32_t *)(tb + a1);
            const uint32_t th2 = *(const uint32_t *)(tb + a2), th3 = *(const uint32_t *)(tb + a3);
            accept_shift(rw.w0, rw.w1, rw.w2, rw.w3, th0, th1, th2, th3, f0, f1, f2, f3);
            if (NEV) {
                // a class that can never flip at this temperature has entry
                // 0, which u = 0 would meet: clear the bit just shifted in
                const uint32_t umin = min(min(rw.w0, rw.w1), min(rw.w2, rw.w3));
                if (umin == 0u) {
                    if (rw.w0 == 0u && ((never >> (a0 >> 2)) & 1u)) f0 &= ~1u;
                    if (rw.w1 == 0u && ((never >> (a1 >> 2)) & 1u)) f1 &= ~1u;
                    if (rw.w2 == 0u && ((never >> (a2 >> 2)) & 1u)) f2 &= ~1u;
                    if (rw.w3 == 0u && ((never >> (a3 >> 2)) & 1u)) f3 &= ~1u;
                }
            }
        } else {
            const f32x4 hf = HF[b];
            const uint32_t t0 = cont_bound(tb, a0, hf.x), t1 = cont_bound(tb, a1, hf.y);
            const uint32_t t2 = cont_bound(tb, a2, hf.z), t3 = cont_bound(tb, a3, hf.w);
            accept_shift(rw.w0, rw.w1, rw.w2, rw.w3, t0, t1, t2, t3, f0, f1, f2, f3);
        }
    }
    return f0 | (f1 << 8) | (f2 << 16) | (f3 << 24);
}

__host__ __device__ constexpr int bits_wg(int L) { return L == 64 ? 128 : 256; }

// BATCH: the replicas of several realizations that share L and the field
// kind, one map entry per replica (x = (realization << 16) | replica) and
// 2^lbpr workgroups each; else replicas r0.. of lat0.
// Bound by instruction issue: 496 VALU instructions per wavefront of 2048
// +-1 attempts, of them 144 64-bit products (Gaussian 630), 514 (650) with
// the neighbour words indexed by words and a three-XOR swap in the transpose.
// A sweep then and now, production path: L = 64, R = 192, +-1 23.1 -> 22.4 us,
// Gaussian 27.7 -> 25.7; L = 128, R = 64, +-1 54.0 -> 50.9.  Thresholds from
// lane registers (ds_bpermute) instead of the LDS table save another 8 per
// wavefront and were no faster, slower for few replicas (L = 64, R = 32: 10.9
// against 9.2).
template <int KIND, int ENERGY, bool BATCH>
__global__ __launch_bounds__(kBitsThreads) void sweep_bits(Lattice lat0, const Lattice *__restrict__ lats,
                                                          const uint2 *__restrict__ map, int colour, int toff,
                                                          int r0, int lbpr, int remap) {
    __shared__ __align__(16) uint32_t sthr[32];   // +-1 thresholds or the continuous-field table
    uint32_t blk = blockIdx.x;
    if (remap) {
        const uint32_t per = gridDim.x >> 3;
        blk = (blk & 7u) * per + (blk >> 3);
    }
    const uint32_t e = BATCH ? map[blk >> lbpr].x : 0u;
    const Lattice &lat = BATCH ? lats[e >> 16] : lat0;
    const uint32_t r = BATCH ? (e & 0xFFFFu) : (uint32_t)r0 + (blk >> lbpr);
    const uint32_t gb = blk & ((1u << lbpr) - 1u);
    const uint32_t W1 = (uint32_t)lat.N >> 6;            // words per colour
    const uint32_t w = gb * blockDim.x + threadIdx.x;
    const uint32_t c = (uint32_t)colour;
    const BitsAround at = bits_around(lat, w, c);
    GAS uint32_t *own = gptr(lat.bits) + ((size_t)r * 2u + c) * W1;
    GAS const uint32_t *oth = gptr(lat.bits) + ((size_t)r * 2u + (1u - c)) * W1;
    const uint32_t S = bits_word(own, at.own);
    const uint32_t W = bits_word(oth, at.own), Wn = bits_word(oth, at.x);
    const uint32_t Wyp = bits_word(oth, at.yp), Wym = bits_word(oth, at.ym);
    const uint32_t Wzp = bits_word(oth, at.zp), Wzm = bits_word(oth, at.zm);
    uint32_t F = 0;
    f32x4 HF[8];
    if (KIND == 0) {
        F = gptr(lat.fbw)[(size_t)c * W1 + w];
    } else {
        GAS const f32x4 *hf = (GAS const f32x4 *)(gptr(lat.fhw) + (size_t)c * lat.half) +
                              (size_t)(w >> 6) * 512u + (w & 63u);
#pragma unroll
        for (int b = 0; b < 8; ++b) HF[b] = hf[b * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
    const int slot = gptr(lat.r2t)[r];
    const uint32_t t = (uint32_t)(gptr(lat.ctrs)[0] + (uint64_t)toff);
    uint32_t never = 0;
    const float beta = KIND == 1 ? gptr(lat.betaf)[slot] : 0.0f;
    if (KIND == 0) {
        if (threadIdx.x < 32u) sthr[threadIdx.x] = gptr(lat.thr)[slot * 32 + threadIdx.x];
        __syncthreads();
        never = __builtin_amdgcn_readfirstlane(sthr[31]);
    } else {
        cont_table_fill(sthr, beta, lat.Jf);
        __syncthreads();
    }
    uint32_t U0, U1, U2;
    bits_planes(at.p, W, Wn, Wyp, Wym, Wzp, Wzm, U0, U1, U2);
    const uint32_t c1w = 2u * t + c, c3w = (kTagSweep << 28) | lat.rho;
    uint32_t Acls[8];
    class_offsets(U0, U1, U2, S, KIND == 0 ? F : 0u, Acls);
    const uint32_t m0v = __builtin_amdgcn_readfirstlane(kPhiloxM0);   // held in one VGPR below
    // `never` is the same for the whole workgroup: the common case (no class
    // that can never flip) runs without the per-block check
    const uint32_t flips =
        KIND == 0 && never != 0u
            ? word_flips<KIND, true>(sthr, never, Acls, HF, w, m0v, c1w, r, c3w, lat.key0, lat.key1)
            : word_flips<KIND, false>(sthr, never, Acls, HF, w, m0v, c1w, r, c3w, lat.key0, lat.key1);
    const uint32_t Snew = S ^ flips;
    if (flips) *(GAS uint32_t *)((GAS char *)own + at.own) = Snew;
    if (ENERGY) {
        // colour 1 of the last sweep before an exchange: the final state.
        // B counts each bond once through the colour-1 sites: sum of
        // s_i n_i = 2 K - 6 with K the aligned neighbours (up if s = +1,
        // 6 - up if s = -1).
        const int ksum = bits_aligned(U0, U1, U2, Snew);
        const int upsum = __popc(Snew) + __popc(W);
        int eqsum = 0;
        double fsum = 0.0;
        if (KIND == 0) {
            const uint32_t F0 = gptr(lat.fbw)[w];
            eqsum = __popc(~(Snew ^ F)) + __popc(~(W ^ F0));
        } else {
            const uint32_t w0 = w & ~63u;
            fsum = bits_field_sum(gptr(lat.fraw) + lat.half, w0, Snew) + bits_field_sum(gptr(lat.fraw), w0, W);
        }
        block_partial<KIND>(gptr(lat.part) + ((size_t)gb * lat.pstride + r) * 3, 32, ksum, upsum, eqsum, fsum);
    }
}

// Byte spins <-> bit spins (one thread per 32-site word) and the +-1 field
// words.
__global__ __launch_bounds__(256) void pack_bits_kernel(Lattice lat) {
    const uint32_t W1 = (uint32_t)lat.N >> 6;
    const uint32_t e = blockIdx.x * 256u + threadIdx.x;     // word of (replica, colour)
    if (e >= (uint32_t)lat.R * 2u * W1) return;
    const uint8_t *src = lat.spins + (size_t)e * 32u;       // [r][c][32w..] matches the byte layout
    uint32_t v = 0;
#pragma unroll
    for (uint32_t i = 0; i < 32; ++i) v |= (uint32_t)(src[i] & 1u) << bit_of_index(i);
    lat.bits[e] = v;
    if (e < 2u * W1 && lat.kind == 0) {
        uint32_t f = 0;
        const uint8_t *fb = lat.fbits + (size_t)e * 32u;
#pragma unroll
        for (uint32_t i = 0; i < 32; ++i) f |= (uint32_t)((fb[i] >> 2) & 1u) << bit_of_index(i);
        ((uint32_t *)lat.fbw)[e] = f;
    }
    if (e < 2u * W1 && lat.kind == 1) {
        // word w of colour c: its eight float4 blocks to the bit sweep's order
        const uint32_t c = e / W1, w = e - c * W1;
        const f32x4 *src4 = (const f32x4 *)(lat.fhf + (size_t)c * lat.half) + (size_t)w * 8u;
        f32x4 *dst4 = (f32x4 *)(lat.fhw + (size_t)c * lat.half) + (size_t)(w >> 6) * 512u + (w & 63u);
#pragma unroll
        for (uint32_t b = 0; b < 8; ++b) dst4[b * 64u] = src4[b];
    }
}

__global__ __launch_bounds__(256) void unpack_bits_kernel(Lattice lat) {
    const uint32_t W1 = (uint32_t)lat.N >> 6;
    const uint32_t e = blockIdx.x * 256u + threadIdx.x;
    if (e >= (uint32_t)lat.R * 2u * W1) return;
    const uint32_t v = lat.bits[e];
    uint8_t *dst = lat.spins + (size_t)e * 32u;
#pragma unroll
    for (uint32_t i = 0; i < 32; ++i) dst[i] = (uint8_t)((v >> bit_of_index(i)) & 1u);
}

// ---------------------------------------------------------------------
// Natural site order <-> the device layout (index only), for the calls that
// read or write configurations and fields: `dst` / `src` are pinned host
// memory, sites first .. first + count - 1 of the replicas' [R][N] (a
// multiple of the unit a thread takes).  Bound by the host link: the kernels
// read and write it in whole 16-byte (or 4-byte) pieces, in order.  The host
// did this site by site, with three divisions each, on a copy of the byte
// array: 3.4 ns a site and pass.
// ---------------------------------------------------------------------

// Bytes 1 / 0 to +1 / -1 (0x01 / 0xFF), four at a time.
__device__ __forceinline__ uint32_t signs_of(uint32_t b) { return 0xFFFFFFFFu ^ (b * 0xFEu); }

// Bytes a0 b0 a1 b1 and a2 b2 a3 b3.
__device__ __forceinline__ void interleave(uint32_t a, uint32_t b, uint32_t &lo, uint32_t &hi) {
    lo = __builtin_amdgcn_perm(b, a, 0x05010400u);
    hi = __builtin_amdgcn_perm(b, a, 0x07030602u);
}

// The replica and the site of natural index e, and whether the even x of its
// row belong to colour 1.
struct NaturalPlace {
    uint32_t r, i, odd_row;
};

__device__ __forceinline__ NaturalPlace natural_place(const Lattice &lat, const FastDiv &by_l, size_t e) {
    NaturalPlace p;
    p.r = (uint32_t)(e / (size_t)(uint32_t)lat.N);
    p.i = (uint32_t)(e - (size_t)p.r * (size_t)(uint32_t)lat.N);
    const uint32_t row = div_by(p.i, by_l), z = div_by(row, by_l);
    p.odd_row = (row - z * (uint32_t)lat.L + z) & 1u;
    return p;
}

template <int V, bool BITS>
__global__ __launch_bounds__(256) void spins_out_kernel(Lattice lat, FastDiv by_l, size_t first, size_t count,
                                                         int8_t *__restrict__ dst) {
    const size_t u = (size_t)V * (blockIdx.x * 256u + threadIdx.x);
    if (u >= count) return;
    const NaturalPlace p = natural_place(lat, by_l, first + u);
    const uint32_t j = p.i >> 1;
    if constexpr (V == 16) {
        // eight pairs: eight bytes (two Philox blocks' bits) of each colour
        uint32_t c[2][2];
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            if (BITS) {
                const uint32_t w = gptr((const uint32_t *)lat.bits)[((size_t)p.r * 2u + col) * ((uint32_t)lat.N >> 6) + (j >> 5)];
                const uint32_t b = (j & 31u) >> 2;
                c[col][0] = (w >> b) & 0x01010101u;
                c[col][1] = (w >> (b + 1u)) & 0x01010101u;
            } else {
                load_words<2>(gptr((const uint8_t *)lat.spins) + (size_t)p.r * lat.N + (size_t)col * lat.half, j, c[col]);
            }
        }
        u32x4 v;
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            interleave(p.odd_row ? c[1][q] : c[0][q], p.odd_row ? c[0][q] : c[1][q], o[2 * q], o[2 * q + 1]);
        v.x = signs_of(o[0]);
        v.y = signs_of(o[1]);
        v.z = signs_of(o[2]);
        v.w = signs_of(o[3]);
        *(u32x4 *)(dst + u) = v;
    } else {
        // four sites, which may lie in two rows
        uint32_t v = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const NaturalPlace s = natural_place(lat, by_l, first + u + q);
            const uint32_t col = s.odd_row ^ (s.i & 1u);
            v |= (uint32_t)gptr((const uint8_t *)lat.spins)[(size_t)s.r * lat.N + (size_t)col * lat.half + (s.i >> 1)] << (8u * q);
        }
        *(uint32_t *)(dst + u) = signs_of(v);
    }
}

// +1 / -1 bytes to 1 / 0.
__device__ __forceinline__ uint32_t ups_of(uint32_t v) { return ~(v >> 7) & 0x01010101u; }

// The bytes of even and of odd x among eight sites (lo: the first four).
__device__ __forceinline__ void deinterleave(uint32_t lo, uint32_t hi, uint32_t &even, uint32_t &odd) {
    even = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
    odd = __builtin_amdgcn_perm(hi, lo, 0x07050301u);
}

template <int V>
__global__ __launch_bounds__(256) void spins_in_kernel(Lattice lat, FastDiv by_l, size_t first, size_t count,
                                                        const int8_t *__restrict__ src) {
    const size_t u = (size_t)V * (blockIdx.x * 256u + threadIdx.x);
    if (u >= count) return;
    if constexpr (V == 16) {
        const NaturalPlace p = natural_place(lat, by_l, first + u);
        const u32x4 v = *(const u32x4 *)(src + u);
        uint32_t even[2], odd[2];
        deinterleave(ups_of(v.x), ups_of(v.y), even[0], odd[0]);
        deinterleave(ups_of(v.z), ups_of(v.w), even[1], odd[1]);
        GAS uint8_t *base = gptr(lat.spins) + (size_t)p.r * lat.N;
        store_words<2>(base + (p.odd_row ? (size_t)lat.half : 0u), p.i >> 1, even);
        store_words<2>(base + (p.odd_row ? 0u : (size_t)lat.half), p.i >> 1, odd);
    } else {
        const uint32_t v = ups_of(*(const uint32_t *)(src + u));
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const NaturalPlace s = natural_place(lat, by_l, first + u + q);
            const uint32_t col = s.odd_row ^ (s.i & 1u);
            gptr(lat.spins)[(size_t)s.r * lat.N + (size_t)col * lat.half + (s.i >> 1)] = (uint8_t)(v >> (8u * q));
        }
    }
}

// Bit storage: 64 sites of a row are one word of each colour.
__global__ __launch_bounds__(256) void bits_in_kernel(Lattice lat, FastDiv by_l, size_t first, size_t count,
                                                       const int8_t *__restrict__ src) {
    const size_t u = 64u * (size_t)(blockIdx.x * 256u + threadIdx.x);
    if (u >= count) return;
    const NaturalPlace p = natural_place(lat, by_l, first + u);
    uint32_t even = 0, odd = 0;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const u32x4 v = *(const u32x4 *)(src + u + 16u * q);
        uint32_t e, o;
        deinterleave(ups_of(v.x), ups_of(v.y), e, o);       // pairs 8q .. 8q + 3: block 2q of the word
        even |= e << (2u * q);
        odd |= o << (2u * q);
        deinterleave(ups_of(v.z), ups_of(v.w), e, o);
        even |= e << (2u * q + 1u);
        odd |= o << (2u * q + 1u);
    }
    const uint32_t W1 = (uint32_t)lat.N >> 6;
    GAS uint32_t *base = gptr(lat.bits) + (size_t)p.r * 2u * W1 + (p.i >> 6);
    base[p.odd_row ? W1 : 0u] = even;
    base[p.odd_row ? 0u : W1] = odd;
}

// Fields h_i in natural order to the sweeps' arrays, four sites a thread.
__global__ __launch_bounds__(256) void fields_in_kernel(Lattice lat, FastDiv by_l, size_t first, size_t count,
                                                         const float *__restrict__ src) {
    const size_t u = 4u * (size_t)(blockIdx.x * 256u + threadIdx.x);
    if (u >= count) return;
    const f32x4 v = *(const f32x4 *)(src + u);
    const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const NaturalPlace s = natural_place(lat, by_l, first + u + q);
        const size_t at = (size_t)(s.odd_row ^ (s.i & 1u)) * lat.half + (s.i >> 1);
        if (lat.kind == 0) {
            ((GAS uint8_t *)lat.fbits)[at] = f[q] > 0.0f ? 4 : 0;
        } else {
            ((GAS float *)lat.fraw)[at] = f[q];
            ((GAS float *)lat.fhf)[at] = (float)(lat.h * (double)f[q] - 6.0 * lat.J);
        }
    }
}

// The workgroup's writes to pinned host memory are done: the host, which polls
// the word, sees them all once it sees the 1.  A readout of a small lattice
// waits for little else than this; with a stream synchronisation instead
// (which has the device run a barrier packet and signal its end) such a call
// took 14 us, not 9.5.
// Only the waves that wrote have a fence to wait for.
__device__ __forceinline__ void signal_done(uint32_t *done, bool wrote) {
    if (wrote) __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Two arrays of a handle's counters or sums to zero in one launch, 2.7 us to
// issue (a memset call took 2.6 us for each array).
__global__ __launch_bounds__(256) void clear_kernel(uint64_t *a, uint32_t na, uint64_t *b, uint32_t nb) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < na) a[i] = 0ull;
    if (i < nb) b[i] = 0ull;
}

// Workgroups that copy one array: 16 bytes a thread and step, and few of them,
// since each ends its writes to the host for itself (13 ns).
constexpr uint32_t kCopyUnit = 4u * 256u, kCopyBlocks = 32;
__host__ __device__ inline uint32_t copy_blocks(uint32_t words) {
    const uint32_t n = (words + kCopyUnit - 1u) / kCopyUnit;
    return n < kCopyBlocks ? n : kCopyBlocks;
}

// Device arrays to pinned host memory (both 16-byte aligned), in one launch.
// Observables of R = 3000 (144 KB) 30.3 us a call with a dword a thread and 141
// workgroups for each of the three arrays, empty ones too; a staged copy took
// 17.3.
__global__ __launch_bounds__(256) void copy_out_kernel(CopyOut c) {
    uint32_t q = 0, b = blockIdx.x;
    while (b >= copy_blocks(c.words[q])) b -= copy_blocks(c.words[q++]);
    const uint32_t n = c.words[q], n4 = n / 4u, step = 256u * copy_blocks(n);
    GAS const uint32_t *src = (GAS const uint32_t *)c.src[q];
    uint32_t *dst = (uint32_t *)c.dst[q];
    uint32_t w = b * 256u + threadIdx.x;
    const bool wrote = 4u * w < n;
    for (; w < n4; w += step) ((u32x4 *)dst)[w] = ((GAS const u32x4 *)src)[w];
    if (w == n4)                            // the one thread whose turn the last 1 to 3 words are
        for (uint32_t i = 4u * n4; i < n; ++i) dst[i] = src[i];
    signal_done(c.done + blockIdx.x, wrote);
}

// ---------------------------------------------------------------------
// Energy partials (Eq. 1) of a state at rest, for the calls that read
// energies and for the sweeps that do not write partials themselves.  Every
// bond joins a colour-0 and a colour-1 site, so B = sum over colour-1 sites
// of s_i n_i counts each bond once; F and M run over both colours.  Grid
// (nblk, R); fixed reduction order.
//
// Bound: memory (one byte, or one bit, per spin, once).  L = 64, R = 192 in
// bits: 5.3 us; L = 128, R = 64: 9.8 us.  Both were unpacked to bytes first
// and then read one site per step with divisions by L (126 and 336 us).
// ---------------------------------------------------------------------

// What an energy kernel does with a workgroup's sums: the partial of block
// blockIdx.x of replica r or, where the workgroup took the whole replica
// (WHOLE), its energy and magnetisation for the reader: one launch less (a
// call at L = 16, R = 32 that took 18 us takes 12 with it and the polled end;
// L = 32, R = 64 18.9 and 15.5).
constexpr int kWholeEnergyThreads = 1024;

template <int KIND, bool WHOLE>
__device__ __forceinline__ void energy_sums(const Lattice &lat, const Readout &out, uint32_t r, int nsite, int ksum, int upsum,
                                            int eqsum, double fsum) {
    if constexpr (!WHOLE) {
        block_partial<KIND>(gptr(lat.part) + ((size_t)blockIdx.x * lat.pstride + r) * 3, nsite, ksum, upsum, eqsum, fsum);
    } else {
        __shared__ double tot[3];
        const int slot = gptr(lat.r2t)[r];
        block_partial<KIND>(tot, nsite, ksum, upsum, eqsum, fsum);
        __syncthreads();
        if (threadIdx.x == 0) {
            if (out.B) out.B[r] = (int64_t)tot[0];
            if (out.F) out.F[r] = tot[1];
            if (out.M) out.M[r] = (int64_t)tot[2];
            if (out.E_slot) out.E_slot[slot] = energy_of(lat, tot[0], tot[1]);
            if (out.M_slot) out.M_slot[slot] = (int64_t)tot[2];
            __hip_atomic_store(out.done + r, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Rows of whole dwords (L a multiple of 8 NW): chunks as in the sweeps.
template <int KIND, int NW, bool WHOLE>
__global__ __launch_bounds__(WHOLE ? kWholeEnergyThreads : 256) void energy_rows(Lattice lat, FastDiv by_row, FastDiv by_l,
                                                                                 Readout out) {
    const uint32_t r = blockIdx.y, L = (uint32_t)lat.L, half = (uint32_t)lat.half;
    GAS const uint8_t *s0 = gptr((const uint8_t *)lat.spins) + (size_t)r * lat.N;
    GAS const uint8_t *s1 = s0 + half;
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fraw = gptr(lat.fraw);
    int ksum = 0, upsum = 0, eqsum = 0, n = 0;
    double fsum = 0.0;
    for (uint32_t j0 = 4u * NW * (blockIdx.x * blockDim.x + threadIdx.x); j0 < half;
         j0 += 4u * NW * blockDim.x * gridDim.x, ++n) {
        const Chunk c = row_chunk<NW>(j0, 1u, L, by_row, by_l);
        uint32_t S1[NW], W[NW], U[NW], F1[NW];
        load_words<NW>(s1, j0, S1);
        if (KIND == 0) load_words<NW>(fbits + half, j0, F1);
        neighbour_counts<NW>(s0, j0, c, W, U);
        chunk_energy<KIND, NW>(lat, S1, W, U, F1, fbits, fraw + half, fraw, j0, ksum, upsum, eqsum, fsum);
    }
    energy_sums<KIND, WHOLE>(lat, out, r, 4 * NW * n, ksum, upsum, eqsum, fsum);
}

// Any even L: four consecutive pairs per step, which may lie in two rows.
template <int KIND, bool WHOLE>
__global__ __launch_bounds__(WHOLE ? kWholeEnergyThreads : 256) void energy_sites(Lattice lat, FastDiv by_row, FastDiv by_l,
                                                                                  Readout out) {
    const uint32_t r = blockIdx.y, half = (uint32_t)lat.half;
    GAS const uint8_t *s0 = gptr((const uint8_t *)lat.spins) + (size_t)r * lat.N;
    GAS const uint8_t *s1 = s0 + half;
    GAS const uint8_t *fbits = gptr(lat.fbits);
    GAS const float *fraw = gptr(lat.fraw);
    int ksum = 0, upsum = 0, eqsum = 0, n = 0;
    double fsum = 0.0;
    for (uint32_t j0 = 4u * (blockIdx.x * blockDim.x + threadIdx.x); j0 < half; j0 += 4u * blockDim.x * gridDim.x, ++n) {
        uint32_t S1[1], W[1], U[1], F1[1];
        load_words<1>(s1, j0, S1);
        load_words<1>(s0, j0, W);
        if (KIND == 0) load_words<1>(fbits + half, j0, F1);
        U[0] = site_counts(s0, j0, W[0], 1u, (uint32_t)lat.L, by_row, by_l);
        chunk_energy<KIND, 1>(lat, S1, W, U, F1, fbits, fraw + half, fraw, j0, ksum, upsum, eqsum, fsum);
    }
    energy_sums<KIND, WHOLE>(lat, out, r, 4 * n, ksum, upsum, eqsum, fsum);
}

// Bit storage: a thread takes whole words of colour 1, as the bit sweep's
// energy pass does (W1 is a multiple of the threads of the grid's row).
template <int KIND>
__global__ __launch_bounds__(256) void energy_bits(Lattice lat) {
    const uint32_t r = blockIdx.y, W1 = (uint32_t)lat.N >> 6;
    GAS const uint32_t *b0 = gptr((const uint32_t *)lat.bits) + (size_t)r * 2u * W1, *b1 = b0 + W1;
    int ksum = 0, upsum = 0, eqsum = 0, n = 0;
    double fsum = 0.0;
    for (uint32_t w = blockIdx.x * 256u + threadIdx.x; w < W1; w += 256u * gridDim.x, ++n) {
        const BitsAround at = bits_around(lat, w, 1u);
        const uint32_t S = bits_word(b1, at.own), W = bits_word(b0, at.own);
        uint32_t U0, U1, U2;
        bits_planes(at.p, W, bits_word(b0, at.x), bits_word(b0, at.yp), bits_word(b0, at.ym), bits_word(b0, at.zp),
                    bits_word(b0, at.zm), U0, U1, U2);
        ksum += bits_aligned(U0, U1, U2, S);
        upsum += __popc(S) + __popc(W);
        if (KIND == 0) {
            eqsum += __popc(~(S ^ bits_word(gptr(lat.fbw) + W1, at.own))) + __popc(~(W ^ bits_word(gptr(lat.fbw), at.own)));
        } else {
            const uint32_t w0 = w & ~63u;
            fsum += bits_field_sum(gptr(lat.fraw) + lat.half, w0, S) + bits_field_sum(gptr(lat.fraw), w0, W);
        }
    }
    block_partial<KIND>(gptr(lat.part) + ((size_t)blockIdx.x * lat.pstride + r) * 3, 32 * n, ksum, upsum, eqsum, fsum);
}

// ---------------------------------------------------------------------
// Exchange step k (Eq. 2): pairs (p, p+1) with p = k mod 2; temperatures
// move through t2r / r2t (Sec. 3.3).  One workgroup of kExchangeThreads.
// ---------------------------------------------------------------------
// The ranges of block partials replica_totals adds: G ranges of `per` blocks.
__host__ __device__ inline void partial_ranges(int R, int nblk, int *groups, int *per) {
    int G = 1;
    while (2 * G <= nblk && 2 * G <= 64 && (long long)R * 2 * G <= kExchangeThreads) G *= 2;
    *groups = G;
    *per = (nblk + G - 1) / G;
}

// Energy and magnetisation of every replica from its partials (B, F, M per
// block, block-major).  Thread (g, r) sums blocks [g per, min((g+1) per,
// nblk)) of replica r in order -- consecutive threads take consecutive
// replicas, so every load is coalesced -- issuing up to 8 blocks' loads
// before it adds any, so the range costs a few memory round trips rather than
// one per block; then one thread per replica adds its G range sums in order.
// nblk need not be a power of two (the generic kernel's is not).  The order
// is fixed for a given launch shape and replica count, so FP64 totals are
// reproducible.  Writes E and Mr, and B, F, M when asked (observables).
template <int B>
__device__ __forceinline__ void sum_range(GAS const double *pp, size_t qstride, int q_end, double &b, double &f,
                                          double &m) {
    for (int q0 = 0; q0 < q_end; q0 += B) {
        // loads past the range re-read its last block (always in bounds, no
        // branch between the loads); their adds are skipped
        double vb[B], vf[B], vm[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            GAS const double *pq = pp + (size_t)min(q0 + j, q_end - 1) * qstride;
            vb[j] = pq[0];
            vf[j] = pq[1];
            vm[j] = pq[2];
        }
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const bool in = q0 + j < q_end;
            b = in ? b + vb[j] : b;
            f = in ? f + vf[j] : f;
            m = in ? m + vm[j] : m;
        }
    }
}

__device__ __forceinline__ void replica_totals(const Lattice &lat, const double *part, const Readout &out = Readout{},
                                               double *sE = nullptr, double *sM = nullptr) {
    __shared__ double red[kExchangeThreads * 3];
    const int R = lat.R, nblk = lat.nblk;
    int G, per;
    partial_ranges(R, nblk, &G, &per);
    const int tile = kExchangeThreads / G;
    const int g = (int)threadIdx.x / tile, rl = (int)threadIdx.x % tile;
    const int q_end = min(per, nblk - g * per);   // blocks in this thread's range (may be <= 0)
    const size_t qstride = (size_t)lat.pstride * 3;
    for (int r0 = 0; r0 < R; r0 += tile) {
        const int r = r0 + rl;
        double b = 0.0, f = 0.0, m = 0.0;
        if (r < R) {
            GAS const double *pp = gptr(part) + ((size_t)g * per * lat.pstride + r) * 3;
            if (per == 1)       // the batch width follows the range (uniform per block)
                sum_range<1>(pp, qstride, q_end, b, f, m);
            else if (per == 2)
                sum_range<2>(pp, qstride, q_end, b, f, m);
            else if (per <= 4)
                sum_range<4>(pp, qstride, q_end, b, f, m);
            else
                sum_range<8>(pp, qstride, q_end, b, f, m);
        }
        red[3 * threadIdx.x + 0] = b;
        red[3 * threadIdx.x + 1] = f;
        red[3 * threadIdx.x + 2] = m;
        __syncthreads();
        if ((int)threadIdx.x < tile && r0 + (int)threadIdx.x < R) {
            double B = red[3 * threadIdx.x + 0], F = red[3 * threadIdx.x + 1], M = red[3 * threadIdx.x + 2];
            for (int q = 1; q < G; ++q) {
                const double *rr = red + 3 * (q * tile + threadIdx.x);
                B += rr[0];
                F += rr[1];
                M += rr[2];
            }
            const int rt = r0 + (int)threadIdx.x;
            const double E = energy_of(lat, B, F);
            lat.E[rt] = E;
            lat.Mr[rt] = M;
            if (sE) {
                sE[rt] = E;
                sM[rt] = M;
            }
            if (out.B) out.B[rt] = (int64_t)B;
            if (out.F) out.F[rt] = F;
            if (out.M) out.M[rt] = (int64_t)M;
            if (out.E_slot || out.M_slot) {
                const int slot = gptr(lat.r2t)[rt];
                if (out.E_slot) out.E_slot[slot] = E;
                if (out.M_slot) out.M_slot[slot] = (int64_t)M;
            }
        }
        __syncthreads();
    }
}

// Totals per replica id for the calls that read energies.  The sums are the
// exchange step's, but over partials of their own (energy_blocks): with
// continuous fields the energies read and those of a step may differ in the last
// bits, with +-1 fields both are exact.
__global__ __launch_bounds__(kExchangeThreads) void reduce_kernel(Lattice lat, Readout out) {
    replica_totals(lat, lat.part, out);
    signal_done(out.done, (int)threadIdx.x < lat.R);
}

// One exchange step per workgroup (one realization each).  Up to
// kExchangeThreads replicas the step runs out of LDS: the permutation, the
// inverse temperatures, the slot's observable sums and the pair counters are
// loaded together with the energy partials, so the whole step costs about
// two memory round trips; more replicas take the same steps through global
// memory.
__global__ __launch_bounds__(kExchangeThreads) void exchange_kernel(const Lattice *__restrict__ lats, int tadv, StepIn in) {
    __shared__ double sE[kExchangeThreads], sM[kExchangeThreads];
    __shared__ int32_t st2r[kExchangeThreads];
    const Lattice &lat = lats[blockIdx.x];
    const bool pending = in.part != nullptr;      // then R <= kExchangeThreads
    const uint64_t k = pending ? in.k : lat.ctrs[1];
    const int R = lat.R, t = (int)threadIdx.x;
    if (R <= kExchangeThreads) {
        // inputs that do not depend on the energies, fetched first
        const bool mine = t < R;
        const int tc = mine ? t : 0;
        // (global-typed loads: flat ones would also hold up the scalar waits)
        const int32_t my_t2r = gptr(pending ? in.t2r : (const int32_t *)lat.t2r)[tc];
        GAS const double *beta = gptr(lat.beta);
        const double my_beta = beta[tc], my_beta1 = beta[min(tc + 1, R - 1)];
        const bool pair = t + 1 < R && (t & 1) == (int)(k & 1);
        const int pc = min(tc, max(R - 2, 0));
        const uint64_t my_att = gptr(lat.att)[pc], my_acc = gptr(lat.acc)[pc];
        double o[6];
        GAS const double *orow = gptr(lat.obs) + 6 * (size_t)tc;
#pragma unroll
        for (int q = 0; q < 6; ++q) o[q] = orow[q];
        replica_totals(lat, pending ? in.part : lat.part, Readout{}, sE, sM);
        if (mine) st2r[t] = my_t2r;
        __syncthreads();
        // pairs (p, p+1) with p = k mod 2: thread p decides its pair; the
        // pairs are disjoint, so every slot is written by at most one thread
        if (pair) {
            const int a = st2r[t], b = st2r[t + 1];
            const double delta = (my_beta1 - my_beta) * (sE[b] - sE[a]);
            lat.att[t] = my_att + 1;
            if (exchange_accept(lat, t, k, delta)) {
                lat.acc[t] = my_acc + 1;
                st2r[t] = b;
                st2r[t + 1] = a;
                lat.t2r[t] = b;
                lat.t2r[t + 1] = a;
                lat.r2t[a] = t + 1;
                lat.r2t[b] = t;
            }
        }
        __syncthreads();
        // one measurement per exchange step (Sec. 7), by temperature slot
        if (mine) {
            const int a = st2r[t];
            if (pending) {                        // the permutation may come from its other copy
                lat.t2r[t] = a;
                lat.r2t[a] = t;
            }
            const double e = sE[a], m = sM[a], m2 = m * m;
            double *op = lat.obs + 6 * (size_t)t;
            op[0] = o[0] + 1.0;
            op[1] = o[1] + e;
            op[2] = o[2] + e * e;
            op[3] = o[3] + fabs(m);
            op[4] = o[4] + m2;
            op[5] = o[5] + m2 * m2;
        }
    } else {
        replica_totals(lat, lat.part);
        __syncthreads();
        for (int p = (int)(k & 1) + 2 * t; p + 1 < R; p += 2 * kExchangeThreads) {
            const int a = lat.t2r[p], b = lat.t2r[p + 1];
            const double delta = (lat.beta[p + 1] - lat.beta[p]) * (lat.E[b] - lat.E[a]);
            lat.att[p] += 1;
            if (exchange_accept(lat, p, k, delta)) {
                lat.t2r[p] = b;
                lat.t2r[p + 1] = a;
                lat.r2t[a] = p + 1;
                lat.r2t[b] = p;
                lat.acc[p] += 1;
            }
        }
        __syncthreads();
        for (int q = t; q < R; q += kExchangeThreads) {
            const int a = lat.t2r[q];
            const double e = lat.E[a], m = lat.Mr[a], m2 = m * m;
            double *o = lat.obs + 6 * (size_t)q;
            o[0] += 1.0;
            o[1] += e;
            o[2] += e * e;
            o[3] += fabs(m);
            o[4] += m2;
            o[5] += m2 * m2;
        }
    }
    if (threadIdx.x == 0) {
        lat.ctrs[0] += (uint64_t)tadv;
        lat.ctrs[1] = k + 1;
    }
}

__global__ void advance_kernel(uint64_t *ctrs, int tadv) {
    if (threadIdx.x == 0 && blockIdx.x == 0) ctrs[0] += (uint64_t)tadv;
}

}  // namespace

bool shape_valid(int L, int mode, int nw, int wg) {
    const bool pow2 = L >= 8 && (L & (L - 1)) == 0;
    if (!pow2) return mode == 0 && nw == 0 && wg == 0;      // generic kernel, fixed shape
    if (mode >= 2 && mode <= 4) {
        // slabs: nw = slabs per replica, mode - 1 sweeps per launch
        if (L != 16 && L != 32) return false;
        if (nw != 2 && nw != 4 && nw != 8) return false;
        if (L / nw < 2) return false;
        if (L / nw + 4 * slab_sweeps_per_launch(mode) > L) return false;   // the box must not wrap onto itself
        if (slab_lds_bytes(L, mode, nw) > 65536) return false;
        if (wg != 128 && wg != 256 && wg != 512 && wg != 1024) return false;
        return slab_positions_per_thread(L, mode, nw, wg) <= 2;
    }
    if (nw != 1 && nw != 2 && nw != 4 && nw != 8) return false;
    if (4 * nw > L / 2) return false;                        // a chunk lies inside one row
    const long long chunks = (long long)L * L * L / 8 / nw;  // per colour and replica
    if (mode == 0) {
        if (wg != 64 && wg != 128 && wg != 256) return false;
        return chunks % wg == 0 || chunks < wg;
    }
    if (mode == 1) {
        if (L > 32 || nw > 4) return false;                  // one replica must fit in LDS
        return wg == 64 || wg == 128 || wg == 256 || wg == 512 || wg == 1024;
    }
    return false;
}

int blocks_per_replica(int L, int mode, int nw, int wg) {
    const bool pow2 = L >= 8 && (L & (L - 1)) == 0;
    if (generic_resident(L)) return 1;
    if (!pow2) {
        const long long G = (long long)L * L * L / 8;
        long long nb = (G + 255) / 256;
        if (nb > 64) nb = 64;
        return (int)(nb < 1 ? 1 : nb);
    }
    if (mode == 1) return 1;
    if (mode >= 2) return nw;                                // one partial per slab
    const long long chunks = (long long)L * L * L / 8 / nw;
    if (chunks < wg) return 1;
    const long long nb = chunks / wg;
    return nb > kMaxFusedBlocks ? 64 : (int)nb;
}

int stream_blocks_per_replica(int L, int nw, int wg) {
    const long long chunks = (long long)L * L * L / 8 / nw;
    const long long w = chunks < wg ? chunks : wg;
    return (int)(chunks / w);
}

bool fused_energy(const Lattice &lat) {
    if (lat.log2L < 3) return generic_resident(lat.L);
    if (lat.mode >= 1) return true;
    const long long chunks = (long long)lat.N / 8 / lat.nw;
    return chunks <= (long long)lat.wg * kMaxFusedBlocks;
}

hipError_t launch_init(const Lattice &lat, int r0, int r1, hipStream_t s) {
    if (r1 <= r0) return hipSuccess;
    const int G = lat.N >> 2;
    dim3 grid((G + 255) / 256, r1 - r0);
    hipLaunchKernelGGL(init_kernel, grid, dim3(256), 0, s, lat, r0);
    return hipGetLastError();
}

template <int KIND, int ENERGY, bool BATCH>
static void launch_pow2(const Launch &ln, const Lattice &lat0, int colour, int toff, hipStream_t s) {
    const int remap = (ln.nblocks % 8 == 0) ? 1 : 0;
    // a replica smaller than one workgroup gets a workgroup of its size:
    // the block map counts one block per replica then, and every thread of
    // a block must own a chunk of that replica
    const long long chunks = (long long)ln.L * ln.L * ln.L / 8 / ln.nw;
    const int wg = chunks < ln.wg ? (int)chunks : ln.wg;
    const int lwpr = __builtin_ctzll((unsigned long long)(chunks / wg));   // a power of two
    const dim3 grid(ln.nblocks), block(wg);
    if (ln.nw == 8)
        hipLaunchKernelGGL((sweep_pow2<KIND, 8, ENERGY, BATCH>), grid, block, 0, s, lat0, ln.lats, ln.map, colour,
                           toff, remap, lwpr, ln.r0);
    else if (ln.nw == 4)
        hipLaunchKernelGGL((sweep_pow2<KIND, 4, ENERGY, BATCH>), grid, block, 0, s, lat0, ln.lats, ln.map, colour,
                           toff, remap, lwpr, ln.r0);
    else if (ln.nw == 2)
        hipLaunchKernelGGL((sweep_pow2<KIND, 2, ENERGY, BATCH>), grid, block, 0, s, lat0, ln.lats, ln.map, colour,
                           toff, remap, lwpr, ln.r0);
    else
        hipLaunchKernelGGL((sweep_pow2<KIND, 1, ENERGY, BATCH>), grid, block, 0, s, lat0, ln.lats, ln.map, colour,
                           toff, remap, lwpr, ln.r0);
}

// Workgroups of `kernel` one CU holds at once (0 if unknown), cached in
// `slot` (-1: not asked yet), and the current device's CU count.
static int resident_blocks_per_cu(std::atomic<int> &slot, const void *kernel, int wg, size_t lds) {
    int n = slot.load(std::memory_order_relaxed);
    if (n >= 0) return n;
    n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, wg, lds) != hipSuccess) {
        (void)hipGetLastError();
        n = 0;
    }
    slot.store(n, std::memory_order_relaxed);
    return n;
}

static int device_cus() {
    static std::atomic<int> cache[16] = {};
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (dev >= 0 && dev < 16 && (n = cache[dev].load(std::memory_order_relaxed)) > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (dev >= 0 && dev < 16) cache[dev].store(n, std::memory_order_relaxed);
    return n;
}

template <int KIND, int NW, bool BATCH>
static void launch_res_nw(const Launch &ln, const Lattice &lat0, const StepIn &in, int nsweep, int energy, hipStream_t s) {
    const size_t lds = (size_t)ln.L * ln.L * ln.L;
    const dim3 grid(ln.nblocks), block(ln.wg);
    // one chunk per thread and colour: the register-field form, unless its
    // extra registers would leave fewer workgroups per CU than the plain
    // form while there are more workgroups than the device holds at once
    bool one = (long long)ln.L * ln.L * ln.L / 8 / NW == ln.wg;
    if (one) {
        // per instantiation, (L, wg) is fixed by chunks == wg up to the two
        // L of NW = 1; index the cache by L
        static std::atomic<int> occ[2][6] = {{-1, -1, -1, -1, -1, -1}, {-1, -1, -1, -1, -1, -1}};
        const int li = ln.L == 8 ? 0 : (ln.L == 16 ? 1 : (ln.L == 32 ? 2 : 3));
        const int b1 = resident_blocks_per_cu(occ[1][li], (const void *)sweep_resident<KIND, NW, BATCH, true, false>,
                                              ln.wg, lds);
        const int b0 = resident_blocks_per_cu(occ[0][li], (const void *)sweep_resident<KIND, NW, BATCH, false, false>,
                                              ln.wg, lds);
        const long long cus = device_cus();
        if (b1 < b0 && (long long)ln.nblocks > cus * b1) one = false;
    }
    const bool step = !BATCH && in.part != nullptr;
    if (!BATCH && NW == 1 && ln.L == 8 && ln.wg == 64 && ln.nblocks <= kAheadMaxReplicas) {
        if (step)
            hipLaunchKernelGGL((sweep_resident_ahead<KIND, true>), grid, dim3(256), 0, s, lat0, in, nsweep, energy);
        else
            hipLaunchKernelGGL((sweep_resident_ahead<KIND, false>), grid, dim3(256), 0, s, lat0, in, nsweep, energy);
        return;
    }
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, lat0, ln.lats, ln.map, in, nsweep, energy);
    };
    if (one)
        step ? go(sweep_resident<KIND, NW, BATCH, true, !BATCH>) : go(sweep_resident<KIND, NW, BATCH, true, false>);
    else
        step ? go(sweep_resident<KIND, NW, BATCH, false, !BATCH>) : go(sweep_resident<KIND, NW, BATCH, false, false>);
}

template <int KIND, bool BATCH>
static void launch_res(const Launch &ln, const Lattice &lat0, const StepIn &in, int nsweep, int energy, hipStream_t s) {
    if (ln.nw == 4)
        launch_res_nw<KIND, 4, BATCH>(ln, lat0, in, nsweep, energy, s);
    else if (ln.nw == 2)
        launch_res_nw<KIND, 2, BATCH>(ln, lat0, in, nsweep, energy, s);
    else
        launch_res_nw<KIND, 1, BATCH>(ln, lat0, in, nsweep, energy, s);
}

hipError_t launch_stream_sweep(const Launch &ln, int colour, int toff, int energy, hipStream_t s) {
    if (ln.nblocks == 0) return hipSuccess;
    const bool e = energy && colour == 1;
    const bool b = ln.single == nullptr;
    const Lattice lat0 = b ? Lattice{} : *ln.single;
    if (ln.kind == 0) {
        if (e) b ? launch_pow2<0, 1, true>(ln, lat0, colour, toff, s) : launch_pow2<0, 1, false>(ln, lat0, colour, toff, s);
        else b ? launch_pow2<0, 0, true>(ln, lat0, colour, toff, s) : launch_pow2<0, 0, false>(ln, lat0, colour, toff, s);
    } else {
        if (e) b ? launch_pow2<1, 1, true>(ln, lat0, colour, toff, s) : launch_pow2<1, 1, false>(ln, lat0, colour, toff, s);
        else b ? launch_pow2<1, 0, true>(ln, lat0, colour, toff, s) : launch_pow2<1, 0, false>(ln, lat0, colour, toff, s);
    }
    return hipGetLastError();
}

hipError_t launch_resident(const Launch &ln, const StepIn &in, int nsweep, int energy, hipStream_t s) {
    if (ln.nblocks == 0) return hipSuccess;
    const bool b = ln.single == nullptr;
    const Lattice lat0 = b ? Lattice{} : *ln.single;
    if (ln.kind == 0) b ? launch_res<0, true>(ln, lat0, in, nsweep, energy, s) : launch_res<0, false>(ln, lat0, in, nsweep, energy, s);
    else b ? launch_res<1, true>(ln, lat0, in, nsweep, energy, s) : launch_res<1, false>(ln, lat0, in, nsweep, energy, s);
    return hipGetLastError();
}

bool generic_resident(int L) { return L <= kGenericResidentMaxL && (L % 4 == 2 || L == 4); }

template <int KIND>
static void launch_generic_kind(const Lattice &lat, const StepIn &in, int colour, int toff, int nsweep, int energy,
                                hipStream_t s) {
    const FastDiv by_row = fast_div((uint32_t)lat.L / 2u), by_l = fast_div((uint32_t)lat.L);
    const int G = lat.half >> 2;
    const unsigned nb = (unsigned)((G + 255) / 256);
    if (nsweep > 0) {
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)lat.R), dim3((unsigned)std::min(1024, (G + 63) / 64 * 64)), (size_t)lat.N,
                               s, lat, in, by_row, by_l, nsweep, energy);
        };
        in.part ? go(sweep_generic_resident<KIND, true>) : go(sweep_generic_resident<KIND, false>);
        return;
    }
    // a launch has fewer than 2^32 threads in a row: R L^3 from 2^35 on takes several
    const int most = (int)(0xFFFFFFFFu / 256u / nb);
    for (int r0 = 0; r0 < lat.R; r0 += most) {
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(nb * (unsigned)std::min(most, lat.R - r0)), dim3(256), 0, s, lat, by_row, by_l,
                               fast_div(nb), r0, colour, toff);
        };
        lat.L % 8 == 0 ? go(sweep_generic<KIND, true>) : go(sweep_generic<KIND, false>);
    }
}

static hipError_t launch_generic(const Lattice &lat, const StepIn &in, int colour, int toff, int nsweep, int energy,
                                 hipStream_t s) {
    if (lat.kind == 0)
        launch_generic_kind<0>(lat, in, colour, toff, nsweep, energy, s);
    else
        launch_generic_kind<1>(lat, in, colour, toff, nsweep, energy, s);
    return hipGetLastError();
}

hipError_t launch_generic_sweep(const Lattice &lat, int colour, int toff, hipStream_t s) {
    return launch_generic(lat, StepIn{}, colour, toff, 0, 0, s);
}

hipError_t launch_generic_resident(const Lattice &lat, const StepIn &in, int nsweep, int energy, hipStream_t s) {
    if (nsweep < 1) return hipSuccess;
    return launch_generic(lat, in, 0, 0, nsweep, energy, s);
}

size_t box_lds_bytes(int L, int planes) { return (size_t)planes * (size_t)L * (size_t)L; }   // both colours

// Microseconds of a sweep, from measurements on gfx950 at L = 20 .. 96 and
// R = 8 .. 300 (within about 15 % of them): a launch of boxes costs 5 us, the
// planes staged and written back at 16 KB/us a CU, and 0.18 us for every
// block of a wave and SIMD (0.25 where neighbours are gathered as bytes); a
// half-sweep launch 3.3 us and 0.49 (1.4) us per 2^20 sites of all replicas.
static double box_cost(int L, long long R, int np, int K) {
    const long long bpp = (long long)L * L / 8, slabs = (L + np - 1) / np;
    const bool whole = slabs == 1;
    const long long P = whole ? L : np + 4 * K, G = std::min(1024 / bpp, whole ? P : P - 2);
    const double wgs = std::ceil((double)(R * slabs) / 256.0);         // a CU's workgroups
    const double waves = std::ceil(wgs * (double)((G * bpp + 63) / 64) / 4.0);
    double steps = 0.0;
    for (int st = 0; st < 2 * K; ++st) {
        const long long active = whole ? L : P - 2 - 2 * st;
        steps += (double)((active + G - 1) / G);
    }
    return (5.0 + (double)(P + np) * (double)(L * L) * wgs / 16000.0 + (L % 8 ? 0.25 : 0.18) * waves * steps) / K;
}

static double half_sweeps_cost(int L, long long R) {
    return 2.0 * (3.3 + (L % 8 ? 1.4 : 0.49) * (double)R * L * L * L / 1048576.0);
}

BoxPlan box_plan(int L, int R) {
    BoxPlan best = {0, 0};
    if (L % 4 != 0 || L < 12 || L > kBoxMaxL || (L & (L - 1)) == 0) return best;
    double cost = half_sweeps_cost(L, R);
    for (int np = 1; np <= L; ++np) {
        const bool whole = np == L;
        if ((L + np - 1) / np > kMaxBoxSlabs) continue;
        // a whole replica runs any number of sweeps in a launch: as many as
        // an exchange interval has; ten stand for it here
        for (int K = whole ? 10 : 1; K <= (whole ? 10 : 8); ++K) {
            if (!whole && 4 * K >= L) break;
            if (box_lds_bytes(L, whole ? L : np + 4 * K) > 65536) break;
            const double c = box_cost(L, R, np, K);
            if (c < cost) {
                best = {np, K};
                cost = c;
            }
        }
    }
    return best;
}

template <int KIND, bool ROWS>
static void launch_box_form(const Lattice &lat, const StepIn &in, const uint8_t *src, uint8_t *dst, int np, int nsweep,
                            int toff, int energy, hipStream_t s) {
    const uint32_t L = (uint32_t)lat.L, slabs = (L + (uint32_t)np - 1u) / (uint32_t)np, bpp = L * L / 8u;
    const bool whole = slabs == 1u;
    const uint32_t active = whole ? L : (uint32_t)(np + 4 * nsweep - 2);     // planes of the largest half-sweep
    const dim3 grid((unsigned)lat.R * slabs), block(bpp * std::min(1024u / bpp, active));
    const FastDiv by_row = fast_div(L / 2u), by_plane = fast_div(bpp), by_slab = fast_div(slabs);
    const size_t lds = box_lds_bytes(lat.L, whole ? lat.L : np + 4 * nsweep);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, lat, in, by_row, by_plane, by_slab, src, dst, np, nsweep, toff, energy);
    };
    if (whole)
        in.part ? go(sweep_box<KIND, ROWS, true, true>) : go(sweep_box<KIND, ROWS, true, false>);
    else
        in.part ? go(sweep_box<KIND, ROWS, false, true>) : go(sweep_box<KIND, ROWS, false, false>);
}

hipError_t launch_box(const Lattice &lat, const StepIn &in, const uint8_t *src, uint8_t *dst, const BoxPlan &plan,
                      int nsweep, int toff, int energy, hipStream_t s) {
    const int np = plan.planes;
    const bool whole = np >= lat.L;
    if (np < 1 || nsweep < 1 || lat.L % 4 != 0 || lat.L > kBoxMaxL) return hipErrorInvalidValue;
    if (!whole && (4 * nsweep >= lat.L || src == dst)) return hipErrorInvalidValue;
    if (box_lds_bytes(lat.L, whole ? lat.L : np + 4 * nsweep) > 65536) return hipErrorInvalidValue;
    const bool rows = lat.L % 8 == 0;
    if (lat.kind == 0)
        rows ? launch_box_form<0, true>(lat, in, src, dst, np, nsweep, toff, energy, s)
             : launch_box_form<0, false>(lat, in, src, dst, np, nsweep, toff, energy, s);
    else
        rows ? launch_box_form<1, true>(lat, in, src, dst, np, nsweep, toff, energy, s)
             : launch_box_form<1, false>(lat, in, src, dst, np, nsweep, toff, energy, s);
    return hipGetLastError();
}

int slab_sweeps_per_launch(int mode) { return mode >= 2 ? mode - 1 : 0; }

size_t slab_lds_bytes(int L, int mode, int nslab) {
    const int P = L / nslab + 4 * slab_sweeps_per_launch(mode);
    return (size_t)P * (size_t)L * L;          // both colours: L^2 / 2 bytes each
}

int slab_positions_per_thread(int L, int mode, int nslab, int wg) {
    const long long items = (long long)(L / nslab + 4 * slab_sweeps_per_launch(mode)) * L * L / 16;
    return (int)((items + wg - 1) / wg);
}

template <int KIND>
static void launch_slab_kind(const Lattice &lat, const StepIn &in, const uint8_t *src, uint8_t *dst, int np, int nslab, int wg,
                             size_t lds, int nsweep, int toff, int energy, hipStream_t s) {
    const dim3 grid((unsigned)(lat.R * nslab)), block((unsigned)wg);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, lat, in, src, dst, nslab, nsweep, toff, energy);
    };
    if (np == 1)
        in.part ? go(sweep_slabs<KIND, 1, true>) : go(sweep_slabs<KIND, 1, false>);
    else
        in.part ? go(sweep_slabs<KIND, 2, true>) : go(sweep_slabs<KIND, 2, false>);
}

hipError_t launch_slab_sweep(const Lattice &lat, const StepIn &in, const uint8_t *src, uint8_t *dst, int mode, int nslab,
                             int wg, int nsweep, int toff, int energy, hipStream_t s) {
    const size_t lds = slab_lds_bytes(lat.L, mode, nslab);
    const int np = slab_positions_per_thread(lat.L, mode, nslab, wg);
    if (np < 1 || np > 2 || nsweep < 1 || nsweep > slab_sweeps_per_launch(mode)) return hipErrorInvalidValue;
    if (lat.kind == 0)
        launch_slab_kind<0>(lat, in, src, dst, np, nslab, wg, lds, nsweep, toff, energy, s);
    else
        launch_slab_kind<1>(lat, in, src, dst, np, nslab, wg, lds, nsweep, toff, energy, s);
    return hipGetLastError();
}

bool tile_shape_valid(int L, const TileShape &ts) {
    if (L < 16 || L > 1024 || (L & (L - 1))) return false;
    const int t[3] = {ts.tx, ts.ty, ts.tz};
    for (int d = 0; d < 3; ++d)
        if (t[d] < 1 || L % t[d] != 0 || ((L / t[d]) & 1)) return false;
    if (ts.tx % 8 != 0) return false;
    const long long threads = (long long)(ts.tx / 8) * ts.ty * ts.tz;
    if (threads < 64 || threads > 1024 || threads % 64 != 0) return false;
    if (tile_lds_bytes(ts) > 65536) return false;
    return ts.hits >= 1 && ts.hits <= 65536;
}

size_t tile_lds_bytes(const TileShape &ts) {
    return 2u * (size_t)(4 * (ts.tx / 8 + 2)) * (size_t)(ts.ty + 2) * (size_t)(ts.tz + 2);
}

hipError_t launch_tile_sweep(const Lattice &lat, const TileShape &ts, int coarse, int toff, hipStream_t s) {
    const int ntile = (lat.L / ts.tx) * (lat.L / ts.ty) * (lat.L / ts.tz) / 2;
    const dim3 grid((unsigned)(ntile * lat.R)), block((unsigned)((ts.tx / 8) * ts.ty * ts.tz));
    if (lat.kind == 0)
        hipLaunchKernelGGL(sweep_tiles<0>, grid, block, tile_lds_bytes(ts), s, lat, ts, coarse, toff);
    else
        hipLaunchKernelGGL(sweep_tiles<1>, grid, block, tile_lds_bytes(ts), s, lat, ts, coarse, toff);
    return hipGetLastError();
}

bool bits_valid(int L) { return L == 64 || L == 128 || L == 256; }

int bits_blocks_per_replica(int L) { return (int)(((long long)L * L * L / 64) / bits_wg(L)); }

namespace {
template <bool BATCH>
void launch_bits(const Lattice &lat0, const Lattice *lats, const uint2 *map, int L, int kind, int r0, int nrep,
                 int colour, int toff, int energy, hipStream_t s) {
    const int bpr = bits_blocks_per_replica(L);
    const int lbpr = __builtin_ctz((unsigned)bpr);
    const int nb = bpr * nrep;
    const int remap = nb % 8 == 0 ? 1 : 0;
    const dim3 grid((unsigned)nb), block((unsigned)bits_wg(L));
    const bool e = energy && colour == 1;
    if (kind == 0) {
        if (e) hipLaunchKernelGGL((sweep_bits<0, 1, BATCH>), grid, block, 0, s, lat0, lats, map, colour, toff, r0, lbpr, remap);
        else hipLaunchKernelGGL((sweep_bits<0, 0, BATCH>), grid, block, 0, s, lat0, lats, map, colour, toff, r0, lbpr, remap);
    } else {
        if (e) hipLaunchKernelGGL((sweep_bits<1, 1, BATCH>), grid, block, 0, s, lat0, lats, map, colour, toff, r0, lbpr, remap);
        else hipLaunchKernelGGL((sweep_bits<1, 0, BATCH>), grid, block, 0, s, lat0, lats, map, colour, toff, r0, lbpr, remap);
    }
}
}  // namespace

hipError_t launch_bits_sweep(const Lattice &lat, int r0, int nrep, int colour, int toff, int energy, hipStream_t s) {
    if (nrep <= 0) return hipSuccess;
    launch_bits<false>(lat, nullptr, nullptr, lat.L, lat.kind, r0, nrep, colour, toff, energy, s);
    return hipGetLastError();
}

hipError_t launch_bits_batch(const Launch &ln, int colour, int toff, int energy, hipStream_t s) {
    if (ln.nblocks <= 0) return hipSuccess;
    launch_bits<true>(Lattice{}, ln.lats, ln.map, ln.L, ln.kind, 0, ln.nblocks, colour, toff, energy, s);
    return hipGetLastError();
}

hipError_t launch_pack_bits(const Lattice &lat, hipStream_t s) {
    const long long words = (long long)lat.R * 2 * (lat.N / 64);
    hipLaunchKernelGGL(pack_bits_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, lat);
    return hipGetLastError();
}

hipError_t launch_unpack_bits(const Lattice &lat, hipStream_t s) {
    const long long words = (long long)lat.R * 2 * (lat.N / 64);
    hipLaunchKernelGGL(unpack_bits_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, lat);
    return hipGetLastError();
}

// Workgroups per replica of the energy kernels in a readout, whose reduction
// does not have to match the sweep's: a step of every thread in each, 64 at
// most (the arena holds at least 64 partials per replica).
static int energy_blocks(const Lattice &lat) {
    const int unit = lat.bits ? 256 * 32 : 256 * 4 * (lat.L % 32 == 0 ? 4 : 1);
    return std::min(64, (lat.half + unit - 1) / unit);
}

template <int KIND, bool WHOLE>
static void launch_energy_kind(const Lattice &lat, dim3 grid, dim3 block, const Readout &out, hipStream_t s) {
    const FastDiv by_row = fast_div((uint32_t)lat.L / 2u), by_l = fast_div((uint32_t)lat.L);
    if (lat.bits)
        hipLaunchKernelGGL(energy_bits<KIND>, grid, block, 0, s, lat);
    else if (lat.L % 32 == 0)
        hipLaunchKernelGGL((energy_rows<KIND, 4, WHOLE>), grid, block, 0, s, lat, by_row, by_l, out);
    else if (lat.L % 8 == 0)
        hipLaunchKernelGGL((energy_rows<KIND, 1, WHOLE>), grid, block, 0, s, lat, by_row, by_l, out);
    else
        hipLaunchKernelGGL((energy_sites<KIND, WHOLE>), grid, block, 0, s, lat, by_row, by_l, out);
}

hipError_t launch_energy(const Lattice &lat, hipStream_t s) {
    const dim3 grid((unsigned)lat.nblk, (unsigned)lat.R), block(256);
    if (lat.kind == 0)
        launch_energy_kind<0, false>(lat, grid, block, Readout{}, s);
    else
        launch_energy_kind<1, false>(lat, grid, block, Readout{}, s);
    return hipGetLastError();
}

// One workgroup takes a whole replica up to L = 32 (at most 16 sites of each
// colour per thread; beyond, too few workgroups would read too much each) and
// 256 replicas: every workgroup ends its writes to the host for itself, 13 ns
// each (L = 8, R = 100 13 us against 17.5 with two launches, R = 500 20.5
// against 17.8; L = 32, R = 256 21.4 and 21.4).
static bool whole_energy(const Lattice &lat) {
    return !lat.bits && lat.half <= 16 * kWholeEnergyThreads && lat.R <= 256;
}

unsigned readout_flags(const Lattice &lat) { return whole_energy(lat) ? (unsigned)lat.R : 1u; }

hipError_t launch_readout(const Lattice &lat0, const Readout &out, hipStream_t s) {
    Lattice lat = lat0;
    if (whole_energy(lat)) {
        const unsigned chunks = (unsigned)(lat.half / 4 + 3) / (lat.L % 32 == 0 ? 4u : 1u);
        const dim3 grid(1, (unsigned)lat.R), block(std::min<unsigned>(kWholeEnergyThreads, (chunks + 63u) & ~63u));
        if (lat.kind == 0)
            launch_energy_kind<0, true>(lat, grid, block, out, s);
        else
            launch_energy_kind<1, true>(lat, grid, block, out, s);
        return hipGetLastError();
    }
    lat.nblk = energy_blocks(lat);
    const hipError_t e = launch_energy(lat, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(kExchangeThreads), 0, s, lat, out);
    return hipGetLastError();
}

hipError_t launch_clear(void *a, size_t na, void *b, size_t nb, hipStream_t s) {
    const size_t most = std::max(na, nb);
    if (most == 0) return hipSuccess;
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, s, (uint64_t *)a, (uint32_t)na,
                       (uint64_t *)b, (uint32_t)nb);
    return hipGetLastError();
}

unsigned copy_out_flags(const CopyOut &c) {
    unsigned n = 0;
    for (const uint32_t w : c.words) n += copy_blocks(w);
    return n;
}

hipError_t launch_copy_out(const CopyOut &c, hipStream_t s) {
    const unsigned nb = copy_out_flags(c);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(copy_out_kernel, dim3(nb), dim3(256), 0, s, c);
    return hipGetLastError();
}

// Units of 16 sites where a row holds whole units, else of 4 (a whole number
// of them in every replica).
static int natural_unit(const Lattice &lat) { return lat.L % 16 == 0 ? 16 : 4; }

hipError_t launch_spins_out(const Lattice &lat, size_t first, size_t count, int8_t *dst, hipStream_t s) {
    if (count == 0) return hipSuccess;
    const FastDiv by_l = fast_div((uint32_t)lat.L);
    const unsigned nb = (unsigned)((count / (size_t)natural_unit(lat) + 255) / 256);
    if (lat.bits)
        hipLaunchKernelGGL((spins_out_kernel<16, true>), dim3(nb), dim3(256), 0, s, lat, by_l, first, count, dst);
    else if (natural_unit(lat) == 16)
        hipLaunchKernelGGL((spins_out_kernel<16, false>), dim3(nb), dim3(256), 0, s, lat, by_l, first, count, dst);
    else
        hipLaunchKernelGGL((spins_out_kernel<4, false>), dim3(nb), dim3(256), 0, s, lat, by_l, first, count, dst);
    return hipGetLastError();
}

hipError_t launch_spins_in(const Lattice &lat, size_t first, size_t count, const int8_t *src, hipStream_t s) {
    if (count == 0) return hipSuccess;
    const FastDiv by_l = fast_div((uint32_t)lat.L);
    const size_t unit = lat.bits ? 64 : (size_t)natural_unit(lat);
    const unsigned nb = (unsigned)((count / unit + 255) / 256);
    if (lat.bits)
        hipLaunchKernelGGL(bits_in_kernel, dim3(nb), dim3(256), 0, s, lat, by_l, first, count, src);
    else if (unit == 16)
        hipLaunchKernelGGL(spins_in_kernel<16>, dim3(nb), dim3(256), 0, s, lat, by_l, first, count, src);
    else
        hipLaunchKernelGGL(spins_in_kernel<4>, dim3(nb), dim3(256), 0, s, lat, by_l, first, count, src);
    return hipGetLastError();
}

hipError_t launch_fields_in(const Lattice &lat, size_t first, size_t count, const float *src, hipStream_t s) {
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(fields_in_kernel, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, s, lat,
                       fast_div((uint32_t)lat.L), first, count, src);
    return hipGetLastError();
}

int partials_per_range(int R, int nblk) {
    int groups, per;
    partial_ranges(R, nblk, &groups, &per);
    return per;
}

hipError_t launch_exchange(const Lattice *lats, int n, int tadv, const StepIn &in, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(exchange_kernel, dim3(n), dim3(kExchangeThreads), 0, s, lats, tadv, in);
    return hipGetLastError();
}

hipError_t launch_advance(const Lattice &lat, int tadv, hipStream_t s) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(64), 0, s, lat.ctrs, tadv);
    return hipGetLastError();
}

}  // namespace rfim_dev
