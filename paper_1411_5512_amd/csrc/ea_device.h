// ea_device.h -- device-side building blocks shared by the gfx950 kernels:
// the counter-based random words, the packed lattice layout and the
// bit-sliced Metropolis decision.
//
// Packed layout.  Each colour c of each replica is stored as L*L rows, one
// per (y, z), row index y + L z.  A row holds the R = L/2 sites of colour c
// with that (y, z), ordered by xh = x >> 1 (so x = 2 xh + ((y + z + c) & 1)),
// split into RW words of W bits (R = W RW, W a multiple of 4, at most 32);
// bit b of word w is the site xh = W w + b, and bits W..31 are zero.  Spins
// carry 1 for S = -1, couplings 1 for J = -1; a site's three couplings to its
// +x, +y, +z neighbours ("left/up" bonds, Sec. III) live in three planes
// laid out like the spins of the site's colour.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ea {

// ---------------------------------------------------------------------------
// Counter-based random words: Philox4x32-10 (Salmon et al., SC'11).  The key
// is the run's seed, the counter names what the words are for; see ea.h for
// the keying.  Key and the upper counter words are wave-uniform, so the
// compiler keeps them (and the first round's product of word 2) in SGPRs.

struct Words4 {
    uint32_t v[4];
};

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ Words4 philox10(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                           uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t m0 = (uint64_t)x0 * 0xD2511F53u;
        const uint64_t m2 = (uint64_t)x2 * 0xCD9E8D57u;
        const uint32_t y0 = xor3((uint32_t)(m2 >> 32), x1, k0);
        const uint32_t y2 = xor3((uint32_t)(m0 >> 32), x3, k1);
        x1 = (uint32_t)m2;
        x3 = (uint32_t)m0;
        x0 = y0;
        x2 = y2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    Words4 r;
    r.v[0] = x0;
    r.v[1] = x1;
    r.v[2] = x2;
    r.v[3] = x3;
    return r;
}

// Counter word 1 of block J of a packed word of W sites is quad0 + J, where
// quad0 (the word's first 4-site block) is a multiple of W/4: rows and words
// hold whole numbers of blocks.  For W/4 a power of two the sum has no carry
// and equals quad0 | J, which the first round folds into its XOR.
template <int W>
constexpr bool kQuadOr = ((W / 4) & (W / 4 - 1)) == 0;

constexpr int kBitopOrXor = 0x56;  // (src0 | src1) ^ src2, bitwise

// How a gfx950 SIMD issues (probed with one instruction class at a time and
// mixed, two to eight waves per SIMD; cycles per wave instruction at 2.4 GHz):
// additions, right shifts and bitwise operations whose operands are VGPRs or
// constants issue from two waves at once (2.3); compares, carries, selects
// and any operation that reads an SGPR do not pair with each other (4.3) but
// do pair with one of the first kind; the 32 x 32 -> 64-bit multiply-add
// (4.3) pairs with nothing.  The oldest wave goes first, so waves that mix
// the kinds freely hardly ever meet at a pair (alternating multiply-adds and
// XORs: 4.25 each, as if nothing paired).  Raising a wave's priority while it
// runs its multiplies or compares lets the waves catch up there and meet in
// their XORs: 3.4 each at four waves.  Hence the phases below (PHASED), and
// the round keys and the wavefront-uniform words of the first rounds in
// VGPRs.  A wave that runs alone on its SIMD issues one instruction of any
// kind per 4.6 cycles, priority changes included, and takes the plain forms.
// The multiplies of a phase are one asm block between its two priority
// changes (the compiler would move plain multiplies across them).
#define EA_MAD(d, x, m) "v_mad_u64_u32 %" d ", vcc, %" x ", %" m ", 0\n\t"
#define EA_MULS_BEGIN "s_setprio 2\n\t"
#define EA_MULS_END "s_setprio 0"

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM2 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxK0 = 0x9E3779B9u, kPhiloxK1 = 0xBB67AE85u;

// p[g] = x[g] M
template <bool PHASED, int G>
__device__ __forceinline__ void mul_phase(uint64_t (&p)[G], const uint32_t (&x)[G], uint32_t M)
{
    static_assert(G >= 1 && G <= 4, "blocks side by side");
    if constexpr (!PHASED) {
#pragma unroll
        for (int g = 0; g < G; ++g) p[g] = (uint64_t)x[g] * M;
    } else if constexpr (G == 1)
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "1", "2") EA_MULS_END : "=&v"(p[0]) : "v"(x[0]), "s"(M) : "vcc");
    else if constexpr (G == 2)
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "2", "4") EA_MAD("1", "3", "4") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(p[1])
                     : "v"(x[0]), "v"(x[1]), "s"(M)
                     : "vcc");
    else if constexpr (G == 3)
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "3", "6") EA_MAD("1", "4", "6") EA_MAD("2", "5", "6") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2])
                     : "v"(x[0]), "v"(x[1]), "v"(x[2]), "s"(M)
                     : "vcc");
    else
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "4", "8") EA_MAD("1", "5", "8") EA_MAD("2", "6", "8")
                         EA_MAD("3", "7", "8") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3])
                     : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "s"(M)
                     : "vcc");
}

// p[g] = x[g] M0 and r[g] = y[g] M2
template <bool PHASED, int G>
__device__ __forceinline__ void mul_phase(uint64_t (&p)[G], const uint32_t (&x)[G], uint64_t (&r)[G],
                                          const uint32_t (&y)[G])
{
    static_assert(G >= 1 && G <= 4, "blocks side by side");
    if constexpr (!PHASED) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            p[g] = (uint64_t)x[g] * kPhiloxM0;
            r[g] = (uint64_t)y[g] * kPhiloxM2;
        }
    } else if constexpr (G == 1)
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "2", "4") EA_MAD("1", "3", "5") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(r[0])
                     : "v"(x[0]), "v"(y[0]), "s"(kPhiloxM0), "s"(kPhiloxM2)
                     : "vcc");
    else if constexpr (G == 2)
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "4", "8") EA_MAD("1", "5", "8") EA_MAD("2", "6", "9")
                         EA_MAD("3", "7", "9") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(r[0]), "=&v"(r[1])
                     : "v"(x[0]), "v"(x[1]), "v"(y[0]), "v"(y[1]), "s"(kPhiloxM0), "s"(kPhiloxM2)
                     : "vcc");
    else if constexpr (G == 3)
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "6", "12") EA_MAD("1", "7", "12") EA_MAD("2", "8", "12")
                         EA_MAD("3", "9", "13") EA_MAD("4", "10", "13") EA_MAD("5", "11", "13") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2])
                     : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(y[0]), "v"(y[1]), "v"(y[2]), "s"(kPhiloxM0),
                       "s"(kPhiloxM2)
                     : "vcc");
    else
        asm volatile(EA_MULS_BEGIN EA_MAD("0", "8", "16") EA_MAD("1", "9", "16") EA_MAD("2", "10", "16")
                         EA_MAD("3", "11", "16") EA_MAD("4", "12", "17") EA_MAD("5", "13", "17")
                             EA_MAD("6", "14", "17") EA_MAD("7", "15", "17") EA_MULS_END
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3]), "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]),
                       "=&v"(r[3])
                     : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]),
                       "s"(kPhiloxM0), "s"(kPhiloxM2)
                     : "vcc");
}
#undef EA_MAD

// A wavefront-uniform value held in a VGPR.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v)
{
    asm("" : "+v"(v));
    return v;
}

// The uniform part of the blocks of one half-step: counter words 0, 2, 3 and
// the key are the same for every lane, so only word 1's path is per lane in
// the first rounds (word 0 from round 1 on, word 2 from round 2 on, all four
// from round 4 on).  Rounds are numbered from 0.
template <bool PHASED>
struct PhiloxStep {
    uint32_t h;           // round 0: word 0 = counter word 1 ^ h
    uint32_t e1;          // round 1: word 2 = hi(m0) ^ e1
    uint32_t e2, e3;      // round 2: word 0 = hi(m2) ^ e2, word 2 = word 3 ^ e3
    uint32_t e4;          // round 3: word 2 = hi(m0) ^ e4
    uint32_t k0, k1;      // keys of round 3
};

template <bool PHASED = true>
__device__ __forceinline__ PhiloxStep<PHASED> philox_step(uint32_t x0, uint32_t x2, uint32_t x3, uint32_t k0, uint32_t k1)
{
    const uint64_t n0 = (uint64_t)x0 * kPhiloxM0, n2 = (uint64_t)x2 * kPhiloxM2;
    const uint32_t b2 = (uint32_t)(n0 >> 32) ^ x3 ^ k1;                      // word 2 after round 0
    const uint64_t p2 = (uint64_t)b2 * kPhiloxM2;                            // round 1
    const uint32_t c0 = (uint32_t)(p2 >> 32) ^ (uint32_t)n2 ^ (k0 + kPhiloxK0);  // word 0 after round 1
    const uint64_t q0 = (uint64_t)c0 * kPhiloxM0;                            // round 2
    auto hold = [](uint32_t v) { return PHASED ? in_vgpr(v) : v; };
    PhiloxStep<PHASED> s;
    s.h = hold((uint32_t)(n2 >> 32) ^ k0);
    s.e1 = hold((uint32_t)n0 ^ (k1 + kPhiloxK1));
    s.e2 = hold((uint32_t)p2 ^ (k0 + 2 * kPhiloxK0));
    s.e3 = hold((uint32_t)(q0 >> 32) ^ (k1 + 2 * kPhiloxK1));
    s.e4 = hold((uint32_t)q0 ^ (k1 + 3 * kPhiloxK1));
    s.k0 = hold(k0 + 3 * kPhiloxK0);
    s.k1 = hold(k1 + 3 * kPhiloxK1);
    return s;
}

// Blocks J, J - 1, ... J - G + 1 of a word side by side, round by round: each
// round's 2 G multiplies, then its 2 G XORs and the next keys.
template <int G, bool ORQ, bool PHASED>
__device__ __forceinline__ void philox10_group(const PhiloxStep<PHASED> &s, uint32_t quad0, int J, Words4 (&w)[G])
{
    uint32_t x0[G], x1[G], x2[G], x3[G];
    uint64_t m0[G], m2[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t j = (uint32_t)(J - g);
        x0[g] = ORQ ? __builtin_amdgcn_bitop3_b32(quad0, j, s.h, kBitopOrXor) : ((quad0 + j) ^ s.h);
    }
    mul_phase<PHASED>(m0, x0, kPhiloxM0);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        x2[g] = (uint32_t)(m0[g] >> 32) ^ s.e1;
        x3[g] = (uint32_t)m0[g];
    }
    mul_phase<PHASED>(m2, x2, kPhiloxM2);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        x0[g] = (uint32_t)(m2[g] >> 32) ^ s.e2;
        x1[g] = (uint32_t)m2[g];
        x2[g] = x3[g] ^ s.e3;
    }
    uint32_t k0 = s.k0, k1 = s.k1;
#pragma unroll
    for (int round = 3; round < 10; ++round) {
        mul_phase<PHASED>(m0, x0, m2, x2);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            x0[g] = xor3((uint32_t)(m2[g] >> 32), x1[g], k0);
            x2[g] = round == 3 ? (uint32_t)(m0[g] >> 32) ^ s.e4 : xor3((uint32_t)(m0[g] >> 32), x3[g], k1);
            x1[g] = (uint32_t)m2[g];
            x3[g] = (uint32_t)m0[g];
        }
        k0 += kPhiloxK0;
        k1 += kPhiloxK1;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        w[g].v[0] = x0[g];
        w[g].v[1] = x1[g];
        w[g].v[2] = x2[g];
        w[g].v[3] = x3[g];
    }
}

// Blocks taken together when n are left: at most four, and never all of a
// word's, so that its lattice reads and its table reads each have a group's
// rounds to arrive in.
constexpr int philox_group(int n) { return n >= 7 ? 4 : (n >= 5 ? 3 : (n >= 3 ? 2 : n)); }

enum : uint32_t { TAG_METRO = 0u, TAG_BOND = 1u, TAG_INIT = 2u };

__device__ __forceinline__ uint32_t counter_word2(uint32_t tag, uint32_t colour, uint32_t replica)
{
    return (tag << 8) | (colour << 1) | replica;
}

// ---------------------------------------------------------------------------
// Packed-row helpers.

template <int W>
__device__ __forceinline__ constexpr uint32_t word_mask()
{
    return W >= 32 ? 0xffffffffu : ((1u << W) - 1u);
}

// Word w of a row shifted so that bit b holds site xh - 1 (periodic in R):
// cur = word w, prev = word w-1 (mod RW).
template <int W>
__device__ __forceinline__ uint32_t take_minus1(uint32_t cur, uint32_t prev)
{
    return ((cur << 1) | (prev >> (W - 1))) & word_mask<W>();
}

// Word w of a row shifted so that bit b holds site xh + 1: next = word w+1.
template <int W>
__device__ __forceinline__ uint32_t take_plus1(uint32_t cur, uint32_t next)
{
    return (cur >> 1) | ((next & 1u) << (W - 1));
}

// Workgroups are handed to the 8 XCDs in turn (block b to XCD b mod 8), each
// XCD with its own L2.  Renumbering block b as (b mod 8) n/8 + b/8 gives each
// XCD a contiguous run of logical blocks, so that neighbouring rows of the
// lattice are read through the same L2 (n a multiple of 8; else unchanged).
__device__ __forceinline__ int xcd_block(int b, int n)
{
    return (n & 7) ? b : (b & 7) * (n >> 3) + (b >> 3);
}

// Debug order of a launch's workgroups (ea_set_debug).  order = 0 keeps
// block b; otherwise bit 31 reverses the order and bits 0..30 rotate it.
// Always a permutation of [0, n), so every tile is still taken exactly once.
__device__ __forceinline__ int debug_block(int b, int n, uint32_t order)
{
    if (order == 0) return b;
    if (order & 0x80000000u) b = n - 1 - b;
    return (int)(((uint32_t)b + (order & 0x7fffffffu) % (uint32_t)n) % (uint32_t)n);
}

// Debug fill of LDS words [0, n) (ea_set_debug's poison; 0 = off), so that a
// word read before the kernel wrote it shows up as a wrong result instead of
// a stale value that happens to be right.  The caller synchronises after it.
__device__ __forceinline__ void debug_poison(uint32_t *lds, int n, uint32_t poison, int tid, int nthreads)
{
    if (poison == 0) return;
    for (int i = tid; i < n; i += nthreads) lds[i] = poison ^ (uint32_t)i * 0x01000193u;
}

__device__ __forceinline__ int wrap(int v, int L)
{
    return v < 0 ? v + L : (v >= L ? v - L : v);
}

// ---------------------------------------------------------------------------
// Bit-sliced Metropolis decision for W sites of one colour (eq. 9).
//
// a1..a6 hold, per site, whether each of its six bonds is unsatisfied
// (J S_i S_j = -1).  With n unsatisfied bonds the flip costs dE = 12 - 4n:
// n >= 3 always flips, n = 2, 1, 0 flip iff the site's word is below
// thr1, thr2, thr3.  The counter is reduced with two full adders:
// n = s + 2 (c0 + c1 + c2), so "any" = (c0|c1|c2) means n >= 2 and
// "always" = maj(c0,c1,c2) | (any & s) means n >= 3.
constexpr int kBitopMaj = 0xE8, kBitopOr3 = 0xFE, kBitopOrAnd = 0xF8;  // 0xF8: src0 | (src1 & src2)

__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, kBitopMaj);
}

struct Decision {
    uint32_t always;  // n >= 3
    uint32_t any;     // n >= 2
    uint32_t odd;     // n odd
};

__device__ __forceinline__ Decision classify(uint32_t a1, uint32_t a2, uint32_t a3, uint32_t a4,
                                             uint32_t a5, uint32_t a6)
{
    const uint32_t s1 = xor3(a1, a2, a3), c1 = maj3(a1, a2, a3);
    const uint32_t s2 = xor3(a4, a5, a6), c2 = maj3(a4, a5, a6);
    const uint32_t s = s1 ^ s2;
    const uint32_t c0 = s1 & s2;
    Decision d;
    d.any = __builtin_amdgcn_bitop3_b32(c0, c1, c2, kBitopOr3);
    d.odd = s;
    d.always = __builtin_amdgcn_bitop3_b32(maj3(c0, c1, c2), d.any, s, kBitopOrAnd);
    return d;
}

// Per-site acceptance, branch-free.  For site bit I the threshold is picked
// with two sign-extended bit fields: any -> thr1 (n = 2), else odd -> thr2
// (n = 1), else thr3 (n = 0); sites with n >= 3 are covered by the "always"
// mask.  The accept word is built from the highest site bit down, one
// Philox block (four sites) at a time, by append_below4.
//
// v_bitop3_b32 truth tables are indexed by (src0 << 2) | (src1 << 1) | src2.
constexpr int kBitopSelect = 0xCA;   // src0 ? src1 : src2, bitwise

// accept = 16 accept + 8 [u3 < t3] + 4 [u2 < t2] + 2 [u1 < t1] + [u0 < t0].
// Each unsigned compare writes its lane mask to an SGPR pair and an add with
// carry-in (accept + accept + carry) appends the bit: two instructions per
// site.  gfx950 needs two wait states between a VALU write of an SGPR and a
// VALU read of it as a carry, so the four compares are issued first: every
// mask is read three instructions after it is written.
__device__ __forceinline__ uint32_t append_below4(uint32_t accept, uint32_t u3, uint32_t t3, uint32_t u2,
                                                  uint32_t t2, uint32_t u1, uint32_t t1, uint32_t u0,
                                                  uint32_t t0)
{
    uint64_t m3, m2, m1, m0, co;
    asm("v_cmp_lt_u32_e64 %1, %6, %7\n\t"
        "v_cmp_lt_u32_e64 %2, %8, %9\n\t"
        "v_cmp_lt_u32_e64 %3, %10, %11\n\t"
        "v_cmp_lt_u32_e64 %4, %12, %13\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %5, %0, %0, %4"
        : "+v"(accept), "=&s"(m3), "=&s"(m2), "=&s"(m1), "=&s"(m0), "=&s"(co)
        : "v"(u3), "v"(t3), "v"(u2), "v"(t2), "v"(u1), "v"(t1), "v"(u0), "v"(t0));
    return accept;
}

// Two blocks' bits (a above b) in one phase.
__device__ __forceinline__ uint32_t append_below8(uint32_t accept, const uint32_t (&a)[4], const uint4 &ta,
                                                  const uint32_t (&b)[4], const uint4 &tb)
{
    uint64_t m3, m2, m1, m0, co;
    asm volatile("s_setprio 1\n\t"
                 "v_cmp_lt_u32_e64 %1, %6, %7\n\t"
                 "v_cmp_lt_u32_e64 %2, %8, %9\n\t"
                 "v_cmp_lt_u32_e64 %3, %10, %11\n\t"
                 "v_cmp_lt_u32_e64 %4, %12, %13\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %1\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %2\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %3\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %4\n\t"
                 "v_cmp_lt_u32_e64 %1, %14, %15\n\t"
                 "v_cmp_lt_u32_e64 %2, %16, %17\n\t"
                 "v_cmp_lt_u32_e64 %3, %18, %19\n\t"
                 "v_cmp_lt_u32_e64 %4, %20, %21\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %1\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %2\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %3\n\t"
                 "v_addc_co_u32_e64 %0, %5, %0, %0, %4\n\t"
                 "s_setprio 0"
                 : "+&v"(accept), "=&s"(m3), "=&s"(m2), "=&s"(m1), "=&s"(m0), "=&s"(co)
                 : "v"(a[3]), "v"(ta.w), "v"(a[2]), "v"(ta.z), "v"(a[1]), "v"(ta.y), "v"(a[0]), "v"(ta.x),
                   "v"(b[3]), "v"(tb.w), "v"(b[2]), "v"(tb.z), "v"(b[1]), "v"(tb.y), "v"(b[0]), "v"(tb.x));
    return accept;
}

template <int I>
__device__ __forceinline__ uint32_t bit_as_mask(uint32_t word)
{
    // Written as an instruction so that the compiler does not rebuild it as
    // a compare and a lane-mask select.
    uint32_t m;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(word), "i"(I));
    return m;
}

template <int I>
__device__ __forceinline__ uint32_t site_threshold(const Decision &d, uint32_t thr1, uint32_t thr2, uint32_t thr3)
{
    const uint32_t m_any = bit_as_mask<I>(d.any);
    const uint32_t m_odd = bit_as_mask<I>(d.odd);
    return __builtin_amdgcn_bitop3_b32(m_any, thr1, __builtin_amdgcn_bitop3_b32(m_odd, thr2, thr3, kBitopSelect),
                                       kBitopSelect);
}

template <int J, int I, int G>
__device__ __forceinline__ uint32_t append_blocks_reg(uint32_t accept, const Decision &d, const Words4 (&u)[G],
                                                      uint32_t thr1, uint32_t thr2, uint32_t thr3)
{
    accept = append_below4(accept, u[I].v[3], site_threshold<4 * J + 3>(d, thr1, thr2, thr3), u[I].v[2],
                           site_threshold<4 * J + 2>(d, thr1, thr2, thr3), u[I].v[1],
                           site_threshold<4 * J + 1>(d, thr1, thr2, thr3), u[I].v[0],
                           site_threshold<4 * J>(d, thr1, thr2, thr3));
    if constexpr (I + 1 < G)
        return append_blocks_reg<J - 1, I + 1, G>(accept, d, u, thr1, thr2, thr3);
    else
        return accept;
}

// Blocks N-1 down to 0: block J covers sites 4J..4J+3 and has counter word 1
// equal to quad0 + J.
template <int W, int N>
__device__ __forceinline__ uint32_t accept_blocks(uint32_t accept, const Decision &d, const PhiloxStep<true> &s,
                                                  uint32_t quad0, uint32_t thr1, uint32_t thr2, uint32_t thr3)
{
    constexpr int G = philox_group(N);
    Words4 u[G];
    philox10_group<G, kQuadOr<W>>(s, quad0, N - 1, u);
    accept = append_blocks_reg<N - 1, 0, G>(accept, d, u, thr1, thr2, thr3);
    if constexpr (N > G)
        return accept_blocks<W, N - G>(accept, d, s, quad0, thr1, thr2, thr3);
    else
        return accept;
}

// Flip mask of one packed word of W sites (bits W..31 stay zero).
template <int W>
__device__ __forceinline__ uint32_t flip_mask(const Decision &d, const PhiloxStep<true> &s, uint32_t quad0, uint32_t thr1,
                                              uint32_t thr2, uint32_t thr3)
{
    return d.always | accept_blocks<W, W / 4>(0u, d, s, quad0, thr1, thr2, thr3);
}

// The same flip mask in two steps, for kernels that wait on global loads:
// first the W random words (they depend only on the counter, so they can be
// computed while the neighbour words are in flight), then the decisions.
template <int N, int W, bool PHASED>
__device__ __forceinline__ void random_words(const PhiloxStep<PHASED> &s, uint32_t quad0, uint32_t (&u)[W])
{
    constexpr int G = PHASED ? philox_group(N) : (N >= 2 ? 2 : 1);
    Words4 w[G];
    philox10_group<G, kQuadOr<W>>(s, quad0, N - 1, w);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) u[4 * (N - 1 - g) + i] = w[g].v[i];
    if constexpr (N > G) random_words<N - G, W, PHASED>(s, quad0, u);
}

template <int J, int W>
__device__ __forceinline__ uint32_t accept_words(uint32_t accept, const Decision &d, const uint32_t (&u)[W],
                                                 uint32_t thr1, uint32_t thr2, uint32_t thr3)
{
    accept = append_below4(accept, u[4 * J + 3], site_threshold<4 * J + 3>(d, thr1, thr2, thr3), u[4 * J + 2],
                           site_threshold<4 * J + 2>(d, thr1, thr2, thr3), u[4 * J + 1],
                           site_threshold<4 * J + 1>(d, thr1, thr2, thr3), u[4 * J],
                           site_threshold<4 * J>(d, thr1, thr2, thr3));
    if constexpr (J > 0)
        return accept_words<J - 1, W>(accept, d, u, thr1, thr2, thr3);
    else
        return accept;
}

// ---------------------------------------------------------------------------
// Threshold select through an LDS table, four sites per read.  A 4-site
// block has class bits any (n >= 2) and odd (n odd) for its four sites; the
// byte any_nibble | odd_nibble << 4 indexes a 256-entry table of 16-byte
// entries holding the block's four thresholds (any -> thr1, else odd ->
// thr2, else thr3; a site with n >= 3 is covered by the "always" mask, its
// entry is 0).  The index bytes of all blocks of a word come from two
// interleaves of the class masks: lo = (any & 0x0F0F0F0F) | (odd << 4 &
// 0xF0F0F0F0) holds those of blocks 0, 2, 4, 6, hi = (any >> 4 & 0x0F0F0F0F)
// | (odd & 0xF0F0F0F0) those of blocks 1, 3, 5, 7, so an entry's byte offset
// is one byte extract and shift: per 8 sites one interleave op, two extracts
// and two 16-byte reads.
//
// Layout (words): entry e at [4e, 4e + 4).

constexpr int kSelectTableWords = 4 * 256;

// Fill the table (any thread count; caller synchronises before use).
__device__ __forceinline__ void fill_select_tables(uint32_t *tab, uint32_t thr1, uint32_t thr2, uint32_t thr3,
                                                   int tid, int nthreads)
{
    for (int i = tid; i < kSelectTableWords; i += nthreads) {
        const int idx = i >> 2, q = i & 3;
        const int any = (idx >> q) & 1, odd = (idx >> (4 + q)) & 1;
        tab[i] = any ? (odd ? 0u : thr1) : (odd ? thr2 : thr3);
    }
}

// Index bytes of a word's blocks: those of blocks 0, 2, 4, 6 and 1, 3, 5, 7.
struct SelectIndex {
    uint32_t lo, hi;
};

__device__ __forceinline__ SelectIndex select_index(const Decision &d)
{
    const uint32_t nib = in_vgpr(0x0F0F0F0Fu);
    SelectIndex x;
    x.lo = __builtin_amdgcn_bitop3_b32(nib, d.any, d.odd << 4, kBitopSelect);
    x.hi = __builtin_amdgcn_bitop3_b32(nib, d.any >> 4, d.odd, kBitopSelect);
    return x;
}

// The four thresholds of block g from the table (16-byte aligned).
__device__ __forceinline__ uint4 select_block(const SelectIndex &x, const uint32_t *tab, int g)
{
    const uint32_t src = (g & 1) ? x.hi : x.lo;
    const uint32_t byte_off = ((src >> (8 * (g >> 1))) & 0xffu) << 4;
    return *(const uint4 *)((const char *)tab + byte_off);
}

// The bits of G blocks, the first uppermost.
template <int G>
__device__ __forceinline__ uint32_t append_blocks(uint32_t accept, const Words4 (&u)[G], const uint4 (&t)[G])
{
#pragma unroll
    for (int g = 0; g + 1 < G; g += 2) accept = append_below8(accept, u[g].v, t[g], u[g + 1].v, t[g + 1]);
    if constexpr (G & 1) {
        const Words4 &e = u[G - 1];
        const uint4 &f = t[G - 1];
        accept = append_below4(accept, e.v[3], f.w, e.v[2], f.z, e.v[1], f.y, e.v[0], f.x);
    }
    return accept;
}

// Blocks M-1 down to 0 after the group above them (G blocks, words u and
// thresholds t): this group's thresholds are read, its words drawn, and only
// then is the group above compared, so neither the table reads nor the
// compares wait.
template <int W, int M, int G>
__device__ __forceinline__ uint32_t accept_rest(uint32_t accept, const SelectIndex &x, const PhiloxStep<true> &s,
                                                uint32_t quad0, const uint32_t *tab, const Words4 (&u)[G],
                                                const uint4 (&t)[G])
{
    if constexpr (M > 0) {
        constexpr int G2 = philox_group(M);
        uint4 t2[G2];
        Words4 u2[G2];
#pragma unroll
        for (int g = 0; g < G2; ++g) t2[g] = select_block(x, tab, M - 1 - g);
        philox10_group<G2, kQuadOr<W>>(s, quad0, M - 1, u2);
        accept = append_blocks(accept, u, t);
        return accept_rest<W, M - G2, G2>(accept, x, s, quad0, tab, u2, t2);
    } else {
        return append_blocks(accept, u, t);
    }
}

// Flip mask of one packed word of W sites, thresholds from the LDS table
// (tab = kSelectTableWords words filled by fill_select_tables, 16-byte
// aligned).  decide() classifies the word; it is called after the first
// group's words are drawn, so that the lattice loads it waits for (issued
// before this call) are in flight meanwhile.
template <int W, class Decide>
__device__ __forceinline__ uint32_t flip_mask_lds(const PhiloxStep<true> &s, uint32_t quad0, const uint32_t *tab,
                                                  const Decide &decide)
{
    constexpr int N = W / 4, G = philox_group(N);
    Words4 u[G];
    philox10_group<G, kQuadOr<W>>(s, quad0, N - 1, u);
    const Decision d = decide();
    const SelectIndex x = select_index(d);
    uint4 t[G];
#pragma unroll
    for (int g = 0; g < G; ++g) t[g] = select_block(x, tab, N - 1 - g);
    return d.always | accept_rest<W, N - G, G>(0u, x, s, quad0, tab, u, t);
}

}  // namespace ea
