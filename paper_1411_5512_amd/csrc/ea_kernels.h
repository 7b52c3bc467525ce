// ea_kernels.h -- gfx950 kernels of the plain form: initial state, one
// checkerboard half-step per launch, snapshots and the measurement
// reductions.  Layout and random words are described in ea_device.h.
#pragma once

#include "ea_device.h"

namespace ea {

// Geometry of one packed lattice, passed by value to every kernel.
struct Geom {
    int L;       // side length
    int R;       // sites of one colour per row, L / 2
    int RW;      // words per row
    int rows;    // L * L
    int plane;   // words per colour plane, rows * RW
    uint32_t order = 0;  // debug order of the half-step launches' blocks (debug_block)
};

// Device pointers of one run.
struct Lattice {
    uint32_t *spins;  // [replica 2][colour 2][plane]
    uint32_t *bonds;  // [direction 3][colour 2][plane]
};

__device__ __forceinline__ size_t plane_off(const Geom &g, int a, int c)
{
    return ((size_t)a * 2 + (size_t)c) * (size_t)g.plane;
}

// --------------------------------------------------------------------------
// Initial state (Sec. II): couplings with P(J = -1) = p and two replicas of
// uniformly random spins.

// One packed word of colour c, from block quad0 on; what = 0..2: couplings of
// that direction, 3..4: spins of replica 0 / 1.
template <int W>
__device__ __forceinline__ uint32_t init_word(int what, int c, uint32_t quad0, uint32_t sample, uint32_t k0,
                                              uint32_t k1, uint64_t pcut)
{
    const bool is_bond = what < 3;
    const uint32_t aux = is_bond ? (uint32_t)what : 0u;
    const uint32_t rep = is_bond ? 0u : (uint32_t)(what - 3);
    const uint32_t c2 = counter_word2(is_bond ? TAG_BOND : TAG_INIT, (uint32_t)c, rep);
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < W / 4; ++j) {
        const Words4 u = philox10(aux, quad0 + (uint32_t)j, c2, sample, k0, k1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t bit = is_bond ? (uint32_t)((uint64_t)u.v[q] < pcut) : (u.v[q] >> 31);
            bits |= bit << (4 * j + q);
        }
    }
    return bits;
}

// One thread per (row, word) of one colour; grid.y selects what is drawn: 0..2
// the coupling planes of direction d, 3..4 the spins of replica 0 / 1; grid.z
// the colour.
// The first block also clears the caller's error word and n_clear counters
// (err may be null).
template <int W>
__global__ __launch_bounds__(256) void init_kernel(Lattice lat, Geom g, uint32_t k0, uint32_t k1,
                                                   uint32_t sample, uint64_t pcut, uint32_t *err,
                                                   unsigned long long *clear, int n_clear)
{
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    if (err && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) {
        if (threadIdx.x == 0) *err = 0u;
        for (int i = threadIdx.x; i < n_clear; i += blockDim.x) clear[i] = 0ull;
    }
    if (tid >= g.plane) return;
    const int what = blockIdx.y;
    const int c = blockIdx.z;
    const int row = tid / g.RW;
    const int w = tid - row * g.RW;
    const uint32_t quad0 = (uint32_t)((row * g.R + w * W) >> 2);
    const bool is_bond = what < 3;
    const uint32_t bits = init_word<W>(what, c, quad0, sample, k0, k1, pcut);
    uint32_t *dst = is_bond ? lat.bonds + plane_off(g, what, c) : lat.spins + plane_off(g, what - 3, c);
    dst[tid] = bits;
}

// Bit i set iff u[i] < thr, for all W words (two instructions per site).
template <int J, int W>
__device__ __forceinline__ uint32_t below_words(uint32_t accept, const uint32_t (&u)[W], uint32_t thr)
{
    accept = append_below4(accept, u[4 * J + 3], thr, u[4 * J + 2], thr, u[4 * J + 1], thr, u[4 * J], thr);
    if constexpr (J > 0)
        return below_words<J - 1, W>(accept, u, thr);
    else
        return accept;
}

// The same acceptance as accept_words, cheaper where uphill moves of
// dE >= 8 are rare.  If none of the W random words falls below thr2 (and
// thr3 <= thr2), every site with n = 1 or n = 0 is rejected, and a site with
// n = 2 (any & ~always) flips iff its word is below thr1: one compare and
// one append per site instead of a per-site threshold select.  Lanes where
// some word is below thr2 take the general select, so the decisions are the
// same either way.  Used only while a wave meets such a word rarely (thr2 W
// < 2^24, i.e. 64 W thr2 / 2^32 < 1/4 expected per wave), where both
// branches would otherwise run in most waves, and only in launches with
// several waves per SIMD (SCREEN): a wave that runs alone on its SIMD
// is bound by its chain of dependent instructions, which the screen
// lengthens (measured 9% slower for one L = 128 run, 7-12% faster for 5-16
// runs in one launch).  A separate instantiation, so that the unscreened
// kernels keep their own schedule.
template <int W, bool SCREEN>
__device__ __forceinline__ uint32_t accept_screened(const Decision &d, const uint32_t (&u)[W], uint32_t thr1,
                                                    uint32_t thr2, uint32_t thr3)
{
    if constexpr (!SCREEN) return accept_words<W / 4 - 1, W>(0u, d, u, thr1, thr2, thr3);
    const bool rare = (uint64_t)thr2 * (uint64_t)W < (1ull << 24) && thr3 <= thr2;  // uniform
    if (rare) {
        // the n = 2 compares and a three-way minimum tree (depth 4 for
        // W = 32) are independent, so their latencies overlap
        const uint32_t a1 = below_words<W / 4 - 1, W>(0u, u, thr1);
        uint32_t v[W];
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] = u[i];
#pragma unroll
        for (int n = W; n > 1; n = (n + 2) / 3) {
#pragma unroll
            for (int i = 0; 3 * i < n; ++i) {
                uint32_t m = v[3 * i];
                if (3 * i + 1 < n) m = min(m, v[3 * i + 1]);
                if (3 * i + 2 < n) m = min(m, v[3 * i + 2]);
                v[i] = m;
            }
        }
        if (v[0] >= thr2) return a1 & d.any & ~d.always;
    }
    return accept_words<W / 4 - 1, W>(0u, d, u, thr1, thr2, thr3);
}

// --------------------------------------------------------------------------
// One checkerboard half-step (Sec. III, eq. 9) of sweep t = *t_base + t_off
// (the base lives on the device so that a captured graph of sweeps can be
// replayed).  grid.y = replica r, which updates colour c = r ^ half; all six
// neighbours of a colour-c site have colour 1 - c, so every thread reads the
// other colour and writes only its own word.  One thread per (row, word).
template <int W, bool SCREEN>
__device__ __forceinline__ void half_step_word(const Lattice &lat, const Geom &g, int half, uint32_t t, int r,
                                               int tid, uint32_t k0, uint32_t k1, uint32_t sample, uint32_t thr1,
                                               uint32_t thr2, uint32_t thr3)
{
    const int c = r ^ half;
    const int row = tid / g.RW;
    const int w = tid - row * g.RW;
    const int y = row % g.L;
    const int z = row / g.L;
    const int par = (y + z + c) & 1;  // x = 2 xh + par on this row
    const int wm = w == 0 ? g.RW - 1 : w - 1;
    const int wp = w == g.RW - 1 ? 0 : w + 1;
    const int row_ym = wrap(y - 1, g.L) + g.L * z, row_yp = wrap(y + 1, g.L) + g.L * z;
    const int row_zm = y + g.L * wrap(z - 1, g.L), row_zp = y + g.L * wrap(z + 1, g.L);

    uint32_t *own = lat.spins + plane_off(g, r, c);
    const uint32_t *oth = lat.spins + plane_off(g, r, c ^ 1);
    const uint32_t *bx_own = lat.bonds + plane_off(g, 0, c);
    const uint32_t *by_own = lat.bonds + plane_off(g, 1, c);
    const uint32_t *bz_own = lat.bonds + plane_off(g, 2, c);
    const uint32_t *bx_oth = lat.bonds + plane_off(g, 0, c ^ 1);
    const uint32_t *by_oth = lat.bonds + plane_off(g, 1, c ^ 1);
    const uint32_t *bz_oth = lat.bonds + plane_off(g, 2, c ^ 1);

    const int base = row * g.RW;
    const uint32_t S = own[base + w];
    const uint32_t O = oth[base + w], Om = oth[base + wm], Op = oth[base + wp];
    const uint32_t Xo = bx_oth[base + w], Xom = bx_oth[base + wm];
    const uint32_t Bx = bx_own[base + w], By = by_own[base + w], Bz = bz_own[base + w];
    const uint32_t Yp = oth[row_yp * g.RW + w], Ym = oth[row_ym * g.RW + w], Bym = by_oth[row_ym * g.RW + w];
    const uint32_t Zp = oth[row_zp * g.RW + w], Zm = oth[row_zm * g.RW + w], Bzm = bz_oth[row_zm * g.RW + w];

    // the random words do not depend on the lattice: computed here, they
    // overlap the latency of the loads above (the scheduling barrier keeps
    // every load issued before them)
    __builtin_amdgcn_sched_barrier(0);
    uint32_t u[W];
    random_words<W / 4, W>(philox_step<SCREEN>(t, counter_word2(TAG_METRO, (uint32_t)c, (uint32_t)r), sample, k0, k1),
                           (uint32_t)((row * g.R + w * W) >> 2), u);

    // x neighbours: on even rows (par = 0) the +x neighbour shares xh and the
    // -x neighbour sits at xh - 1; on odd rows the +x neighbour is at xh + 1
    // and the -x neighbour shares xh.  The -x bond is stored at the -x site.
    // (selected with a mask rather than a branch, so that no load waits
    // inside a divergent branch before the random words are computed)
    const uint32_t pm = 0u - (uint32_t)par;
    const uint32_t xp = __builtin_amdgcn_bitop3_b32(pm, take_plus1<W>(O, Op), O, kBitopSelect);
    const uint32_t xm = __builtin_amdgcn_bitop3_b32(pm, O ^ Xo, take_minus1<W>(O ^ Xo, Om ^ Xom), kBitopSelect);
    const uint32_t a1 = S ^ xp ^ Bx;
    const uint32_t a2 = S ^ xm;
    const uint32_t a3 = xor3(S, Yp, By);
    const uint32_t a4 = xor3(S, Ym, Bym);
    const uint32_t a5 = xor3(S, Zp, Bz);
    const uint32_t a6 = xor3(S, Zm, Bzm);

    const Decision d = classify(a1, a2, a3, a4, a5, a6);
    // register selects, no LDS table: a table would add a fill and a barrier
    // to every block of a launch this short
    const uint32_t flips = d.always | accept_screened<W, SCREEN>(d, u, thr1, thr2, thr3);
    own[base + w] = S ^ flips;
}

template <int W, bool SCREEN>
__global__ __launch_bounds__(256) void half_step_kernel(Lattice lat, Geom g, int half,
                                                        const uint32_t *__restrict__ t_base, uint32_t t_off,
                                                        uint32_t k0, uint32_t k1, uint32_t sample,
                                                        uint32_t thr1, uint32_t thr2, uint32_t thr3)
{
    const int blk = debug_block((int)blockIdx.x, (int)gridDim.x, g.order);
    const int tid = xcd_block(blk, (int)gridDim.x) * (int)blockDim.x + (int)threadIdx.x;
    if (tid >= g.plane) return;
    half_step_word<W, SCREEN>(lat, g, half, *t_base + t_off, (int)blockIdx.y, tid, k0, k1, sample, thr1, thr2,
                              thr3);
}

// Several runs of the same geometry in one launch: grid.z = member.  Each
// member keeps its own couplings, key, thresholds and sweep counter, so the
// launch is the members' own half-steps side by side.
constexpr int kGroupMax = 16;

struct GroupMember {
    Lattice lat;
    const uint32_t *t_base;
    uint32_t k0, k1, sample, thr1, thr2, thr3;
};

struct GroupArgs {
    GroupMember m[kGroupMax];
};

template <int W, bool SCREEN>
__global__ __launch_bounds__(256) void group_half_step_kernel(GroupArgs a, Geom g, int half, uint32_t t_off)
{
    const int blk = debug_block((int)blockIdx.x, (int)gridDim.x, g.order);
    const int tid = xcd_block(blk, (int)gridDim.x) * (int)blockDim.x + (int)threadIdx.x;
    if (tid >= g.plane) return;
    const GroupMember &M = a.m[blockIdx.z];
    half_step_word<W, SCREEN>(M.lat, g, half, *M.t_base + t_off, (int)blockIdx.y, tid, M.k0, M.k1, M.sample,
                              M.thr1, M.thr2, M.thr3);
}

// --------------------------------------------------------------------------
// Reductions.  Sums are popcounts (number of set bits); the host turns them
// into the +-1 sums of ea_obs.  Each wave reduces with cross-lane shuffles
// and adds its total to a 64-bit counter (integer, so the result does not
// depend on the order of the atomics).

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ void wave_add(unsigned long long *dst, uint32_t v)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, (unsigned long long)v);
}

// Counter layout of one measurement (all uint64):
//   [0,1] unsatisfied bonds of replica 0/1
//   [2,3] spins with S = -1, replica 0/1
//   [4]   sites with S_0 != S_1
//   [5 + 2k + r] sites with S_r(t) != S_r(tw_k)
// followed by the C4 block: [c4_base + d (R+1) + rho] sites with q(s) != q(s + rho e_d).
enum { M_UNSAT = 0, M_DOWN = 2, M_QDIFF = 4, M_AUTO = 5 };

// q = S_0 xor S_1 of word w of a packed row.
__device__ __forceinline__ uint32_t q_word(const Lattice &lat, const Geom &g, int c, int row, int w)
{
    const size_t i = (size_t)row * g.RW + (size_t)w;
    return lat.spins[plane_off(g, 0, c) + i] ^ lat.spins[plane_off(g, 1, c) + i];
}

// A measurement in one launch.  Its blocks, in order:
//   nb blocks           unsatisfied bonds, down spins, the overlap
//   n_slots * nb        the autocorrelation with slot k
//   3 L (c4 wanted)     the axis correlations: L blocks per axis, one plane
//                       of lines each
// The counters are added to, never cleared: the caller subtracts what they
// held before (a clearing launch costs as much as the measurement of a small
// lattice).  The slabs' error word rides along in the C4 block's rho = 0
// entry, whose count is 0 by definition, so that one copy brings everything.
//
// Bounds, at L = 256: 2 x 10 MB read and 2 x 10^8 XOR-popcounts.  One block
// row per displacement and block sums for every quantity took 700 + 170 us
// there (60 + 24 us at L = 128); now each line is read once into LDS and each
// thread keeps one displacement.  A whole ea_measure call, before and now:
// L = 16 39 -> 28 us, L = 64 62 -> 35, L = 128 108 -> 46, L = 256 830 -> 102.
constexpr int kMeasThreads = 256;
constexpr int kMeasBlocks = 512;  // at most, per quantity: more only adds atomics on the same counters

// 32 bits of the periodic q row (c, row) of R bits, from bit `start` (< 2R) on.
template <int W>
__device__ __forceinline__ uint32_t q_bits(const Lattice &lat, const Geom &g, int c, int row, int start)
{
    int pos = start >= g.R ? start - g.R : start;
    uint32_t out = 0;
    for (int have = 0; have < 32;) {
        const int w = pos / W, off = pos - w * W;
        out |= (q_word(lat, g, c, row, w) >> off) << have;
        have += W - off;
        pos = (w + 1) * W;
        if (pos == g.R) pos = 0;
    }
    return out;
}

__device__ __forceinline__ int meas_row_words(int R) { return (R + 31) / 32; }
// Words of a row repeated far enough for every shift up to R / 2 + 1.
__device__ __forceinline__ int meas_shift_words(int R) { return (R + R / 2 + 66) / 32 + 1; }

// One plane of L lines along axis D (0 x, 1 y, 2 z): the q words of both
// colours go to LDS -- along x every row, repeated periodically; along y and
// z column-wise, twice, so that the line shifted by rho is contiguous -- and
// thread (part, rho) counts displacement rho = 1 .. R over its part of the
// plane.  The partner of site (x,y,z) is (x,y,z) + rho e_d, of colour
// c ^ (rho & 1).  Along y and z it sits at the same half index of the partner
// row; along x, on a row with x = 2 xh + par, its half index is xh + rho/2
// (rho even) or xh + (rho-1)/2 + par (rho odd), modulo R.
template <int W>
__device__ __forceinline__ void measure_axis(const Lattice &lat, const Geom &g, int D, int o, uint32_t *lds,
                                             uint32_t *sums, unsigned long long *acc)
{
    const int tid = (int)threadIdx.x, L = g.L, R = g.R;
    const int nw = meas_row_words(R);
    const uint32_t last = (R & 31) ? (1u << (R & 31)) - 1u : 0xffffffffu;  // sites of a row's last word
    const int parts = kMeasThreads / R, part = tid / R, rho = 1 + tid - part * R;
    const int odd = rho & 1;
    for (int i = tid; i < R; i += kMeasThreads) sums[i] = 0u;
    uint32_t diff = 0;
    if (D == 0) {
        // lds[c][y][nx]: plane z = o
        const int nx = meas_shift_words(R);
        for (int i = tid; i < 2 * L * nx; i += kMeasThreads) {
            const int j = i % nx, k = i / nx, y = k % L, c = k / L;
            lds[i] = q_bits<W>(lat, g, c, y + L * o, (32 * j) % R);
        }
        __syncthreads();
        if (part < parts)
            for (int y = part; y < L; y += parts) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int sh = (rho >> 1) + (odd ? (y + o + c) & 1 : 0);
                    const uint32_t *own = lds + (c * L + y) * nx;
                    const uint32_t *other = lds + ((c ^ odd) * L + y) * nx + (sh >> 5);
                    uint32_t prev = other[0];
                    for (int j = 0; j < nw; ++j) {
                        const uint32_t next = other[j + 1];
                        const uint32_t win = __builtin_amdgcn_alignbit(next, prev, (uint32_t)sh & 31u);
                        diff += __popc((own[j] ^ win) & (j + 1 == nw ? last : 0xffffffffu));
                        prev = next;
                    }
                }
            }
    } else {
        // lds[c][word][2L]: along y the plane z = o, along z the plane y = o
        for (int i = tid; i < 2 * nw * L; i += kMeasThreads) {
            const int j = i % nw, k = i / nw, n = k % L, c = k / L;
            const int row = D == 1 ? n + L * o : o + L * n;
            const uint32_t v = q_bits<W>(lat, g, c, row, 32 * j) & (j + 1 == nw ? last : 0xffffffffu);
            uint32_t *dst = lds + (c * nw + j) * 2 * L + n;
            dst[0] = v;
            dst[L] = v;
        }
        __syncthreads();
        if (part < parts)
            for (int cj = 0; cj < 2 * nw; ++cj) {
                const int c = cj >= nw ? 1 : 0, j = cj - c * nw;
                const uint32_t *own = lds + (c * nw + j) * 2 * L;
                const uint32_t *other = lds + ((c ^ odd) * nw + j) * 2 * L + rho;
                for (int n = part; n < L; n += parts) diff += __popc(own[n] ^ other[n]);
            }
    }
    if (part < parts) atomicAdd(sums + rho - 1, diff);
    __syncthreads();
    for (int i = tid; i < R; i += kMeasThreads)
        if (sums[i]) atomicAdd(acc + D * (R + 1) + 1 + i, (unsigned long long)sums[i]);
}

template <int W>
__global__ __launch_bounds__(kMeasThreads) void measure_kernel(Lattice lat, Geom g, const uint32_t *snaps, int nb,
                                                               int n_slots, unsigned long long *acc, int c4_base,
                                                               const uint32_t *err)
{
    // 2 colours x 256 rows x 9 words (x), 2 x 4 words x 512 (y, z)
    __shared__ uint32_t lds[2 * 256 * 9];
    __shared__ uint32_t sums[128];
    const int tid = (int)threadIdx.x;
    int b = (int)blockIdx.x;
    if (b >= nb * (1 + n_slots)) {
        b -= nb * (1 + n_slots);
        measure_axis<W>(lat, g, b / g.L, b % g.L, lds, sums, acc + c4_base);
        return;
    }
    const int k = b / nb - 1;  // -1: the configuration itself, else a slot
    b -= (k + 1) * nb;
    uint32_t cnt[5] = {0u, 0u, 0u, 0u, 0u};
    if (k < 0) {
        if (b == 0 && tid == 0) acc[c4_base] = *err;
        for (int gid = b * kMeasThreads + tid; gid < 2 * g.plane; gid += nb * kMeasThreads) {
            const int c = gid >= g.plane ? 1 : 0;
            const int at = gid - c * g.plane;
            const int row = at / g.RW;
            const int w = at - row * g.RW;
            const int z = row / g.L, y = row - z * g.L;
            const int par = (y + z + c) & 1;
            const int wp = w == g.RW - 1 ? at - w : at + 1;
            const int yp = y == g.L - 1 ? at - (g.L - 1) * g.RW : at + g.RW;
            const int zp = z == g.L - 1 ? at - (g.L - 1) * g.L * g.RW : at + g.L * g.RW;
            const uint32_t Bx = lat.bonds[plane_off(g, 0, c) + at], By = lat.bonds[plane_off(g, 1, c) + at],
                           Bz = lat.bonds[plane_off(g, 2, c) + at];
            uint32_t S[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const uint32_t *oth = lat.spins + plane_off(g, r, c ^ 1);
                S[r] = lat.spins[plane_off(g, r, c) + at];
                const uint32_t O = oth[at];
                const uint32_t xp = par ? take_plus1<W>(O, oth[wp]) : O;
                cnt[M_UNSAT + r] += __popc(xor3(S[r], xp, Bx)) + __popc(xor3(S[r], oth[yp], By)) +
                                    __popc(xor3(S[r], oth[zp], Bz));
                cnt[M_DOWN + r] += __popc(S[r]);
            }
            cnt[M_QDIFF] += __popc(S[0] ^ S[1]);
        }
    } else {
        const uint32_t *ref = snaps + (size_t)k * 4 * (size_t)g.plane;
        for (int r = 0; r < 2; ++r)
            for (int i = b * kMeasThreads + tid; i < 2 * g.plane; i += nb * kMeasThreads)
                cnt[r] += __popc(lat.spins[plane_off(g, r, 0) + i] ^ ref[plane_off(g, r, 0) + i]);
    }
    // one atomic per block and quantity
    if (tid < 5) sums[tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const uint32_t v = wave_sum(cnt[i]);
        if ((tid & 63) == 0 && v) atomicAdd(sums + i, v);
    }
    __syncthreads();
    const int n = k < 0 ? 5 : 2, first = k < 0 ? 0 : M_AUTO + 2 * k;
    if (tid < n && sums[tid]) atomicAdd(acc + first + tid, (unsigned long long)sums[tid]);
}

// --------------------------------------------------------------------------
// Full-vector C4 (eq. 3 over every displacement r), summed by minimum-image
// distance shells k = |r|^2.  q = S_0 xor S_1 is first rewritten in natural
// x order, one doubled row per (y, z): bits [0, L) hold x = 0..L-1 and bits
// [L, 2L) repeat them, in dw 64-bit words, so that the row shifted
// cyclically by rx is the window of L bits starting at bit rx.

// Bits 0 .. 31 of v moved to the even bits of the result.
__device__ __forceinline__ unsigned long long even_bits(uint32_t v)
{
    unsigned long long x = v;
    x = (x | x << 16) & 0x0000ffff0000ffffull;
    x = (x | x << 8) & 0x00ff00ff00ff00ffull;
    x = (x | x << 4) & 0x0f0f0f0f0f0f0f0full;
    x = (x | x << 2) & 0x3333333333333333ull;
    return (x | x << 1) & 0x5555555555555555ull;
}

// One thread per (row, word of the doubled row): the row's 32 sites of each
// colour from R (j 32 / R) on, taken word by word and then interleaved.  Bound
// by the launch: 3.2 us at L = 128; one site at a time took 15.
template <int W>
__global__ __launch_bounds__(256) void dense_q_kernel(Lattice lat, Geom g, int dw, unsigned long long *qd)
{
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= g.rows * dw) return;
    const int row = gid / dw, j = gid - row * dw, z = row / g.L, y = row - z * g.L;
    const int c0 = (y + z) & 1;  // colour of the even x
    const int n = min(32, g.L - 32 * j);  // sites of either colour; the doubled row has L
    unsigned long long bits = 0;
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) {
        const size_t base = plane_off(g, 0, c0 ^ odd) + (size_t)row * g.RW;
        const size_t to_s1 = plane_off(g, 1, 0) - plane_off(g, 0, 0);
        uint32_t v = 0;
        for (int i = 0; i < n;) {
            const int h = (32 * j + i) % g.R, w = h / W, off = h - w * W, take = min(W - off, n - i);
            const uint32_t q = lat.spins[base + w] ^ lat.spins[base + to_s1 + w];
            v |= ((q >> off) & (0xffffffffu >> (32 - take))) << i;
            i += take;
        }
        bits |= even_bits(v) << odd;
    }
    qd[gid] = bits;
}

constexpr int kShellRx = 16;  // displacements along x per workgroup

__device__ __forceinline__ int min_image_sq(int r, int L)
{
    const int m = r < L - r ? r : L - r;
    return m * m;
}

// Workgroup (rx chunk, ry + L rz): every thread takes source rows with a
// stride, holds the source row (NW words) and the partner row at
// (y + ry, z + rz) (doubled, 2 NW words) in registers, counts the sites where
// q differs from q at x + r for the kShellRx displacements rx of the chunk,
// the workgroup adds the counts, and sum_x q(x) q(x + r) = N - 2 * count is
// added to the shell of r.  NW = ceil(L / 64) words per row (L <= 128).
template <int NW>
__global__ __launch_bounds__(256) void c4_shell_kernel(const unsigned long long *qd, int L, int n_shells,
                                                       unsigned long long *shells)
{
    constexpr int DW = 2 * NW;  // words of a doubled row
    __shared__ unsigned int part[kShellRx][256 / 64];
    const int rx0 = blockIdx.x * kShellRx;
    const int ry = (int)(blockIdx.y % (unsigned)L), rz = (int)(blockIdx.y / (unsigned)L);
    const int kyz = min_image_sq(ry, L) + min_image_sq(rz, L);
    int kmin = 1 << 30;
    for (int i = 0; i < kShellRx; ++i)
        if (rx0 + i < L) kmin = min(kmin, kyz + min_image_sq(rx0 + i, L));
    if (kmin >= n_shells) return;  // whole workgroup: no barrier passed yet
    const int tail = L - 64 * (NW - 1);  // bits used in the last word of a row
    const unsigned long long last_mask = tail == 64 ? ~0ull : ((1ull << tail) - 1ull);
    unsigned int cnt[kShellRx];
#pragma unroll
    for (int i = 0; i < kShellRx; ++i) cnt[i] = 0;
    const int rows = L * L;
    for (int row = (int)threadIdx.x; row < rows; row += (int)blockDim.x) {
        const int y = row % L, z = row / L;
        const int prow = (y + ry) % L + L * ((z + rz) % L);
        unsigned long long src[NW], par[DW];
#pragma unroll
        for (int j = 0; j < NW; ++j) src[j] = qd[(size_t)row * DW + j];
#pragma unroll
        for (int j = 0; j < DW; ++j) par[j] = qd[(size_t)prow * DW + j];
#pragma unroll
        for (int i = 0; i < kShellRx; ++i) {
            const int rx = rx0 + i;  // uniform across the workgroup
            if (rx >= L) break;
            const int w0 = rx >> 6, off = rx & 63;
            unsigned int c = 0;
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                // words w0 + j and w0 + j + 1 of the doubled row (w0 is 0 or 1)
                unsigned long long lo = par[j], hi = j + 1 < DW ? par[j + 1] : 0ull;
                if (NW > 1 && w0 == 1) {
                    lo = par[j + 1];
                    hi = j + 2 < DW ? par[j + 2] : 0ull;
                }
                const unsigned long long win = off ? ((lo >> off) | (hi << (64 - off))) : lo;
                unsigned long long d = src[j] ^ win;
                if (j == NW - 1) d &= last_mask;
                c += (unsigned int)__popcll(d);
            }
            cnt[i] += c;
        }
    }
    // workgroup sums: within a wave by shuffles, then across the four waves
#pragma unroll
    for (int i = 0; i < kShellRx; ++i) {
        const uint32_t v = wave_sum(cnt[i]);
        if ((threadIdx.x & 63) == 0) part[i][threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x < kShellRx) {
        const int i = (int)threadIdx.x;
        const int rx = rx0 + i;
        const int k = kyz + min_image_sq(rx, L);
        if (rx < L && k < n_shells) {
            unsigned long long diff = 0;
            for (int w = 0; w < (int)(blockDim.x / 64); ++w) diff += part[i][w];
            const long long n = (long long)L * L * L;
            atomicAdd(shells + k, (unsigned long long)(n - 2 * (long long)diff));
        }
    }
}

// --------------------------------------------------------------------------
// The caller's int8 +-1 arrays in canonical order.  Eight consecutive x of a
// row are four half indices of each colour (even x: colour (y + z) & 1), and
// since words hold whole 4-site blocks, one nibble of one word per colour.
// Memory bound: 1 byte written or read per site (the conversion on the host,
// one division-laden address per site, took 80 ms per replica at L = 256).

// Bits 0..3 of even and odd as the bytes +1 / -1 of eight consecutive x.
__device__ __forceinline__ uint2 pm1_bytes(uint32_t even, uint32_t odd)
{
    uint32_t half[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t e = even >> (2 * i), o = odd >> (2 * i);
        const uint32_t bits = (e & 1u) | (o & 1u) << 8 | (e & 2u) << 15 | (o & 2u) << 23;
        half[i] = 0x01010101u + bits * 0xFEu;
    }
    return make_uint2(half[0], half[1]);
}

// The reverse: bit i set iff byte 2 i (even) or 2 i + 1 (odd) is negative.
__device__ __forceinline__ uint32_t pm1_nibble(uint2 b, int odd)
{
    const uint32_t lo = b.x >> (odd ? 15 : 7), hi = b.y >> (odd ? 15 : 7);
    return (lo & 1u) | (lo >> 15 & 2u) | (hi & 1u) << 2 | (hi >> 15 & 2u) << 2;
}

// Spins (ND = 1, planes = [colour][plane] of one replica) or couplings (ND =
// 3, planes = [direction][colour][plane]) of rows [row0, row0 + rows) to
// out[ND per site], from row row0 on.  One thread per eight x of a row.
template <int W, int ND>
__global__ __launch_bounds__(256) void to_pm1_kernel(const uint32_t *planes, Geom g, int row0, int rows, uint2 *out)
{
    const int per_row = g.L / 8, t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= rows * per_row) return;
    const int row = row0 + t / per_row, k = t % per_row;  // sites xh = 4k .. 4k + 3 of each colour
    const int y = row % g.L, z = row / g.L, w = 4 * k / W, shift = 4 * k - w * W;
    const size_t at = (size_t)row * g.RW + (size_t)w;
    uint2 v[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        const uint32_t even = planes[plane_off(g, d, (y + z) & 1) + at] >> shift;
        const uint32_t odd = planes[plane_off(g, d, (y + z + 1) & 1) + at] >> shift;
        v[d] = pm1_bytes(even, odd);
    }
    if constexpr (ND == 1) {
        out[t] = v[0];
    } else {
        // byte 3 x + d of the 24 is byte x of direction d
        uint32_t b[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            b[i] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int x = (4 * i + j) / 3, d = (4 * i + j) % 3;
                b[i] |= ((x < 4 ? v[d].x >> (8 * x) : v[d].y >> (8 * (x - 4))) & 0xffu) << (8 * j);
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) out[(size_t)3 * t + i] = make_uint2(b[2 * i], b[2 * i + 1]);
    }
}

// The reverse, one thread per packed word of both colours: rows [row0, row0 +
// rows) of `in` (values +-1, checked by the caller) to the planes.
template <int W, int ND>
__global__ __launch_bounds__(256) void from_pm1_kernel(uint32_t *planes, Geom g, int row0, int rows, const uint2 *in)
{
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= rows * g.RW) return;
    const int lrow = t / g.RW, w = t - lrow * g.RW, row = row0 + lrow;
    const int y = row % g.L, z = row / g.L;
    uint32_t bits[ND][2];
#pragma unroll
    for (int d = 0; d < ND; ++d) bits[d][0] = bits[d][1] = 0u;
#pragma unroll
    for (int j = 0; j < W / 4; ++j) {
        const size_t src = (size_t)lrow * (g.L / 8) + (size_t)(w * (W / 4) + j);
        if constexpr (ND == 1) {
            const uint2 b = in[src];
            bits[0][0] |= pm1_nibble(b, 0) << (4 * j);
            bits[0][1] |= pm1_nibble(b, 1) << (4 * j);
        } else {
            uint32_t b[6];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const uint2 q = in[3 * src + i];
                b[2 * i] = q.x;
                b[2 * i + 1] = q.y;
            }
#pragma unroll
            for (int x = 0; x < 8; ++x)
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    const int i = 3 * x + d;
                    bits[d][x & 1] |= (b[i / 4] >> (8 * (i % 4) + 7) & 1u) << (4 * j + x / 2);
                }
        }
    }
    const size_t at = (size_t)row * g.RW + (size_t)w;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        planes[plane_off(g, d, (y + z) & 1) + at] = bits[d][0];
        planes[plane_off(g, d, (y + z + 1) & 1) + at] = bits[d][1];
    }
}

// Plain word copy (snapshots) and fill (clearing counters); kernels rather
// than runtime memset/memcpy so that the same work can sit in a graph.
__global__ __launch_bounds__(256) void copy_words_kernel(uint32_t *dst, const uint32_t *src, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void zero_u64_kernel(unsigned long long *dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0ull;
}

__global__ __launch_bounds__(256) void zero_u32_kernel(uint32_t *dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0u;
}

// Device-side sweep counter: set it, or advance it after a block of sweeps.
__global__ void set_u32_kernel(uint32_t *dst, uint32_t v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *dst = v;
}

__global__ void advance_u32_kernel(uint32_t *dst, uint32_t k)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *dst += k;
}

}  // namespace ea
