// ea_fft.h -- full-vector C4 shells (eq. 3 over every displacement r)
// through the Wiener-Khinchin theorem, for L = 2^k (8 .. 256) and L = 3 2^k
// (24 .. 192), and in a run-time form at the end of this file for the other
// multiples of 8: with F the 3D DFT of q = S_0 S_1, the unnormalised inverse DFT
// of |F|^2 is N sum_x q(x) q(x + r) for every r at once.  Five passes over a
// complex fp64 array of L^2 rows of L/2 + 1 elements, each transforming whole lines
// of one axis in LDS, replace the direct kernel's L^6 / 64 word operations by
// O(L^3 log L) flops and 50 bytes of HBM traffic per site (56 with the
// rows' padding at L = 128).  q is real, so
// only the columns kx <= L/2 are kept between the passes along x, and those
// two passes transform two real rows as one complex line.  At L = 128 the five
// passes take 69 us (79 with all columns), a whole call among others 122 (158);
// each workgroup's chain of load, transform and store bounds them, at 1.1 to 2.9
// TB/s.
//
// The forward transforms are decimation in frequency (natural order in,
// digit-reversed order out along each axis: for L = 3P a radix-3 stage of
// span P first, then radix-2 stages on each third) and the inverse ones
// decimation in time (digit-reversed in, natural out: the same stages in the
// opposite order); |F|^2 is taken pointwise in between, so only the passes
// along x, which pair kx with L - kx, look an index up.  The autocorrelation is
// even, so the last two passes transform only the planes z <= L/2.  The sums are integers of magnitude <= N and the
// rounding error of the fp64 transforms is ~1e-16 log2(N) of the largest
// |F|^2 (<= N^2), i.e. below 1e-7 after the division by N at L = 256: each
// sum is rounded to the nearest integer, and a sum found farther than 1/4
// from an integer sets an error word instead of being trusted.
#pragma once

#include <hip/hip_runtime.h>

namespace ea {

constexpr int kFftTile = 2048;  // complex elements held by one workgroup, at most
constexpr int kFftThreads = 256;

// The passes, in order: forward along x from the dense q rows
// (fft_bits_kernel), forward along y, forward along z + |.|^2 + inverse along
// z, inverse along y, inverse along x + rounding (fft_bin_kernel); then the
// shell sums (fft_shell_sum_kernel).
enum FftOp { kFftFwdY = 1, kFftSquareZ = 2, kFftInvY = 3 };  // the passes along y and z

struct FftArgs {
    double2 *z;                    // element (kx <= L/2, y, z) at (z L + y) fft_stride(L) + kx
    const unsigned long long *qd;  // dense overlap rows (dense_q_kernel): row y + L z, dw words, bit x set iff q = -1
    int dw;
    int n_shells;
    unsigned long long *shells;  // [n_shells] sums; [0] = kFftBad if *err
    unsigned int *err;           // set to 1 if a sum is not within 1/4 of an integer
};

constexpr unsigned long long kFftBad = 1ull << 63;

constexpr bool fft_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }
constexpr int fft_log2(int n) { return n <= 1 ? 0 : 1 + fft_log2(n / 2); }

// Sides the route takes: 2^k for k = 3 .. 8 and 3 2^k for k = 3 .. 6.
constexpr bool fft_side(int L)
{
    return L >= 8 && L <= 256 && (fft_pow2(L) || (L % 3 == 0 && fft_pow2(L / 3) && L / 3 >= 8));
}

// Lines per workgroup tile: the largest power of two B that divides L (so
// that a row holds whole tiles along x), with B <= L and B L <= kFftTile.
constexpr int fft_lines_per_tile(int L)
{
    int b = 1;
    while (L % (2 * b) == 0 && 2 * b <= L && 2 * b * L <= kFftTile) b *= 2;
    return b;
}

template <int L>
struct FftShape {
    static_assert(fft_side(L), "L = 2^k (8 .. 256) or 3 2^k (24 .. 192)");
    static constexpr bool R3 = !fft_pow2(L);    // one radix-3 stage
    static constexpr int P = R3 ? L / 3 : L;    // the power-of-two blocks of the radix-2 stages
    static constexpr int LOG2P = fft_log2(P);
    static constexpr int SC = L / P;            // stride of a P-point twiddle in the L-point table
    static constexpr int NTW = R3 ? L : L / 2;  // twiddle table entries
    static constexpr int B = fft_lines_per_tile(L);
    static constexpr int LP = L + 1;  // LDS stride of a line (padded against bank conflicts)
};

__device__ __forceinline__ double2 cmul(double2 a, double2 w)
{
    return make_double2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}

__device__ __forceinline__ double2 cmulc(double2 a, double2 w)  // a conj(w)
{
    return make_double2(a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y);
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// The P-point block sb of a tile of lines: block r of line b starts at
// b LP + r P.
template <int L>
__device__ __forceinline__ int fft_block_base(int sb)
{
    using S = FftShape<L>;
    return (sb / S::SC) * S::LP + (sb % S::SC) * S::P;
}

// One radix-2 stage of span h = 2^st on every P-point block of the NL lines.
// DIF: (a, b) -> (a + b, (a - b) w); DIT: t = b conj(w), (a, b) -> (a + t,
// a - t); w = exp(-2 pi i pos / 2h), from the table tw[m] = exp(-2 pi i m / L)
// at m = SC pos P / 2h.
template <int L, int NL, bool DIT>
__device__ __forceinline__ void fft_stage2(double2 *s, const double2 *tw, int st, int tid)
{
    using S = FftShape<L>;
    constexpr int H = S::P / 2;
    const int h = 1 << st;
    for (int t = tid; t < NL * S::SC * H; t += kFftThreads) {
        const int sb = t >> (S::LOG2P - 1), kk = t & (H - 1);
        const int pos = kk & (h - 1);
        double2 *p0 = s + fft_block_base<L>(sb) + (((kk >> st) << (st + 1)) | pos), *p1 = p0 + h;
        const double2 w = tw[S::SC * (pos << (S::LOG2P - 1 - st))];
        const double2 x0 = *p0, x1 = *p1;
        if constexpr (DIT) {
            const double2 u = cmulc(x1, w);
            *p0 = cadd(x0, u);
            *p1 = csub(x0, u);
        } else {
            *p0 = cadd(x0, x1);
            *p1 = cmul(csub(x0, x1), w);
        }
    }
}

// Two radix-2 stages, of spans 2h and h (h = 2^sl), in registers on each
// quad {p, p + h, p + 2h, p + 3h}, p = g 4h + pos, pos < h, of a P-point
// block: the span-2h butterflies pair (p, p + 2h) at position pos and
// (p + h, p + 3h) at pos + h, the span-h ones (p, p + h) and (p + 2h, p + 3h),
// both at pos.  DIF takes span 2h first, DIT span h first; the same as the
// two radix-2 stages in turn, with half the LDS traffic and barriers.
template <int L, int NL, bool DIT>
__device__ __forceinline__ void fft_stage4(double2 *s, const double2 *tw, int sl, int tid)
{
    using S = FftShape<L>;
    constexpr int Q = S::P / 4;
    const int h = 1 << sl;
    for (int t = tid; t < NL * S::SC * Q; t += kFftThreads) {
        const int sb = t >> (S::LOG2P - 2), kk = t & (Q - 1);
        const int pos = kk & (h - 1);
        double2 *p = s + fft_block_base<L>(sb) + (((kk >> sl) << (sl + 2)) | pos);
        const double2 wa0 = tw[S::SC * (pos << (S::LOG2P - 2 - sl))];
        const double2 wa1 = tw[S::SC * ((pos + h) << (S::LOG2P - 2 - sl))];
        const double2 wb = tw[S::SC * (pos << (S::LOG2P - 1 - sl))];
        const double2 x0 = p[0], x1 = p[h], x2 = p[2 * h], x3 = p[3 * h];
        if constexpr (DIT) {
            const double2 u1 = cmulc(x1, wb), u3 = cmulc(x3, wb);
            const double2 y0 = cadd(x0, u1), y1 = csub(x0, u1), y2 = cadd(x2, u3), y3 = csub(x2, u3);
            const double2 v2 = cmulc(y2, wa0), v3 = cmulc(y3, wa1);
            p[0] = cadd(y0, v2);
            p[2 * h] = csub(y0, v2);
            p[h] = cadd(y1, v3);
            p[3 * h] = csub(y1, v3);
        } else {
            const double2 y0 = cadd(x0, x2), y2 = cmul(csub(x0, x2), wa0);
            const double2 y1 = cadd(x1, x3), y3 = cmul(csub(x1, x3), wa1);
            p[0] = cadd(y0, y1);
            p[h] = cmul(csub(y0, y1), wb);
            p[2 * h] = cadd(y2, y3);
            p[3 * h] = cmul(csub(y2, y3), wb);
        }
    }
}

// Three radix-2 stages, of spans 4h, 2h and h (h = 2^sl), in registers on
// each octet {p + m h : m = 0 .. 7}, p = g 8h + pos, pos < h, of a P-point
// block: span 4h pairs (m, m + 4) at positions pos + m h, span 2h pairs
// (m, m + 2) of each half at pos + (m & 1) h, span h pairs (m, m + 1) at
// pos.  DIF takes the spans in decreasing order, DIT in increasing order;
// the same as the three radix-2 stages in turn, with a third of their LDS
// round trips and barriers.
template <int L, int NL, bool DIT>
__device__ __forceinline__ void fft_stage8(double2 *s, const double2 *tw, int sl, int tid)
{
    using S = FftShape<L>;
    constexpr int O = S::P / 8;
    const int h = 1 << sl;
    for (int t = tid; t < NL * S::SC * O; t += kFftThreads) {
        const int sb = t >> (S::LOG2P - 3), kk = t & (O - 1);
        const int pos = kk & (h - 1);
        double2 *p = s + fft_block_base<L>(sb) + (((kk >> sl) << (sl + 3)) | pos);
        double2 x[8], wa[4], wb[2];
#pragma unroll
        for (int m = 0; m < 8; ++m) x[m] = p[m * h];
#pragma unroll
        for (int m = 0; m < 4; ++m) wa[m] = tw[S::SC * ((pos + m * h) << (S::LOG2P - 3 - sl))];
#pragma unroll
        for (int m = 0; m < 2; ++m) wb[m] = tw[S::SC * ((pos + m * h) << (S::LOG2P - 2 - sl))];
        const double2 wc = tw[S::SC * (pos << (S::LOG2P - 1 - sl))];
        if constexpr (DIT) {
#pragma unroll
            for (int m = 0; m < 8; m += 2) {
                const double2 u = cmulc(x[m + 1], wc);
                x[m + 1] = csub(x[m], u);
                x[m] = cadd(x[m], u);
            }
#pragma unroll
            for (int m = 0; m < 8; m += (m & 1) ? 3 : 1) {  // 0, 1, 4, 5
                const double2 u = cmulc(x[m + 2], wb[m & 1]);
                x[m + 2] = csub(x[m], u);
                x[m] = cadd(x[m], u);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double2 u = cmulc(x[m + 4], wa[m]);
                x[m + 4] = csub(x[m], u);
                x[m] = cadd(x[m], u);
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double2 a = x[m], b = x[m + 4];
                x[m] = cadd(a, b);
                x[m + 4] = cmul(csub(a, b), wa[m]);
            }
#pragma unroll
            for (int m = 0; m < 8; m += (m & 1) ? 3 : 1) {  // 0, 1, 4, 5
                const double2 a = x[m], b = x[m + 2];
                x[m] = cadd(a, b);
                x[m + 2] = cmul(csub(a, b), wb[m & 1]);
            }
#pragma unroll
            for (int m = 0; m < 8; m += 2) {
                const double2 a = x[m], b = x[m + 1];
                x[m] = cadd(a, b);
                x[m + 1] = cmul(csub(a, b), wc);
            }
        }
#pragma unroll
        for (int m = 0; m < 8; ++m) p[m * h] = x[m];
    }
}

// The radix-3 stage of span P = L / 3 on each line: (x0, x1, x2) at
// (pos, pos + P, pos + 2P).  With w3 = exp(-2 pi i / 3) and W = exp(-2 pi i
// / L), DIF writes x0 + x1 + x2, (x0 + w3 x1 + w3^2 x2) W^pos and (x0 + w3^2 x1
// + w3 x2) W^2pos; DIT takes z1 = x1 conj(W^pos), z2 = x2 conj(W^2pos) and
// writes x0 + z1 + z2, x0 + conj(w3) z1 + w3 z2 and x0 + w3 z1 + conj(w3) z2.
template <int L, int NL, bool DIT>
__device__ __forceinline__ void fft_stage3(double2 *s, const double2 *tw, int tid)
{
    using S = FftShape<L>;
    constexpr int P = S::P;
    constexpr double kS3 = 0.86602540378443864676;  // sqrt(3) / 2
    for (int t = tid; t < NL * P; t += kFftThreads) {
        const int b = t / P, pos = t - b * P;
        double2 *p = s + b * S::LP + pos;
        const double2 w1 = tw[pos], w2 = tw[2 * pos];
        double2 x0 = p[0], x1 = p[P], x2 = p[2 * P];
        if constexpr (DIT) {
            x1 = cmulc(x1, w1);
            x2 = cmulc(x2, w2);
        }
        const double2 t1 = cadd(x1, x2), t2 = csub(x1, x2);
        const double2 u = make_double2(x0.x - 0.5 * t1.x, x0.y - 0.5 * t1.y);
        // DIF: -i sqrt(3)/2 (x1 - x2); DIT: +i sqrt(3)/2 (x1 - x2)
        const double2 v = DIT ? make_double2(-kS3 * t2.y, kS3 * t2.x) : make_double2(kS3 * t2.y, -kS3 * t2.x);
        p[0] = cadd(x0, t1);
        if constexpr (DIT) {
            p[P] = cadd(u, v);
            p[2 * P] = csub(u, v);
        } else {
            p[P] = cmul(cadd(u, v), w1);
            p[2 * P] = cmul(csub(u, v), w2);
        }
    }
}

// The whole transform of the NL lines; ends with a barrier.  DIF: the
// radix-3 stage (L = 3P), then spans P/2 .. 1 on each P-point block, three
// stages per round, the last one or two in a radix-4 or radix-2 round; DIT:
// the same rounds in the opposite order, then the radix-3 stage.
template <int L, int NL, bool DIT>
__device__ __forceinline__ void fft_lines(double2 *s, const double2 *tw, int tid)
{
    using S = FftShape<L>;
    constexpr int LOG2P = S::LOG2P;
    if constexpr (DIT) {
        // the mirror of the DIF grouping: the radix-2 or radix-4 remainder on
        // the smallest spans first, then radix-8 rounds
        int st = 0;
        if constexpr (LOG2P % 3 == 1) {
            fft_stage2<L, NL, true>(s, tw, 0, tid);
            __syncthreads();
            st = 1;
        } else if constexpr (LOG2P % 3 == 2) {
            fft_stage4<L, NL, true>(s, tw, 0, tid);
            __syncthreads();
            st = 2;
        }
        for (; st + 2 < LOG2P; st += 3) {
            fft_stage8<L, NL, true>(s, tw, st, tid);
            __syncthreads();
        }
        if constexpr (S::R3) {
            fft_stage3<L, NL, true>(s, tw, tid);
            __syncthreads();
        }
    } else {
        if constexpr (S::R3) {
            fft_stage3<L, NL, false>(s, tw, tid);
            __syncthreads();
        }
        int st = LOG2P - 1;
        for (; st >= 2; st -= 3) {
            fft_stage8<L, NL, false>(s, tw, st - 2, tid);
            __syncthreads();
        }
        if (st >= 1) {
            fft_stage4<L, NL, false>(s, tw, st - 1, tid);
            __syncthreads();
            st -= 2;
        }
        if (st == 0) {
            fft_stage2<L, NL, false>(s, tw, 0, tid);
            __syncthreads();
        }
    }
}

// tw[m] = exp(-2 pi i m / L), m < NTW; the caller synchronises.
template <int L>
__device__ __forceinline__ void fft_twiddles(double2 *tw, int tid)
{
    for (int m = tid; m < FftShape<L>::NTW; m += kFftThreads) {
        double sn, cs;
        sincospi(2.0 * (double)m / (double)L, &sn, &cs);
        tw[m] = make_double2(cs, -sn);
    }
}

// Elements from row to row: L/2 + 1 of them hold data.  A multiple of 128
// bytes, so that the runs of eight columns that passes along y and z read and
// write are whole cache lines (rows of L/2 + 1: the passes along y of L = 128
// 14.9 and 13.4 us, now 13.0 and 11.2).
__host__ __device__ constexpr int fft_stride(int L) { return (L / 2 + 8) / 8 * 8; }

// Where the forward transform leaves X[k].
template <int L>
__device__ __forceinline__ int fft_place(int k)
{
    using S = FftShape<L>;
    const int r = S::R3 ? k % 3 : 0, j = S::R3 ? k / 3 : k;
    return r * S::P + (int)(__brev((unsigned)j) >> (32 - S::LOG2P));
}

// Element i of line `line` of a pass along y (z): the lines are the columns
// of every z (y), so consecutive lines are consecutive in memory.
template <int OP>
__device__ __forceinline__ size_t fft_element(int L, int line, int i)
{
    const int S = fft_stride(L), o = line / S, x = line - o * S;
    return ((size_t)(OP == kFftSquareZ ? i * L + o : o * L + i)) * S + x;
}

// Lines of such a pass, padding included: kFftInvY needs only the planes z <= L/2 (and
// kFftSquareZ stores only those): the autocorrelation is even, A(-r) = A(r),
// so the shells follow from half of it (fft_bin_kernel).
template <int OP>
__host__ __device__ constexpr int fft_n_lines(int L)
{
    return (OP == kFftInvY ? L / 2 + 1 : L) * fft_stride(L);
}

// Does the line hold data (kx <= L/2, and inside the array)?
template <int OP>
__device__ __forceinline__ bool fft_line_ok(int L, int line)
{
    return line < fft_n_lines<OP>(L) && line % fft_stride(L) <= L / 2;
}

// The two real rows' columns k of a packed line: Zk = Z[k], Zm = Z[L - k].
__device__ __forceinline__ double2 fft_unpack(double2 zk, double2 zm, bool second)
{
    return second ? make_double2(0.5 * (zk.y + zm.y), -0.5 * (zk.x - zm.x))
                  : make_double2(0.5 * (zk.x + zm.x), 0.5 * (zk.y - zm.y));
}

// The tile of the first pass before its transform: 2 B rows, packed in
// pairs as complex lines LP apart.  Their words come through LDS: read where
// the sites are expanded they were a chain of loads (the pass at L = 128 took
// 19 us).
__device__ __forceinline__ void fft_bits(const FftArgs &a, int L, int B, int LP, double2 *s, int tid)
{
    __shared__ unsigned long long rows[256];
    const int nw = (L + 63) / 64, n = 2 * B * nw;  // 64 at most
    if (tid < n) rows[tid] = a.qd[((size_t)blockIdx.x * 2 * B + (size_t)(tid / nw)) * (size_t)a.dw + (size_t)(tid % nw)];
    __syncthreads();
    for (int j = tid; j < B * L; j += kFftThreads) {
        const int line = j / L, i = j - line * L;
        const unsigned long long *q = rows + 2 * line * nw + (i >> 6);
        s[line * LP + i] =
            make_double2((q[0] >> (i & 63)) & 1ull ? -1.0 : 1.0, (q[nw] >> (i & 63)) & 1ull ? -1.0 : 1.0);
    }
}

// The first pass also clears what the last ones add to.
__device__ __forceinline__ void fft_clear(const FftArgs &a, int tid)
{
    for (int k = (int)blockIdx.x * kFftThreads + tid; k < a.n_shells; k += (int)gridDim.x * kFftThreads)
        a.shells[k] = 0ull;
    if (blockIdx.x == 0 && tid == 0) *a.err = 0u;
}

// The first pass: 2 B rows per workgroup, transformed in pairs.
template <int L>
__global__ __launch_bounds__(kFftThreads) void fft_bits_kernel(FftArgs a)
{
    using S = FftShape<L>;
    constexpr int B = S::B, H1 = L / 2 + 1;
    __shared__ double2 s[B * S::LP];
    __shared__ double2 tw[S::NTW];
    const int tid = (int)threadIdx.x, w = (int)blockIdx.x;
    fft_clear(a, tid);
    fft_bits(a, L, B, S::LP, s, tid);
    fft_twiddles<L>(tw, tid);
    __syncthreads();
    fft_lines<L, B, false>(s, tw, tid);
    for (int j = tid; j < 2 * B * H1; j += kFftThreads) {
        const int row = j / H1, k = j - row * H1;
        const double2 *p = s + (row >> 1) * S::LP;
        a.z[((size_t)w * 2 * B + (size_t)row) * fft_stride(L) + (size_t)k] =
            fft_unpack(p[fft_place<L>(k)], p[fft_place<L>(k == 0 ? 0 : L - k)], row & 1);
    }
}

// Passes kFftFwdY .. kFftInvY, B lines per workgroup.  A thread's elements
// all belong to one line; they are on their way while the twiddles are
// computed.
template <int L, int OP>
__global__ __launch_bounds__(kFftThreads) void fft_pass_kernel(FftArgs a)
{
    using S = FftShape<L>;
    constexpr int B = S::B, IS = kFftThreads / B, PER = (L + IS - 1) / IS;
    static_assert(OP == kFftFwdY || OP == kFftSquareZ || OP == kFftInvY, "a pass along y or z");
    static_assert(kFftThreads % B == 0, "one line per thread");
    __shared__ double2 s[B * S::LP];
    __shared__ double2 tw[S::NTW];
    const int tid = (int)threadIdx.x, b = tid % B, i0 = tid / B, line = (int)blockIdx.x * B + b;
    const bool ok = fft_line_ok<OP>(L, line);

    double2 v[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int i = i0 + e * IS;
        v[e] = ok && i < L ? a.z[fft_element<OP>(L, line, i)] : make_double2(0.0, 0.0);
    }
    fft_twiddles<L>(tw, tid);
    double2 *p = s + b * S::LP;
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (i0 + e * IS < L) p[i0 + e * IS] = v[e];
    __syncthreads();

    if constexpr (OP == kFftInvY) {
        fft_lines<L, B, true>(s, tw, tid);
    } else {
        fft_lines<L, B, false>(s, tw, tid);
        if constexpr (OP == kFftSquareZ) {
            for (int i = i0; i < L; i += IS) p[i] = make_double2(p[i].x * p[i].x + p[i].y * p[i].y, 0.0);
            __syncthreads();
            fft_lines<L, B, true>(s, tw, tid);
        }
    }
    if (!ok) return;
    for (int i = i0; i < (OP == kFftSquareZ ? L / 2 + 1 : L); i += IS) a.z[fft_element<OP>(L, line, i)] = p[i];
}

constexpr int kFftBinY = 8;  // y values per workgroup of the last pass

// The sums T(i, y, z) of the last pass, one per |x| = i, |y|, |z| <= L/2,
// at [(z (L/2 + 1) + y) (L/2 + 1) + i], in the planes z > L/2 of the complex
// array (no pass reads those after kFftSquareZ; they hold at least 16 (L/2 - 1)
// L (L/2 + 1) bytes, more than the 8 (L/2 + 1)^3 needed).
__device__ __forceinline__ long long *fft_sums(double2 *z, int L)
{
    return reinterpret_cast<long long *>(z + (size_t)(L / 2 + 1) * L * fft_stride(L));
}

// Columns k and L - k of the line that packs the rows (y, z) and (L - y, z):
// b1 + i b2 and conj(b1) + i conj(b2).  Rows past L/2 and the mirror rows of
// y = 0 and L/2 are taken as 0.
__device__ __forceinline__ void fft_pack(const FftArgs &a, int L, int z, int y, int k, double2 &zk, double2 &zm)
{
    const int H = L / 2, S = fft_stride(L);
    const double2 *at = a.z + (size_t)z * L * S + (size_t)k;
    double2 b1 = make_double2(0.0, 0.0), b2 = b1;
    if (y <= H) b1 = at[(size_t)y * S];
    if (y > 0 && y < H) b2 = at[(size_t)(L - y) * S];
    zk = make_double2(b1.x - b2.y, b1.y + b2.x);
    zm = make_double2(b1.x + b2.y, b2.x - b1.y);
}

// T(i, y, z) from the transformed line p: the rounded sums at x = +-i of both
// rows (the real and the imaginary part), twice for 0 < z < L/2, where the
// row (L - y, L - z), not transformed, holds A(-x, y, z).
__device__ __forceinline__ void fft_bin(const FftArgs &a, int L, const double2 *p, int i, int y, int z, double n)
{
    const int H = L / 2;
    long long sum = 0;
    bool bad = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // bit 0: x -> L - x, bit 1: y -> L - y
        if ((e & 1) && (i == 0 || i == H)) continue;
        if ((e & 2) && (y == 0 || y == H)) continue;
        const double2 c = p[(e & 1) ? L - i : i];
        const double v = (e & 2 ? c.y : c.x) / n;
        const double r = rint(v);
        bad |= !(fabs(v - r) <= 0.25);  // NaN included
        sum += (long long)r;
    }
    if (bad) atomicOr(a.err, 1u);
    fft_sums(a.z, L)[((size_t)z * (H + 1) + (size_t)y) * (H + 1) + (size_t)i] = z == 0 || z == H ? sum : 2 * sum;
}

// The last transform pass, on the planes z = 0 .. L/2: a workgroup takes
// kFftBinY values y <= L/2 of one z and for each the rows y and L - y as one
// complex line, transforms them along x (DIT), and stores the sums over the
// minimum images (+-i, +-y, z).
template <int L>
__global__ __launch_bounds__(kFftThreads) void fft_bin_kernel(FftArgs a)
{
    using S = FftShape<L>;
    constexpr int H = L / 2, LP = S::LP, NL = kFftBinY, PER = (NL * (H + 1) + kFftThreads - 1) / kFftThreads;
    constexpr int YB = (H + 1 + NL - 1) / NL;  // workgroups per plane
    __shared__ double2 s[NL * LP];
    __shared__ double2 tw[S::NTW];
    const int tid = (int)threadIdx.x, w = (int)blockIdx.x;
    const int z = w / YB, y0 = (w - z * YB) * NL;

    double2 zk[PER], zm[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int j = tid + e * kFftThreads, line = j / (H + 1), k = j - line * (H + 1);
        if (line < NL) fft_pack(a, L, z, y0 + line, k, zk[e], zm[e]);
    }
    fft_twiddles<L>(tw, tid);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int j = tid + e * kFftThreads, line = j / (H + 1), k = j - line * (H + 1);
        if (line >= NL) break;
        s[line * LP + fft_place<L>(k)] = zk[e];
        if (k > 0 && k < H) s[line * LP + fft_place<L>(L - k)] = zm[e];
    }
    __syncthreads();
    fft_lines<L, NL, true>(s, tw, tid);
    for (int t = tid; t < NL * (H + 1); t += kFftThreads) {
        const int j = t / (H + 1), i = t - j * (H + 1), y = y0 + j;
        if (y <= H) fft_bin(a, L, s + j * LP, i, y, z, (double)L * L * L);
    }
}

// Shell sums from T: one thread per sorted triple p <= q <= r of |x|, |y|,
// |z| values adds T over the triple's distinct orderings (all of which lie in
// the shell p^2 + q^2 + r^2) in one atomic, a sixth as many as one per
// ordering.  One thread per point of the (L/2 + 1)^3 cube; the others return.
__global__ __launch_bounds__(256) void fft_shell_sum_kernel(FftArgs a, int L)
{
    const int H1 = L / 2 + 1;
    const long long *T = fft_sums(a.z, L);
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= H1 * H1 * H1) return;
    const int p = t % H1, q = (t / H1) % H1, r = t / (H1 * H1);
    if (p > q || q > r) return;
    const int k = p * p + q * q + r * r;
    if (k >= a.n_shells) return;
    auto at = [T, H1](int i, int y, int z) { return T[((size_t)z * H1 + (size_t)y) * H1 + (size_t)i]; };
    long long sum = at(p, q, r);
    if (p == q && q == r) {
        if (k == 0 && *a.err) sum = (long long)kFftBad;  // the only term of shell 0
    } else if (p == q) {  // (p, p, r): also (p, r, p), (r, p, p)
        sum += at(p, r, p) + at(r, p, p);
    } else if (q == r) {  // (p, q, q): also (q, p, q), (q, q, p)
        sum += at(q, p, q) + at(q, q, p);
    } else {
        sum += at(p, r, q) + at(q, p, r) + at(q, r, p) + at(r, p, q) + at(r, q, p);
    }
    atomicAdd(a.shells + k, (unsigned long long)sum);
}

// --------------------------------------------------------------------------
// The other sides, L = m P with m odd (5 .. 31) and P = 8, 16 or 32: the same
// passes with L at run time and each transform in two direct steps.  With
// position a P + b (a < m, b < P), forward: for every b the m-point sums over
// a, times exp(-2 pi i b k / L), at k P + b; then for every k the P-point sums
// over b, at k P + j -- X[k + m j] in an order of its own, which the inverse
// takes as it is: P-point over j, conjugate twiddle, m-point over k.  m + P
// complex multiply-adds an element and transform instead of L; the LDS reads
// of a wave's inputs bound it.  A call against the direct count: L = 72 0.10 ms
// (0.82), L = 136 0.22 (22).
struct FftGeneral {
    int L, m, P, B, LP;  // side = m P; lines per tile; LDS stride of a line
};

constexpr int kFftGeneralPer = 8;                              // elements per thread, at most
constexpr int kFftGeneralLds = kFftTile + kFftTile / 8;        // B lines of L + 1 elements: B (L + 1) <= 2048 + B

__host__ __device__ constexpr int fft_general_p(int L) { return L % 32 == 0 ? 32 : (L % 16 == 0 ? 16 : 8); }

// Sides of this form: multiples of 8 up to 256 that fft_side leaves out.
constexpr bool fft_general_side(int L)
{
    return L >= 8 && L <= 256 && L % 8 == 0 && !fft_side(L);
}

// Sum over i < n of s[base + i stride] w^(i step), w = exp(-+2 pi i / L).
template <bool INV>
__device__ __forceinline__ double2 fft_sum(const double2 *s, int n, int stride, const double2 *tw, int step, int L)
{
    double2 acc = s[0];
    int t = 0;
    for (int i = 1; i < n; ++i) {
        t += step;
        t -= t >= L ? L : 0;
        const double2 x = s[i * stride], w = tw[t];
        acc = cadd(acc, INV ? cmulc(x, w) : cmul(x, w));
    }
    return acc;
}

// The transform of the first n elements (whole lines) of the tile, in LDS;
// begins and ends with a barrier.  A step's outputs wait in registers until
// every thread has read its inputs.
template <bool INV>
__device__ __forceinline__ void fft_general_lines(double2 *s, const double2 *tw, const FftGeneral &f, int n, int tid)
{
    const int L = f.L, m = f.m, P = f.P;
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        const bool over_a = (half == 0) != INV;  // the m-point step: first forward, last backward
        double2 out[kFftGeneralPer];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kFftGeneralPer; ++e) {
            const int j = tid + e * kFftThreads;
            if (j >= n) break;
            const int line = j / L, i = j - line * L, hi = i / P, lo = i - hi * P;
            const double2 *p = s + line * f.LP;
            if (over_a) {
                // output (hi = k or a, lo = b): over the other m-index
                double2 v = fft_sum<INV>(p + lo, m, P, tw, hi * P, L);
                if constexpr (!INV) v = cmul(v, tw[lo * hi]);
                out[e] = v;
            } else {
                // output (hi = k, lo = j or b) over the other P-index
                double2 v = fft_sum<INV>(p + hi * P, P, 1, tw, lo * m, L);
                if constexpr (INV) v = cmulc(v, tw[lo * hi]);
                out[e] = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kFftGeneralPer; ++e) {
            const int j = tid + e * kFftThreads;
            if (j >= n) break;
            const int line = j / L;
            s[line * f.LP + (j - line * L)] = out[e];
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void fft_general_twiddles(double2 *tw, int L, int tid)
{
    for (int i = tid; i < L; i += kFftThreads) {
        double sn, cs;
        sincospi(2.0 * (double)i / (double)L, &sn, &cs);
        tw[i] = make_double2(cs, -sn);
    }
}

__device__ __forceinline__ int fft_general_place(const FftGeneral &f, int k) { return (k % f.m) * f.P + k / f.m; }

// The first pass (fft_bits_kernel).
__global__ __launch_bounds__(kFftThreads) void fft_general_bits_kernel(FftArgs a, FftGeneral f)
{
    __shared__ double2 s[kFftGeneralLds];
    __shared__ double2 tw[256];
    const int tid = (int)threadIdx.x, w = (int)blockIdx.x;
    const int L = f.L, B = f.B, H1 = L / 2 + 1;
    fft_clear(a, tid);
    fft_bits(a, L, B, f.LP, s, tid);
    fft_general_twiddles(tw, L, tid);
    fft_general_lines<false>(s, tw, f, B * L, tid);
    for (int j = tid; j < 2 * B * H1; j += kFftThreads) {
        const int row = j / H1, k = j - row * H1;
        const double2 *p = s + (row >> 1) * f.LP;
        a.z[((size_t)w * 2 * B + (size_t)row) * fft_stride(L) + (size_t)k] =
            fft_unpack(p[fft_general_place(f, k)], p[fft_general_place(f, k == 0 ? 0 : L - k)], row & 1);
    }
}

// Passes kFftFwdY .. kFftInvY (fft_pass_kernel).
template <int OP>
__global__ __launch_bounds__(kFftThreads) void fft_general_pass_kernel(FftArgs a, FftGeneral f)
{
    __shared__ double2 s[kFftGeneralLds];
    __shared__ double2 tw[256];
    const int L = f.L, B = f.B, is = kFftThreads / B;
    const int tid = (int)threadIdx.x, b = tid % B, i0 = tid / B, line = (int)blockIdx.x * B + b;
    const bool ok = fft_line_ok<OP>(L, line);
    double2 v[kFftGeneralPer];
#pragma unroll
    for (int e = 0; e < kFftGeneralPer; ++e) {
        const int i = i0 + e * is;
        v[e] = ok && i < L ? a.z[fft_element<OP>(L, line, i)] : make_double2(0.0, 0.0);
    }
    fft_general_twiddles(tw, L, tid);
    double2 *p = s + b * f.LP;
#pragma unroll
    for (int e = 0; e < kFftGeneralPer; ++e)
        if (i0 + e * is < L) p[i0 + e * is] = v[e];
    if constexpr (OP == kFftInvY) {
        fft_general_lines<true>(s, tw, f, B * L, tid);
    } else {
        fft_general_lines<false>(s, tw, f, B * L, tid);
        if constexpr (OP == kFftSquareZ) {
            for (int i = i0; i < L; i += is) p[i] = make_double2(p[i].x * p[i].x + p[i].y * p[i].y, 0.0);
            fft_general_lines<true>(s, tw, f, B * L, tid);
        }
    }
    if (!ok) return;
    for (int i = i0; i < (OP == kFftSquareZ ? L / 2 + 1 : L); i += is) a.z[fft_element<OP>(L, line, i)] = p[i];
}

// The last transform pass (fft_bin_kernel).
__global__ __launch_bounds__(kFftThreads) void fft_general_bin_kernel(FftArgs a, FftGeneral f)
{
    __shared__ double2 s[kFftGeneralLds];
    __shared__ double2 tw[256];
    const int tid = (int)threadIdx.x, w = (int)blockIdx.x;
    const int L = f.L, H = L / 2, yb = (H + kFftBinY) / kFftBinY;
    const int z = w / yb, y0 = (w - z * yb) * kFftBinY;
    fft_general_twiddles(tw, L, tid);
    for (int j = tid; j < kFftBinY * (H + 1); j += kFftThreads) {
        const int line = j / (H + 1), k = j - line * (H + 1);
        double2 zk, zm;
        fft_pack(a, L, z, y0 + line, k, zk, zm);
        s[line * f.LP + fft_general_place(f, k)] = zk;
        if (k > 0 && k < H) s[line * f.LP + fft_general_place(f, L - k)] = zm;
    }
    fft_general_lines<true>(s, tw, f, kFftBinY * L, tid);
    for (int t = tid; t < kFftBinY * (H + 1); t += kFftThreads) {
        const int j = t / (H + 1), i = t - j * (H + 1), y = y0 + j;
        if (y <= H) fft_bin(a, L, s + j * f.LP, i, y, z, (double)L * L * L);
    }
}

}  // namespace ea
