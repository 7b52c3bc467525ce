// ea_batch_kernels.h -- the batched form: one persistent launch runs many
// independent samples of different size, temperature and coupling
// probability.  Each workgroup owns one replica of one sample ("unit") for
// the whole span of sweeps it is given: the replica's spins and the sample's
// couplings sit in LDS, the checkerboard half-steps are separated by
// workgroup barriers instead of kernel launches, and the scheduled snapshots
// and measurements are taken inside the kernel.
//
// The two replicas of a sample never interact, so they run in separate
// workgroups.  Observables of one replica (energy, magnetisation, C(t, t_w))
// are reduced by its own workgroup; the replica-pair observables (overlap and
// C4) need both configurations at the same time t: each workgroup publishes
// its configuration at a measurement time, and whichever arrives second
// computes them from the two published copies.
#pragma once

#include "ea_kernels.h"

namespace ea {

constexpr int kBatchThreads = 1024;
constexpr int kBatchMaxL = 64;
constexpr int kSplitMinL = 48;  // smallest size whose replicas may be split into two z-slabs

__host__ __device__ constexpr int words_per_row_c(int R)
{
    int rw = (R + 31) / 32;
    while ((R / 4) % rw != 0) ++rw;
    return rw;
}

// The next finer valid packing of a row of R sites: the smallest word count
// above rw that splits the row into whole 4-site blocks (0 if none).
__host__ __device__ constexpr int finer_words_per_row_c(int R, int rw)
{
    for (int d = rw + 1; d <= R / 4; ++d)
        if ((R / 4) % d == 0) return d;
    return 0;
}

// Compile-time geometry of one lattice size and row packing.
template <int L, int RW>
struct Shape {
    static constexpr int R = L / 2;
    static constexpr int W = R / RW;
    static constexpr int POS = L * L * RW;  // packed words per colour
    static constexpr int LATTICE_WORDS = 8 * POS;  // 2 spin planes + 6 coupling planes
    static constexpr int LDS_WORDS = LATTICE_WORDS + 16;  // dynamic LDS: lattice + flag
    static_assert(R % RW == 0 && W % 4 == 0 && W <= 32, "invalid row packing");
};

// Threshold select of the update: through the LDS tables or with register
// bit-field selects.
enum : int { SEL_LDS = 0, SEL_REG = 1 };

constexpr int kBatchPubs = 8;  // publication counters of a split job: [replica][slab][face]

// Device-side description of one sample in a batch.
struct BatchJobDev {
    int32_t L;
    int32_t rw;   // words per row of the packed layout
    int32_t nt;   // threads of the workgroup that work (multiple of 64, <= kBatchThreads)
    int32_t sel;  // SEL_LDS or SEL_REG
    uint32_t k0, k1, sample;
    uint32_t thr1, thr2, thr3;
    uint64_t pcut;
    int32_t n_meas, n_tw, obs_stride;
    uint32_t *spins;          // [replica][colour][POS]: state between launches
    const uint32_t *bonds;    // [direction][colour][POS]
    uint32_t *snaps;          // [slot][replica][colour][POS]
    uint32_t *mspins;         // [measurement][replica][colour][POS]
    const uint32_t *meas_t;   // [n_meas], strictly increasing
    const uint32_t *tw_t;     // [n_tw], strictly increasing
    unsigned long long *obs;  // [n_meas][obs_stride]
    uint32_t *arrive;         // [n_meas] workgroups that reached the measurement
    uint32_t *t_now;          // [2] sweeps done per replica
    int32_t parts;            // workgroups per replica: 1, or 2 for a replica split into z-slabs
    uint32_t *xbuf;           // split: [replica][slab][sweep parity][colour][first/last plane][L * rw]
    unsigned long long *pub;  // split: [replica][slab][face] publications (slab_pub)
    uint32_t *err;            // set when a split pair gave up waiting for its partner
};

// One workgroup's work: replica `replica` of job `job` from its current time
// up to t_stop.
struct BatchUnit {
    int32_t job;
    int32_t replica;
    uint32_t t_stop;
    int32_t first;  // 1 on the job's first span: events at t = 0 are taken too
    int32_t slab;   // split jobs: which z-slab (0 or 1); 0 otherwise
};

// Observable slots of one measurement (popcounts, like the plain form):
// [0,1] unsatisfied bonds, [2,3] spins down, [4] S_0 != S_1,
// [5 + 2k + r] S_r(t) != S_r(tw_k), then [5 + 2 n_tw + d (R+1) + rho] for C4.
__device__ __forceinline__ int batch_c4_base(int n_tw) { return M_AUTO + 2 * n_tw; }

// The workgroup's LDS: the threshold-select tables are a static array (its
// address is a compile-time constant, so table reads need no address add),
// followed by the dynamic part: [colour][POS] spins of the replica,
// [direction][colour][POS] couplings and one word for a broadcast flag.
// Declared at file scope so that every access is a plain ds_read/ds_write.
extern __shared__ uint32_t batch_lds[];
__shared__ __align__(16) uint32_t batch_select_tables[kSelectTableWords];

__device__ __forceinline__ uint32_t *batch_tables() { return batch_select_tables; }

template <class S>
__device__ __forceinline__ uint32_t *lds_spin(int c)
{
    return batch_lds + c * S::POS;
}

template <class S>
__device__ __forceinline__ uint32_t *lds_bond(int d, int c)
{
    return batch_lds + (2 + 2 * d + c) * S::POS;
}

// Update the colour-C words of this workgroup's replica (eq. 9), reading the
// other colour and the couplings from LDS.  The colour is a template
// argument so that every plane's LDS offset is a compile-time constant.
// Bound by VALU issue: the multiplies of a 32-site word's eight Philox blocks
// alone take 128 x 4.3 cycles of its SIMD, its other ~260 instructions as
// much again where they pair perfectly (ea_device.h), 1110 cycles in all.
// Measured per half-step on a full CU: L = 64 9.3 us (1390 cycles per word
// and wave; 11.35 before the multiplies, compares and XORs ran in phases and
// the addresses advanced with z), L = 48 4.5 (5.43), L = 32 1.63 (1.81),
// L = 24 1.05 (1.16).
template <int L, int RW, int SEL, int C>
__device__ __forceinline__ void batch_half_step(const BatchJobDev &J, int r, uint32_t t)
{
    using S = Shape<L, RW>;
    constexpr int W = S::W;
    constexpr int c = C;
    const PhiloxStep<true> step = philox_step(t, counter_word2(TAG_METRO, (uint32_t)c, (uint32_t)r), J.sample, J.k0, J.k1);
    // Recompute the addresses every half-step: hoisting them out of the
    // sweep loop would keep some thirty address registers live and spill.
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    // Each thread keeps one (y, w) column and walks nz consecutive z-planes
    // of it (threads past the last whole column stay idle): the y and x
    // neighbour offsets are computed once per half-step, the word above
    // becomes the next word, and the addresses advance by one plane.  One
    // word at a time: a word already carries W/4 independent Philox blocks of
    // instruction-level parallelism, and unrolling further spills.
    constexpr unsigned PLANE = (unsigned)(L * RW);
    const unsigned groups = (unsigned)J.nt / PLANE, nz = ((unsigned)L + groups - 1) / groups;
    const unsigned q = (unsigned)tid % PLANE, zg = (unsigned)tid / PLANE;
    if (zg >= groups) return;
    const unsigned w = q % RW;
    const unsigned y = q / RW;
    unsigned z = zg * nz;
    const unsigned z_end = min(z + nz, (unsigned)L);
    if constexpr (PLANE % 64 == 0) z = (unsigned)__builtin_amdgcn_readfirstlane((int)z);  // whole waves share a plane
    if (z >= z_end) return;
    // byte offsets from the word to the row's neighbour words (RW > 1) and rows
    const int qm = 4 * (w == 0 ? RW - 1 : -1), qp = 4 * (w == RW - 1 ? 1 - RW : 1);
    const int qym = 4 * (y == 0 ? (L - 1) * RW : -RW), qyp = 4 * (y == L - 1 ? -(L - 1) * RW : RW);
    uint32_t odd = 0u - ((y + z + (unsigned)c) & 1u);  // all ones where x = 2 xh + 1
    // counter word 1 of the word's first block: (row R + w W) / 4, row = y + L z
    uint32_t quad0 = ((y * S::R + w * W) >> 2) + z * (unsigned)(L * S::R / 4);
    // The word's place in the spin and x-coupling planes (lo) and in the y-
    // and z-coupling planes (hi); two addresses, because one LDS access
    // reaches 64 KiB from its address register.
    constexpr int STEP = 4 * (int)PLANE;
    const int p0 = 4 * (int)(z * PLANE + q), below = z == 0 ? (L - 1) * STEP : -STEP;
    char *lo = reinterpret_cast<char *>(batch_lds) + p0;
    const char *hi = reinterpret_cast<char *>(batch_lds) + 16 * S::POS + p0;
    const char *hi_zm = hi + below, *lo_yp = lo + qyp, *lo_ym = lo + qym, *hi_ym = hi + qym;
    auto spin = [](const char *a, int col) { return *reinterpret_cast<const uint32_t *>(a + 4 * col * S::POS); };
    auto xbond = [](const char *a, int col) { return *reinterpret_cast<const uint32_t *>(a + 4 * (2 + col) * S::POS); };
    auto ybond = [](const char *a, int col) { return *reinterpret_cast<const uint32_t *>(a + 4 * col * S::POS); };
    auto zbond = [](const char *a, int col) { return *reinterpret_cast<const uint32_t *>(a + 4 * (2 + col) * S::POS); };
    constexpr int o = c ^ 1;
    uint32_t O = spin(lo, o), Zm = spin(lo + below, o);
#pragma unroll 1
    for (; z < z_end; ++z) {
        char *lo_zp = lo + (z == L - 1 ? -(L - 1) * STEP : STEP);
        const uint32_t S0 = spin(lo, c), Zp = spin(lo_zp, o);
        const uint32_t Om = RW == 1 ? O : spin(lo + qm, o), Op = RW == 1 ? O : spin(lo + qp, o);
        const uint32_t Xo = xbond(lo, o), Xom = RW == 1 ? Xo : xbond(lo + qm, o);
        const uint32_t Bx = xbond(lo, c), By = ybond(hi, c), Bz = zbond(hi, c);
        const uint32_t Yp = spin(lo_yp, o), Ym = spin(lo_ym, o), Bym = ybond(hi_ym, o), Bzm = zbond(hi_zm, o);
        auto decide = [&]() {
            // x neighbours: +x shares xh on even rows and sits at xh + 1 on
            // odd ones, -x at xh - 1 on even rows and shares xh on odd ones
            const uint32_t xp = __builtin_amdgcn_bitop3_b32(odd, take_plus1<W>(O, Op), O, kBitopSelect);
            const uint32_t xm = __builtin_amdgcn_bitop3_b32(odd, O ^ Xo, take_minus1<W>(O ^ Xo, Om ^ Xom), kBitopSelect);
            return classify(xor3(S0, xp, Bx), S0 ^ xm, xor3(S0, Yp, By), xor3(S0, Ym, Bym), xor3(S0, Zp, Bz),
                            xor3(S0, Zm, Bzm));
        };
        uint32_t flips;
        if constexpr (SEL == SEL_LDS)
            flips = flip_mask_lds<W>(step, quad0, batch_tables(), decide);
        else
            flips = flip_mask<W>(decide(), step, quad0, J.thr1, J.thr2, J.thr3);
        *reinterpret_cast<uint32_t *>(lo + 4 * c * S::POS) = S0 ^ flips;
        lo = lo_zp;
        hi_zm = hi;
        hi += STEP;
        lo_yp += STEP;
        lo_ym += STEP;
        hi_ym += STEP;
        Zm = O;
        O = Zp;
        odd = ~odd;
        quad0 += (uint32_t)(L * S::R / 4);
    }
}

// Between half-steps.  A wave's half-step reads the words of its own planes
// and of the planes next to them, so it only has to follow the waves that own
// those: every wave counts its finished half-steps in LDS and starts the next
// one when the waves of its neighbourhood have finished as many.  A neighbour
// is then at most one half-step away, so no word is overwritten that a wave
// still reads, and waves further apart may drift.  Against a workgroup
// barrier, where the SIMD with the most waves sets the pace and its last wave
// runs alone, at a fraction of the issue rate: L = 24 (nine waves) 1.02
// against 1.13 us per half-step, L = 40 3.25 / 3.42, L = 48 4.49 / 4.58,
// L = 56 8.15 / 8.53; but L = 64, whose sixteen waves load the four SIMDs
// evenly, 9.51 / 9.36: where a plane is whole waves the barrier stays.
template <int L, int RW>
constexpr bool kBatchDrift = (L * RW) % 64 != 0;

constexpr int kBatchWaves = kBatchThreads / 64;
__shared__ uint32_t batch_progress[kBatchWaves];

// Waves whose planes touch those of this wave (bit v: wave v), itself left
// out; nt threads work, nz planes each (batch_half_step).
template <int L, int RW>
__device__ __forceinline__ uint32_t batch_neighbours(int nt)
{
    constexpr int PLANE = L * RW;
    const int nz = (L + nt / PLANE - 1) / (nt / PLANE), G = (L + nz - 1) / nz;  // plane groups in use
    const int lane = (int)(threadIdx.x & 63), me = (int)(threadIdx.x >> 6);
    const int a0 = 64 * me / PLANE, b0 = min((64 * me + 63) / PLANE, G - 1);
    const int a1 = 64 * lane / PLANE, b1 = min((64 * lane + 63) / PLANE, G - 1);
    bool near = false;
#pragma unroll
    for (int k = -1; k <= 1; ++k) near |= a1 + k * G <= b0 + 1 && b1 + k * G >= a0 - 1;
    near = near && a0 < G && a1 < G && lane != me && lane < nt / 64;
    return (uint32_t)__ballot(near);
}

template <bool DRIFT>
__device__ __forceinline__ void batch_wait(uint32_t neighbours, uint32_t done)
{
    if constexpr (!DRIFT) return;  // batch_done was a barrier
    for (;;) {
        const uint32_t p = __hip_atomic_load(batch_progress + (threadIdx.x & (kBatchWaves - 1)), __ATOMIC_ACQUIRE,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
        if (((uint32_t)__ballot((int)(p - done) < 0) & neighbours) == 0) return;
        __builtin_amdgcn_s_sleep(1);
    }
}

template <bool DRIFT>
__device__ __forceinline__ void batch_done(uint32_t done)
{
    if constexpr (!DRIFT) {
        __syncthreads();
        return;
    }
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(batch_progress + (threadIdx.x >> 6), done, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The thread's index, opaque, so that what is computed from it stays where it
// is used instead of being kept (and spilled) across the sweep loop.
__device__ __forceinline__ int local_tid()
{
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// Copy this replica's two colour planes between LDS and a global array.
template <class S>
__device__ __forceinline__ void batch_store_spins(uint32_t *dst, int nt)
{
    for (int i = local_tid(); i < 2 * S::POS; i += nt) dst[i] = batch_lds[i];
}

// Load a replica's spins (two colour planes) and the couplings into LDS.
template <class S>
__device__ __forceinline__ void batch_load(const BatchJobDev &J, const uint32_t *spins)
{
    const int nt = J.nt, tid = local_tid();
    for (int i = tid; i < 2 * S::POS; i += nt) batch_lds[i] = spins[i];
    for (int i = tid; i < 6 * S::POS; i += nt) batch_lds[2 * S::POS + i] = J.bonds[i];
}

// The overlap and C4 (eqs. 2, 3) of measurement m from both published
// configurations, by one workgroup: the overlap words of every row (R <= 32
// sites of a colour: one word) go to LDS, lines along y and then along z laid
// out twice end to end, and each thread keeps one displacement rho = 1 .. R
// and a part of the lines.  Overwrites the workgroup's lattice in LDS.
// Bound by LDS reads and population counts, 6 L^2 R of each; a measurement
// of L = 64 (1024 threads) takes 150 us with all its parts.  Reading both
// words of every pair from memory, with one wave sum per displacement, it
// took 400, forty half-steps.
template <int L, int RW>
__device__ void batch_pair(const BatchJobDev &J, int m)
{
    using S = Shape<L, RW>;
    constexpr int W = S::W, POS = S::POS, R = S::R, ROWS = L * L;
    constexpr uint32_t MASK = word_mask<R>();
    // a slab (L >= kSplitMinL) holds four words per row, then two planes' halo
    static_assert(R <= 32 && 4 * ROWS + 3 * R <= (L >= kSplitMinL ? 4 * ROWS + 2 * L : 8 * ROWS),
                  "lines and counts fit the lattice part of LDS");
    const int nt = J.nt, tid = local_tid();
    const uint32_t *q0 = J.mspins + (size_t)m * 4 * POS;
    const uint32_t *q1 = q0 + 2 * POS;
    uint32_t *lines = batch_lds, *counts = batch_lds + 4 * ROWS;
    for (int i = tid; i < 3 * R; i += nt) counts[i] = 0u;
    const int parts = nt / R, part = tid / R, rho = 1 + tid - part * R, odd = rho & 1;
    uint32_t qdiff = 0, diff[3] = {0u, 0u, 0u};
#pragma unroll 1
    for (int d = 1; d <= 2; ++d) {  // lines along y, then along z
#pragma unroll 1
        for (int i = tid; i < 2 * ROWS; i += nt) {
            const int c = i >= ROWS ? 1 : 0, row = i - c * ROWS, z = row / L, y = row - z * L;
            uint32_t v = 0;
#pragma unroll
            for (int w = 0; w < RW; ++w)
                v |= (q0[c * POS + row * RW + w] ^ q1[c * POS + row * RW + w]) << (w * W);
            if (d == 1) qdiff += __popc(v);
            uint32_t *dst = lines + (d == 1 ? (c * L + z) * 2 * L + y : (c * L + y) * 2 * L + z);
            dst[0] = v;
            dst[L] = v;
        }
        __syncthreads();
        if (part < parts) {
#pragma unroll 1
            for (int k = part; k < 2 * L; k += parts) {
                const int c = k >= L ? 1 : 0, o = k - c * L;
                const uint32_t *own = lines + k * 2 * L;
                const uint32_t *other = lines + ((c ^ odd) * L + o) * 2 * L;
                uint32_t n = 0;
#pragma unroll 4
                for (int i = 0; i < L; ++i) n += __popc(own[i] ^ other[rho + i]);
                diff[d == 1 ? 1 : 2] += n;
                if (d == 1) {
                    // along x: the row's own word or the other colour's, rotated
                    n = 0;
#pragma unroll 4
                    for (int y = 0; y < L; ++y) {
                        const int sh = (rho >> 1) + (odd & (y + o + c));
                        const uint64_t p = (uint64_t)other[y] | (uint64_t)other[y] << R;
                        n += __popc((own[y] ^ (uint32_t)(p >> sh)) & MASK);
                    }
                    diff[0] += n;
                }
            }
        }
        __syncthreads();
    }
    if (part < parts)
#pragma unroll
        for (int d = 0; d < 3; ++d) atomicAdd(counts + d * R + rho - 1, diff[d]);
    unsigned long long *o = J.obs + (size_t)m * (size_t)J.obs_stride;
    wave_add(o + M_QDIFF, qdiff);
    __syncthreads();
    unsigned long long *c4 = o + batch_c4_base(J.n_tw);
    for (int i = tid; i < 3 * R; i += nt) {
        const int d = i / R, k = i - d * R;
        if (counts[i]) atomicAdd(c4 + d * (R + 1) + 1 + k, (unsigned long long)counts[i]);
    }
    __syncthreads();
}

// Publish this workgroup's part of replica r's configuration at measurement
// m (rows [row0, row0 + rows) of both colours, taken from LDS spin words
// batch_lds[c * src_stride + i]); the last workgroup of the job to arrive
// computes the replica-pair observables from the published copies.  True if
// this was the one: its LDS lattice is gone and has to be loaded again.
// flag_word is a free LDS word for a broadcast.
template <int L, int RW>
__device__ bool batch_publish_and_pair(const BatchJobDev &J, int r, int m, int row0, int rows, int src_stride,
                                       int flag_word)
{
    using S = Shape<L, RW>;
    constexpr int POS = S::POS;
    const int nt = J.nt;
    uint32_t *dst = J.mspins + ((size_t)m * 2 + (size_t)r) * 2 * POS;
    const int n = rows * RW, tid = local_tid();
#pragma unroll 1
    for (int c = 0; c < 2; ++c)
        for (int i = tid; i < n; i += nt) dst[c * POS + row0 * RW + i] = batch_lds[c * src_stride + i];
    __threadfence();
    __syncthreads();
    uint32_t *flag = batch_lds + flag_word;
    if (threadIdx.x == 0) *flag = atomicAdd(J.arrive + m, 1u);
    __syncthreads();
    const bool last = *flag == (uint32_t)(2 * J.parts - 1);
    __syncthreads();
    if (!last) return false;
    __threadfence();
    batch_pair<L, RW>(J, m);
    return true;
}

// Measurement at time t (index m) of replica r (whole replica in LDS).
template <int L, int RW>
__device__ void batch_measure(const BatchJobDev &J, int r, int m, int n_taken)
{
    using S = Shape<L, RW>;
    constexpr int W = S::W, POS = S::POS;
    const int nt = J.nt;
    unsigned long long *o = J.obs + (size_t)m * (size_t)J.obs_stride;
    uint32_t unsat = 0, down = 0;
#pragma unroll 1
    for (int c = 0; c < 2; ++c) {
        const uint32_t *own = lds_spin<S>(c);
        const uint32_t *oth = lds_spin<S>(c ^ 1);
        for (int p = local_tid(); p < POS; p += nt) {
            const int row = p / RW;
            const int w = p - row * RW;
            const int y = row % L;
            const int z = row / L;
            const int par = (y + z + c) & 1;
            const int wp = w == RW - 1 ? 0 : w + 1;
            const int yp = (y == L - 1 ? 0 : y + 1) + L * z;
            const int zp = y + L * (z == L - 1 ? 0 : z + 1);
            const uint32_t Sv = own[p];
            const uint32_t O = oth[row * RW + w];
            const uint32_t xp = par ? take_plus1<W>(O, oth[row * RW + wp]) : O;
            unsat += __popc(Sv ^ xp ^ lds_bond<S>(0, c)[p]) +
                     __popc(xor3(Sv, oth[yp * RW + w], lds_bond<S>(1, c)[p])) +
                     __popc(xor3(Sv, oth[zp * RW + w], lds_bond<S>(2, c)[p]));
            down += __popc(Sv);
        }
    }
    wave_add(o + M_UNSAT + r, unsat);
    wave_add(o + M_DOWN + r, down);
#pragma unroll 1
    for (int k = 0; k < n_taken; ++k) {
        const uint32_t *ref = J.snaps + ((size_t)k * 2 + (size_t)r) * 2 * POS;
        uint32_t diff = 0;
        for (int i = local_tid(); i < 2 * POS; i += nt) diff += __popc(batch_lds[i] ^ ref[i]);
        wave_add(o + M_AUTO + 2 * k + r, diff);
    }
    if (batch_publish_and_pair<L, RW>(J, r, m, 0, L * L, POS, S::LATTICE_WORDS))
        batch_load<S>(J, J.mspins + ((size_t)m * 2 + (size_t)r) * 2 * POS);
}

// Sweeps t .. t_end - 1; done counts the half-steps of the unit so far.
template <int L, int RW, int SEL>
__device__ __forceinline__ void batch_sweeps(const BatchJobDev &J, int r, uint32_t t, uint32_t t_end,
                                             uint32_t neighbours, uint32_t &done)
{
    constexpr bool D = kBatchDrift<L, RW>;
    for (; t < t_end; ++t) {
        batch_wait<D>(neighbours, done);
        if (r == 0) batch_half_step<L, RW, SEL, 0>(J, r, t);
        else batch_half_step<L, RW, SEL, 1>(J, r, t);
        batch_done<D>(++done);
        batch_wait<D>(neighbours, done);
        if (r == 0) batch_half_step<L, RW, SEL, 1>(J, r, t);
        else batch_half_step<L, RW, SEL, 0>(J, r, t);
        batch_done<D>(++done);
    }
}

// Run one unit: load the replica and the couplings into LDS, sweep up to
// t_stop taking the events scheduled in (t0, t_stop] (and at t0 itself on the
// job's first span), then write the replica back.
template <int L, int RW, int SEL>
__device__ void batch_run_unit(const BatchJobDev &J, int r, uint32_t t_stop, bool first)
{
    using S = Shape<L, RW>;
    const int nt = J.nt;
    if ((int)threadIdx.x >= nt) return;  // whole surplus waves leave the barrier set
    const uint32_t t0 = J.t_now[r];
    if (!first && t0 >= t_stop) return;
    batch_load<S>(J, J.spins + (size_t)r * 2 * S::POS);
    if constexpr (SEL == SEL_LDS) fill_select_tables(batch_tables(), J.thr1, J.thr2, J.thr3, (int)threadIdx.x, nt);
    if (threadIdx.x < kBatchWaves) batch_progress[threadIdx.x] = 0;
    __syncthreads();

    int im = 0, iw = 0;
    while (im < J.n_meas && (J.meas_t[im] < t0 || (!first && J.meas_t[im] == t0))) ++im;
    while (iw < J.n_tw && (J.tw_t[iw] < t0 || (!first && J.tw_t[iw] == t0))) ++iw;

    const uint32_t neighbours = batch_neighbours<L, RW>(nt);
    uint32_t t = t0, done = 0;
    for (;;) {
        if (iw < J.n_tw && J.tw_t[iw] == t) {
            batch_store_spins<S>(J.snaps + ((size_t)iw * 2 + (size_t)r) * 2 * S::POS, nt);
            ++iw;
            __threadfence();
            __syncthreads();
        }
        if (im < J.n_meas && J.meas_t[im] == t) {
            batch_measure<L, RW>(J, r, im, iw);
            ++im;
            __syncthreads();
        }
        if (t >= t_stop) break;
        // to the next event or the end
        uint32_t t_next = t_stop;
        if (iw < J.n_tw) t_next = min(t_next, J.tw_t[iw]);
        if (im < J.n_meas) t_next = min(t_next, J.meas_t[im]);
        batch_sweeps<L, RW, SEL>(J, r, t, t_next, neighbours, done);
        t = t_next;
        __syncthreads();
    }
    batch_store_spins<S>(J.spins + (size_t)r * 2 * S::POS, nt);
    if (threadIdx.x == 0) J.t_now[r] = t;
}

// ---------------------------------------------------------------------------
// Split replicas.  In a batch of uneven sizes one replica of the largest
// sample on one CU sets the length of the launch.  Such a replica can instead
// be cut into two z-slabs of NZ = L/2 planes, each held in LDS by its own
// workgroup.  A site on a slab's first or last plane has one neighbour on the
// other slab's adjacent plane (periodic in z), of the other colour; those
// boundary words pass through a small exchange area in global memory.
//
// In each half-step the first waves update the slab's two boundary planes, a
// wave each (wave 0 both at L = 64, see slab_half_step): a wave waits until the
// partner slab has published its plane next to this one in the previous
// half-step (a counter per plane, agent scope), updates its words and publishes
// them.  The other waves update the interior planes meanwhile, which need
// nothing from the partner, so the exchange latency hides behind interior work;
// the half-step still ends with one workgroup barrier.  Publication counter of
// a plane: 1 once its state at t = 0 is out, 2t + h + 2 after half-step h of
// sweep t.  Boundary words
// written in sweep t go to slot t & 1 (the state at t = 0 to slot 1): a
// measurement at t reads both colours of the partner's slot (t - 1) & 1
// while the partner may already be writing sweep t into the other slot.  A wait gives up
// after kSplitSpinTicks of the 100 MHz real-time counter (20 s), flags J.err
// and ends the unit, so a launch always drains.

constexpr unsigned long long kSplitSpinTicks = 2000000000ull;

template <int L, int RW>
struct Slab {
    static constexpr int R = L / 2, W = R / RW;
    static constexpr int NZ = L / 2;            // planes per slab
    static constexpr int PL = L * RW;           // words of one plane of one colour
    static constexpr int SPOS = NZ * PL;        // slab words of one colour
    static constexpr int POS = L * L * RW;      // whole-lattice words of one colour
    static constexpr int HALO = 8 * SPOS;       // [colour][PL] z couplings of the plane below the slab
    static constexpr int FLAG = HALO + 2 * PL;  // broadcast words
    static constexpr int LDS_WORDS = FLAG + 16;
    static_assert(NZ >= 3 && R % RW == 0 && W % 4 == 0 && W <= 32, "invalid slab");
};

template <class S>
__device__ __forceinline__ uint32_t *slab_spin(int c)
{
    return batch_lds + c * S::SPOS;
}

template <class S>
__device__ __forceinline__ uint32_t *slab_bond(int d, int c)
{
    return batch_lds + (2 + 2 * d + c) * S::SPOS;
}

// Boundary words of (replica r, slab, slot, colour c, plane k: 0 first, 1 last).
template <class S>
__device__ __forceinline__ uint32_t *slab_xbuf(const BatchJobDev &J, int r, int slab, int slot, int c, int k)
{
    return J.xbuf +
           (((((size_t)r * 2 + (size_t)slab) * 2 + (size_t)slot) * 2 + (size_t)c) * 2 + (size_t)k) * S::PL;
}

__device__ __forceinline__ uint32_t load_agent(const uint32_t *p)
{
    return __hip_atomic_load(const_cast<uint32_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave 0: wait until the counter reaches `want`; false on time-out.
__device__ __forceinline__ bool slab_wait(unsigned long long *pub, unsigned long long want)
{
    int ok = 1;
    if (threadIdx.x == 0) {
        const unsigned long long start = __builtin_amdgcn_s_memrealtime();
        while (__hip_atomic_load(pub, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < want) {
            __builtin_amdgcn_s_sleep(1);
            if (__builtin_amdgcn_s_memrealtime() - start > kSplitSpinTicks) {
                ok = 0;
                break;
            }
        }
    }
    ok = __shfl(ok, 0, 64);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return ok != 0;
}

// Wave 0: make this wave's boundary stores visible, then set the counter.
__device__ __forceinline__ void slab_publish(unsigned long long *pub, unsigned long long value)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (threadIdx.x == 0) __hip_atomic_store(pub, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// The half-step exchange without cache maintenance.  The boundary words go
// out with agent-scope stores, which are written through to the level shared
// by all XCDs, and the partner reads them with agent-scope loads, which do
// not hit a stale L2 line; so publishing only has to wait for this wave's
// stores to complete before the counter is set, and waiting only has to see
// the counter -- no L2 write-back or invalidation per half-step.
__device__ __forceinline__ void store_agent(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void slab_publish_words(unsigned long long *pub, unsigned long long value)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(pub, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool slab_wait_words(unsigned long long *pub, unsigned long long want)
{
    int ok = 1;
    if ((threadIdx.x & 63) == 0) {
        const unsigned long long start = __builtin_amdgcn_s_memrealtime();
        while (__hip_atomic_load(pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) {
            __builtin_amdgcn_s_sleep(1);
            if (__builtin_amdgcn_s_memrealtime() - start > kSplitSpinTicks) {
                ok = 0;
                break;
            }
        }
    }
    ok = __shfl(ok, 0, 64);
    asm volatile("" ::: "memory");
    return ok != 0;
}

// New value of slab word p (colour c, sweep t), given its z-1 and z+1
// neighbour words of the other colour and the coupling to the z-1 neighbour.
template <int L, int RW, int SEL>
__device__ __forceinline__ uint32_t slab_new_word(const BatchJobDev &J, const PhiloxStep<true> &step, int c, int z0, int p,
                                                  uint32_t Ozm, uint32_t Ozp, uint32_t Bzm)
{
    using S = Slab<L, RW>;
    constexpr int W = S::W;
    const uint32_t *own = slab_spin<S>(c);
    const uint32_t *oth = slab_spin<S>(c ^ 1);
    const uint32_t *bx_own = slab_bond<S>(0, c), *by_own = slab_bond<S>(1, c), *bz_own = slab_bond<S>(2, c);
    const uint32_t *bx_oth = slab_bond<S>(0, c ^ 1), *by_oth = slab_bond<S>(1, c ^ 1);
    const unsigned row = (unsigned)p / RW;  // slab row y + L zl
    const unsigned w = (unsigned)p - row * RW;
    const unsigned y = row % L;
    const unsigned zl = row / L;
    const int par = (int)((y + zl + (unsigned)z0 + (unsigned)c) & 1u);
    const unsigned wm = w == 0 ? RW - 1 : w - 1;
    const unsigned wp = w == RW - 1 ? 0 : w + 1;
    const unsigned ym = (y == 0 ? L - 1 : y - 1) + L * zl, yp = (y == L - 1 ? 0 : y + 1) + L * zl;
    const unsigned base = row * RW;
    const uint32_t S0 = own[p];
    const uint32_t O = oth[base + w], Om = oth[base + wm], Op = oth[base + wp];
    const uint32_t Xo = bx_oth[base + w], Xom = bx_oth[base + wm];
    const uint32_t Bx = bx_own[p], By = by_own[p], Bz = bz_own[p];
    const uint32_t Yp = oth[yp * RW + w], Ym = oth[ym * RW + w], Bym = by_oth[ym * RW + w];
    auto decide = [&]() {
        const uint32_t odd = 0u - (uint32_t)par;
        const uint32_t xp = __builtin_amdgcn_bitop3_b32(odd, take_plus1<W>(O, Op), O, kBitopSelect);
        const uint32_t xm = __builtin_amdgcn_bitop3_b32(odd, O ^ Xo, take_minus1<W>(O ^ Xo, Om ^ Xom), kBitopSelect);
        return classify(xor3(S0, xp, Bx), S0 ^ xm, xor3(S0, Yp, By), xor3(S0, Ym, Bym), xor3(S0, Ozp, Bz),
                        xor3(S0, Ozm, Bzm));
    };
    const uint32_t quad0 = (uint32_t)(((row + (unsigned)(L * z0)) * S::R + w * W) >> 2);
    uint32_t flips;
    if constexpr (SEL == SEL_LDS)
        flips = flip_mask_lds<W>(step, quad0, batch_tables(), decide);
    else
        flips = flip_mask<W>(decide(), step, quad0, J.thr1, J.thr2, J.thr3);
    return S0 ^ flips;
}

// Publication counter of one face (0 the first plane, 1 the last) of a slab.
__device__ __forceinline__ unsigned long long *slab_pub(const BatchJobDev &J, int r, int slab, int face)
{
    return J.pub + 2 * (2 * r + slab) + face;
}

// Half-step (t, colour c) of one slab.  Returns false (in a boundary wave
// only) if the partner never published.  Waves 0 and 1 take one boundary plane
// each, which waits only for the partner's plane next to it, and the others
// take the interior; where that would leave a few words of the interior to
// another round (L = 64: 30 planes on 14 waves), wave 0 takes both planes in
// turn and 15 waves the interior.  Bound by the boundary's chain: wait, load,
// a word, publish.  Per half-step, with one wave for both planes and now: L = 48
// 4.45 us, 2.97; L = 56 4.82, 4.07; L = 64 5.23, 5.38.
template <int L, int RW, int SEL>
__device__ __forceinline__ bool slab_half_step(const BatchJobDev &J, int r, int slab, int c, uint32_t t,
                                               unsigned long long want, unsigned long long done)
{
    using S = Slab<L, RW>;
    const int z0 = slab * S::NZ;
    uint32_t *own = slab_spin<S>(c);
    const uint32_t *oth = slab_spin<S>(c ^ 1);
    const uint32_t *bz_oth = slab_bond<S>(2, c ^ 1);
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const PhiloxStep<true> step = philox_step(t, counter_word2(TAG_METRO, (uint32_t)c, (uint32_t)r), J.sample, J.k0, J.k1);
    constexpr int N = S::SPOS - 2 * S::PL;  // words of the interior planes 1 .. NZ-2
    const int rest = N % (J.nt - 128), bw = rest > 0 && rest <= 128 ? 1 : 2;
    if (tid >= 64 * bw) {
#pragma unroll 1
        for (int p = S::PL + tid - 64 * bw; p < S::SPOS - S::PL; p += J.nt - 64 * bw)
            own[p] = slab_new_word<L, RW, SEL>(J, step, c, z0, p, oth[p - S::PL], oth[p + S::PL], bz_oth[p - S::PL]);
        return true;
    }
    // colour c ^ 1 was last written in the previous half-step: this sweep's
    // first half-step, or the previous sweep's second
    const int rslot = (int)((c == r ? t + 1 : t) & 1u);
    const int wslot = (int)(t & 1u);
    const uint32_t *halo_bz = batch_lds + S::HALO + (c ^ 1) * S::PL;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll 1
    for (int k = wave; k < 2; k += bw) {  // the wave's face or both in turn
        if (!slab_wait_words(slab_pub(J, r, slab ^ 1, k ^ 1), want)) return false;
        const uint32_t *beyond = slab_xbuf<S>(J, r, slab ^ 1, rslot, c ^ 1, k ^ 1);  // the partner's plane next to it
#pragma unroll 1
        for (int j = tid & 63; j < S::PL; j += 64) {
            const int p = k ? S::SPOS - S::PL + j : j;
            const uint32_t z_out = load_agent(beyond + j), z_in = oth[k ? p - S::PL : p + S::PL];
            const uint32_t bz = k ? bz_oth[p - S::PL] : halo_bz[j];
            const uint32_t v = slab_new_word<L, RW, SEL>(J, step, c, z0, p, k ? z_in : z_out, k ? z_out : z_in, bz);
            own[p] = v;
            store_agent(slab_xbuf<S>(J, r, slab, wslot, c, k) + j, v);
        }
        slab_publish_words(slab_pub(J, r, slab, k), done);
    }
    return true;
}

// Load one slab's part of a replica's spins ([colour][POS]) and of the
// couplings into LDS.
template <int L, int RW>
__device__ __forceinline__ void slab_load(const BatchJobDev &J, int slab, const uint32_t *spins)
{
    using S = Slab<L, RW>;
    const int nt = J.nt, z0 = slab * S::NZ, tid = local_tid();
    const int zb = (z0 + L - 1) % L;  // the plane below the slab
    for (int c = 0; c < 2; ++c)
        for (int i = tid; i < S::SPOS; i += nt)
            batch_lds[c * S::SPOS + i] = spins[(size_t)c * S::POS + (size_t)z0 * S::PL + i];
    for (int dc = 0; dc < 6; ++dc)
        for (int i = tid; i < S::SPOS; i += nt)
            batch_lds[(2 + dc) * S::SPOS + i] = J.bonds[(size_t)dc * S::POS + (size_t)z0 * S::PL + i];
    for (int c = 0; c < 2; ++c)
        for (int i = tid; i < S::PL; i += nt)
            batch_lds[S::HALO + c * S::PL + i] = J.bonds[(size_t)(4 + c) * S::POS + (size_t)zb * S::PL + i];
}

// Measurement m at time t of one slab: its partial sums, then its part of
// the published configuration.  The partner's first plane (the +z neighbour
// of this slab's last plane) comes from the exchange area; wave 0 has waited
// for the partner's state at t.
template <int L, int RW>
__device__ void slab_measure(const BatchJobDev &J, int r, int slab, int m, int n_taken, uint32_t t)
{
    using S = Slab<L, RW>;
    constexpr int W = S::W;
    const int nt = J.nt;
    const int z0 = slab * S::NZ;
    unsigned long long *o = J.obs + (size_t)m * (size_t)J.obs_stride;
    uint32_t unsat = 0, down = 0;
#pragma unroll 1
    for (int c = 0; c < 2; ++c) {
        const uint32_t *own = slab_spin<S>(c);
        const uint32_t *oth = slab_spin<S>(c ^ 1);
        const uint32_t *part_first = slab_xbuf<S>(J, r, slab ^ 1, (int)((t + 1) & 1u), c ^ 1, 0);
        for (int p = local_tid(); p < S::SPOS; p += nt) {
            const int row = p / RW;
            const int w = p - row * RW;
            const int y = row % L;
            const int zl = row / L;
            const int par = (y + zl + z0 + c) & 1;
            const int wp = w == RW - 1 ? 0 : w + 1;
            const int yp = (y == L - 1 ? 0 : y + 1) + L * zl;
            const uint32_t Sv = own[p];
            const uint32_t O = oth[row * RW + w];
            const uint32_t xp = par ? take_plus1<W>(O, oth[row * RW + wp]) : O;
            const uint32_t Ozp = zl + 1 < S::NZ ? oth[p + S::PL] : load_agent(part_first + (p - (S::SPOS - S::PL)));
            unsat += __popc(Sv ^ xp ^ slab_bond<S>(0, c)[p]) +
                     __popc(xor3(Sv, oth[yp * RW + w], slab_bond<S>(1, c)[p])) +
                     __popc(xor3(Sv, Ozp, slab_bond<S>(2, c)[p]));
            down += __popc(Sv);
        }
    }
    wave_add(o + M_UNSAT + r, unsat);
    wave_add(o + M_DOWN + r, down);
#pragma unroll 1
    for (int k = 0; k < n_taken; ++k) {
        const uint32_t *ref = J.snaps + ((size_t)k * 2 + (size_t)r) * 2 * S::POS + (size_t)z0 * S::PL;
        uint32_t diff = 0;
#pragma unroll 1
        for (int c = 0; c < 2; ++c)
            for (int i = local_tid(); i < S::SPOS; i += nt) diff += __popc(batch_lds[c * S::SPOS + i] ^ ref[c * S::POS + i]);
        wave_add(o + M_AUTO + 2 * k + r, diff);
    }
    if (batch_publish_and_pair<L, RW>(J, r, m, z0 * L, S::NZ * L, S::SPOS, S::FLAG))
        slab_load<L, RW>(J, slab, J.mspins + ((size_t)m * 2 + (size_t)r) * 2 * S::POS);
}

// Copy this slab's two colour parts between LDS and a [colour][POS] array.
template <class S>
__device__ __forceinline__ void slab_store(uint32_t *dst, int z0, int nt)
{
#pragma unroll 1
    for (int c = 0; c < 2; ++c)
        for (int i = local_tid(); i < S::SPOS; i += nt)
            dst[(size_t)c * S::POS + (size_t)z0 * S::PL + i] = batch_lds[c * S::SPOS + i];
}

// Run one slab of a split replica up to t_stop (events as in batch_run_unit).
template <int L, int RW, int SEL>
__device__ void batch_run_slab(const BatchJobDev &J, int r, int slab, uint32_t t_stop, bool first)
{
    using S = Slab<L, RW>;
    const int nt = J.nt;
    if ((int)threadIdx.x >= nt) return;
    const uint32_t t0 = J.t_now[r];
    if (!first && t0 >= t_stop) return;
    const int z0 = slab * S::NZ;
    slab_load<L, RW>(J, slab, J.spins + (size_t)r * 2 * S::POS);
    if constexpr (SEL == SEL_LDS) fill_select_tables(batch_tables(), J.thr1, J.thr2, J.thr3, (int)threadIdx.x, nt);
    uint32_t *abort_flag = batch_lds + S::FLAG + 1;
    if (threadIdx.x == 0) *abort_flag = 0;
    __syncthreads();
    if (first && threadIdx.x < 64) {
        // the state at t = 0 of both colours' boundary planes
        for (int c = 0; c < 2; ++c)
            for (int i = (int)threadIdx.x; i < 2 * S::PL; i += 64) {
                const int k = i >= S::PL ? 1 : 0;
                const int j = i - k * S::PL;
                slab_xbuf<S>(J, r, slab, 1, c, k)[j] = batch_lds[c * S::SPOS + (k ? S::SPOS - S::PL : 0) + j];
            }
        for (int k = 0; k < 2; ++k) slab_publish(slab_pub(J, r, slab, k), 1ull);
    }

    int im = 0, iw = 0;
    while (im < J.n_meas && (J.meas_t[im] < t0 || (!first && J.meas_t[im] == t0))) ++im;
    while (iw < J.n_tw && (J.tw_t[iw] < t0 || (!first && J.tw_t[iw] == t0))) ++iw;

    uint32_t t = t0;
    for (;;) {
        if (iw < J.n_tw && J.tw_t[iw] == t) {
            slab_store<S>(J.snaps + ((size_t)iw * 2 + (size_t)r) * 2 * S::POS, z0, nt);
            ++iw;
            __threadfence();
            __syncthreads();
        }
        if (im < J.n_meas && J.meas_t[im] == t) {
            if (threadIdx.x < 64 && !slab_wait(slab_pub(J, r, slab ^ 1, 0), 2ull * t + 1)) {
                if (threadIdx.x == 0) {
                    *abort_flag = 1;
                    atomicOr(J.err, 1u);
                }
            }
            __syncthreads();
            if (*abort_flag) return;
            slab_measure<L, RW>(J, r, slab, im, iw, t);
            ++im;
            __syncthreads();
        }
        if (t >= t_stop) break;
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const unsigned long long want = 2ull * t + (unsigned)h + 1, done = want + 1;
            if (!slab_half_step<L, RW, SEL>(J, r, slab, r ^ h, t, want, done) && (threadIdx.x & 63) == 0) {
                *abort_flag = 1;
                atomicOr(J.err, 1u);
            }
            __syncthreads();
            if (*abort_flag) return;
        }
        ++t;
    }
    slab_store<S>(J.spins + (size_t)r * 2 * S::POS, z0, nt);
    if (threadIdx.x == 0) J.t_now[r] = t;
}

// Dispatch on the packing (finest valid alternative or the default) and the
// select variant for one lattice size.
template <int L>
__device__ __forceinline__ void batch_dispatch_L(const BatchJobDev &J, int r, int slab, uint32_t t_stop, bool first)
{
    constexpr int R = L / 2;
    constexpr int RW0 = words_per_row_c(R);
    constexpr int RW1 = finer_words_per_row_c(R, RW0);
    if constexpr (L >= kSplitMinL) {
        if (J.parts == 2) {
            if (J.rw == RW0 && J.sel == SEL_LDS) batch_run_slab<L, RW0, SEL_LDS>(J, r, slab, t_stop, first);
            return;
        }
    }
    if (J.rw == RW0) {
        if (J.sel == SEL_LDS) batch_run_unit<L, RW0, SEL_LDS>(J, r, t_stop, first);
        else batch_run_unit<L, RW0, SEL_REG>(J, r, t_stop, first);
    } else if constexpr (RW1 != 0) {
        if (J.rw == RW1) {
            if (J.sel == SEL_LDS) batch_run_unit<L, RW1, SEL_LDS>(J, r, t_stop, first);
            else batch_run_unit<L, RW1, SEL_REG>(J, r, t_stop, first);
        }
    }
}

// poison, lds_words: the debug LDS fill (debug_poison; poison = 0: off) of
// the launch's dynamic LDS words and the select tables.
__global__ __launch_bounds__(kBatchThreads) void batch_kernel(const BatchJobDev *__restrict__ jobs,
                                                              const BatchUnit *__restrict__ units,
                                                              uint32_t poison, int lds_words)
{
    if (poison) {
        debug_poison(batch_lds, lds_words, poison, (int)threadIdx.x, kBatchThreads);
        debug_poison(batch_select_tables, kSelectTableWords, poison, (int)threadIdx.x, kBatchThreads);
        __syncthreads();
    }
    const BatchUnit u = units[blockIdx.x];
    const BatchJobDev J = jobs[u.job];
    const bool first = u.first != 0;
    switch (J.L) {
    case 8: batch_dispatch_L<8>(J, u.replica, u.slab, u.t_stop, first); break;
    case 16: batch_dispatch_L<16>(J, u.replica, u.slab, u.t_stop, first); break;
    case 24: batch_dispatch_L<24>(J, u.replica, u.slab, u.t_stop, first); break;
    case 32: batch_dispatch_L<32>(J, u.replica, u.slab, u.t_stop, first); break;
    case 40: batch_dispatch_L<40>(J, u.replica, u.slab, u.t_stop, first); break;
    case 48: batch_dispatch_L<48>(J, u.replica, u.slab, u.t_stop, first); break;
    case 56: batch_dispatch_L<56>(J, u.replica, u.slab, u.t_stop, first); break;
    case 64: batch_dispatch_L<64>(J, u.replica, u.slab, u.t_stop, first); break;
    default: break;
    }
}

// Every job's initial state in one launch: couplings, both replicas' spins,
// and the counters, arrivals, times and publications cleared.  blockIdx.x =
// job, blockIdx.y = plane (6 of couplings, 4 of spins), blockIdx.z = part of
// it.  (With four launches per job, the launches were the time: 256 jobs 3000
// us against 143 now, 16 jobs 238 against 21.)
__global__ __launch_bounds__(256) void batch_reset_kernel(const BatchJobDev *__restrict__ jobs, uint32_t *err)
{
    const BatchJobDev &J = jobs[blockIdx.x];
    const int plane = (int)blockIdx.y, at = (int)(blockIdx.z * blockDim.x + threadIdx.x);
    const int step = (int)(gridDim.z * blockDim.x);
    const int R = J.L / 2, W = R / J.rw, POS = J.L * J.L * J.rw;
    const size_t n = (size_t)J.n_meas * (size_t)J.obs_stride;
    for (size_t i = (size_t)(plane * step + at); i < n; i += (size_t)(10 * step)) J.obs[i] = 0ull;
    if (plane == 0) {
        // arrive[n_meas] and t_now[2] are contiguous
        for (int i = at; i < J.n_meas + 2; i += step) J.arrive[i] = 0u;
        if (at < kBatchPubs) J.pub[at] = 0ull;
        if (blockIdx.x == 0 && at == 0) *err = 0u;
    }
    if (at >= POS) return;
    const int row = at / J.rw, w = at - row * J.rw, c = plane & 1;
    const int what = plane < 6 ? plane >> 1 : 3 + ((plane - 6) >> 1);
    const uint32_t quad0 = (uint32_t)((row * R + w * W) >> 2);
    uint32_t bits = 0;
    switch (W) {
    case 4: bits = init_word<4>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    case 8: bits = init_word<8>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    case 12: bits = init_word<12>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    case 16: bits = init_word<16>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    case 20: bits = init_word<20>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    case 24: bits = init_word<24>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    case 28: bits = init_word<28>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    default: bits = init_word<32>(what, c, quad0, J.sample, J.k0, J.k1, J.pcut); break;
    }
    uint32_t *dst = plane < 6 ? const_cast<uint32_t *>(J.bonds) + (size_t)plane * POS
                              : J.spins + (size_t)(plane - 6) * POS;
    dst[at] = bits;
}

}  // namespace ea
