// integrate.hip -- ForceContainer sum + NewtonIntegrator (section 2.1.5).
//
// One thread per body: the body adds the forces of its candidate pairs one by
// one, in ascending partner id (its row order; the wave helps with the
// gathers of a long row), so the sum is deterministic and needs no atomics;
// then gravity (damped like any force, dampGravity),
// Cundall damping eq. 2.9 per component with the on-step velocity estimate
// v + a dt/2, the leapfrog update, the spherical rotation and, in a periodic
// cell, the homoDeform velocity terms (class Cell).  Energies use the
// mid-step velocities v-, w-.  Each body also accumulates its non-affine
// displacement since the last broad-phase run and raises the step's stall
// flag once it exceeds the Verlet budget (eq. 2.3-2.4).  Energies go to the
// block's own slot; a periodic cell is updated, F+ = (I + L dt) F, by a
// one-block kernel after the step.
#include "dem_internal.hpp"

#include <algorithm>
#include <cstddef>
#include <type_traits>

namespace dem {

namespace {

constexpr int kMaxBlock = 1024;

// The bodies of a block: each XCD takes a contiguous eighth, as the contact
// kernel's pairs, but from its end to its start.  The contact kernel has just
// been at the end of its eighths, so the records written last are the first to
// be read, still in the Infinity Cache (256 MB), and the next step's contact
// kernel starts where this one ended.  us per step, in the contact kernel's
// direction -> against it: 1 M spheres in shear FP32-mixed 318 -> 297, 500,000
// under the controlled cell 250 -> 245, 8 M 2025 -> 2007; scenes that fit the
// caches whole are as fast either way.  The partial sums keep their places:
// `slot` is the block that would have these bodies in the other direction.
__device__ inline int logical_block(int nb, int* slot)
{
    const int b = blockIdx.x;
    const int xcd = b & 7;
    const int q = nb >> 3, r = nb & 7;
    const int idx = q + (xcd < r ? 1 : 0) - 1 - (b >> 3);
    *slot = 8 * idx + xcd;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

__device__ inline double sgn(double x) { return x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0); }

// A history record as it is loaded: parts of 16 bytes.
typedef uint32_t Part __attribute__((ext_vector_type(4)));
template <int PREC>
struct HistParts {
    Part v[sizeof(typename HistOf<PREC>::T) / 16];
};

// One touching pair as a row entry sees it: the force on #2 and n x F, from
// the pair's force record (FREC: F on #2, n x F) or from its history record
// (linear law: F = fn n + Fs).  Without contraction, so that every
// walk over a row (one thread, or the wave together) gives the same bits.
template <int PREC, bool FREC>
__device__ inline void pair_force(const StepArgs& a, uint32_t k, double* f)
{
#pragma clang fp contract(off)
    if constexpr (!FREC) {
        using H = typename HistOf<PREC>::T;
        constexpr int kParts = sizeof(H) / 16;
        const gptr<const Part> p = glb<const Part>(reinterpret_cast<const Part*>(a.pr.h)) + kParts * (size_t)k;
        HistParts<PREC> h;
        for (int c = 0; c < kParts; ++c) h.v[c] = p[c];
        hist_force(__builtin_bit_cast(H, h), f);
    } else if (PREC == DEM_FP32_MIXED) {
        // a record is read as three pairs (it starts on an 8-byte boundary)
        const gptr<const float2> q = glb<const float2>(reinterpret_cast<const float2*>(a.pr.frecf)) + 3 * (size_t)k;
        for (int c = 0; c < 3; ++c) {
            const float2 v = q[c];
            f[2 * c] = v.x;
            f[2 * c + 1] = v.y;
        }
    } else {
        const gptr<const double2> q = glb<const double2>(reinterpret_cast<const double2*>(a.pr.frec)) + 3 * (size_t)k;
        for (int c = 0; c < 3; ++c) {
            const double2 v = q[c];
            f[2 * c] = v.x;
            f[2 * c + 1] = v.y;
        }
    }
}

// Adds one touching entry to the body's sums: the force negated where the
// body is #1; both bodies of a pair feel -r_k (n x F) (lever arms r1 n and
// -r2 n).
__device__ inline void add_entry(uint32_t u, const double* f, double r, double* F, double* T)
{
#pragma clang fp contract(off)
    if (u & kNegSign) {
        F[0] += -f[0];
        F[1] += -f[1];
        F[2] += -f[2];
    } else {
        F[0] += f[0];
        F[1] += f[1];
        F[2] += f[2];
    }
    T[0] += -r * f[3];
    T[1] += -r * f[4];
    T[2] += -r * f[5];
}

// Entries [beg, end) of a row, added in row order (ascending partner id):
// taken four at a time so that their loads are in flight together (no
// branch between them: a position past the end reads the last entry again
// and is then ignored).  An entry carries its pair's touched bit.
template <int PREC, bool FREC>
__device__ inline void row_walk(const StepArgs& a, int beg, int end, double r, double* F, double* T)
{
    const gptr<const uint32_t> ent = glb<const uint32_t>(a.rows.ent);
    constexpr int kB = 4;
    for (int e0 = beg; e0 < end; e0 += kB) {
        uint32_t u[kB];
        bool use[kB];
        for (int j = 0; j < kB; ++j) u[j] = ent[min(e0 + j, end - 1)];
        for (int j = 0; j < kB; ++j) {
            const uint32_t k = u[j] & kPairMask;
            use[j] = (e0 + j < end) && k < (uint32_t)a.npairs && (u[j] & kRealBit) != 0u;
        }
        // the four gathers go out together, with no branch between them: an
        // entry that does not count reads pair 0's record (always cached)
        // and is then ignored
        double f[kB][kForceWords];
        for (int j = 0; j < kB; ++j) pair_force<PREC, FREC>(a, use[j] ? (u[j] & kPairMask) : 0u, f[j]);
        for (int j = 0; j < kB; ++j)
            if (use[j]) add_entry(u[j], f[j], r, F, T);
    }
}

// Resultant contact force and torque on a slot whose row is [beg, end), in
// row order: the forces of its touching pairs, negated where the body is #1.
template <int PREC, bool FREC>
__device__ inline void body_sum(const StepArgs& a, int beg, int end, double r, double* F, double* T)
{
    F[0] = F[1] = F[2] = 0.0;
    T[0] = T[1] = T[2] = 0.0;
    row_walk<PREC, FREC>(a, beg, end, r, F, T);
}

// ---- the same sum in the integrate kernel, by the wave
//
// A lane looks at its row 24 entries at a time, all loaded at once (four per
// load), and keeps the touching ones (a third to a half) in its column of a
// list in LDS; the records are then gathered from the list, so that none is
// read for an entry that does not count, and a row costs one wait for its
// entries instead of one per four of them.
//
// Where the bodies fill the chip the gathers set the pace: a lane's 64-byte
// history record takes four accesses of 16 bytes, each of the 64 lanes in a
// line of its own.  QUAD: the four lanes of a quad read one record together,
// for each of the four in turn, and exchange the parts by quad permutations:
// 16 lines per load instead of 64.  Two records per lane are in flight then
// (three spill: 109 us where two take 96, below).  Where waves are few, the
// exchange only lengthens the chain, and three records are read directly.
// Force records (24 or 48 bytes) are read directly, four in flight.
//
// Before (entries and records four at a time, no list) -> now, per launch:
// 8 M spheres in shear 974 -> 906 us, 500,000 under the controlled cell 126 ->
// 96 us, 1 M in shear FP32-mixed 142 -> 131 us (these three, with the direction
// of the walk and what passes by the caches in large scenes: 875, 93 and 115
// us), 32,000 dense equal spheres 10.8 -> 9.9 us in blocks of 64, 24 scenes of
// 158,625 in all 10.6 -> 9.2 us; a bed of 1,000 within 0.2 us.  Taking the
// wave's rows as one stream of 64 entries per load, ranked by ballots, took 924
// us at 8 M and 5 us more for the 32,000; records brought straight into LDS 951
// us.
//
// What is left of rows much longer than the rest (a large sphere among small
// ones has ~10x their entries) is finished by the wave together, one row's
// next 64 entries per round: each lane reads one record, and six lanes add
// one component each, in row order.  A span or a round costs about two waits
// for memory, so the lanes go on by themselves while none has more than four
// entries left for each row that is not finished.  Sharing every row past 12
// entries instead took one round per lane where all rows are a little longer
// (the 32,000 dense spheres: 75 us per launch).
//
// Every way takes a body's touching entries in row order with the arithmetic
// of row_walk, so the sums are the same bit for bit.
constexpr int kSpan = 24;  // entries of its row that a lane looks at at a time
static_assert(kSpan <= kRowPad && kSpan % 4 == 0, "a span may read past the last row");
union alignas(16) WaveRows {
    uint32_t list[kSpan][64];   // the touching ones of them, per lane
    double f[kForceWords][64];  // a shared round's forces
};
// four entries at once; a row starts anywhere
typedef uint32_t Entries __attribute__((ext_vector_type(4), aligned(4)));

__device__ inline void wave_lds_sync()
{
    // the wave's own LDS accesses before are complete before those after
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// One pair's record per lane, fetched by every lane of the wave (a lane
// without a pair passes 0), and what the sums take from it.
template <int PREC, bool FREC, bool QUAD>
struct Record {
    double f[kForceWords];
    __device__ void fetch(const StepArgs& a, uint32_t k) { pair_force<PREC, FREC>(a, k, f); }
    __device__ void force(double* o)
    {
        for (int q = 0; q < kForceWords; ++q) o[q] = f[q];
    }
};

constexpr int quad_ctrl(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }
template <int CTRL>
__device__ inline Part quad_perm(Part x)
{
    Part y;
    for (int d = 0; d < 4; ++d) y[d] = (uint32_t)__builtin_amdgcn_mov_dpp((int)x[d], CTRL, 0xf, 0xf, true);
    return y;
}
// In: lane s of a quad holds part s of the quad's records 0..3; out: parts
// 0..3 of record s.
__device__ inline void quad_transpose(Part* v)
{
    const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
    for (int p = 0; p < 4; p += 2) {
        const Part a = v[p], b = v[p + 1];
        const Part xa = quad_perm<quad_ctrl(1, 0, 3, 2)>(a), xb = quad_perm<quad_ctrl(1, 0, 3, 2)>(b);
        v[p] = odd ? xb : a;
        v[p + 1] = odd ? b : xa;
    }
    for (int p = 0; p < 2; ++p) {
        const Part a = v[p], b = v[p + 2];
        const Part xa = quad_perm<quad_ctrl(2, 3, 0, 1)>(a), xb = quad_perm<quad_ctrl(2, 3, 0, 1)>(b);
        v[p] = high ? xb : a;
        v[p + 2] = high ? b : xa;
    }
}
template <int PREC>
struct Record<PREC, false, true> {
    using H = typename HistOf<PREC>::T;
    static constexpr int kParts = sizeof(H) / 16;
    Part v[4];
    __device__ void fetch(const StepArgs& a, uint32_t k)
    {
        const gptr<const char> part =
            glb(reinterpret_cast<const char*>(a.pr.h)) + min((int)(threadIdx.x & 3), kParts - 1) * 16;
        const uint32_t q[4] = {(uint32_t)__builtin_amdgcn_mov_dpp((int)k, quad_ctrl(0, 0, 0, 0), 0xf, 0xf, true),
                               (uint32_t)__builtin_amdgcn_mov_dpp((int)k, quad_ctrl(1, 1, 1, 1), 0xf, 0xf, true),
                               (uint32_t)__builtin_amdgcn_mov_dpp((int)k, quad_ctrl(2, 2, 2, 2), 0xf, 0xf, true),
                               (uint32_t)__builtin_amdgcn_mov_dpp((int)k, quad_ctrl(3, 3, 3, 3), 0xf, 0xf, true)};
        for (int i = 0; i < 4; ++i) v[i] = *(gptr<const Part>)(part + (size_t)q[i] * sizeof(H));
    }
    __device__ void force(double* f)
    {
        quad_transpose(v);
        HistParts<PREC> h;
        for (int c = 0; c < kParts; ++c) h.v[c] = v[c];
        hist_force(__builtin_bit_cast(H, h), f);
    }
};

// Entries [at, at + n) (at most 64) of the row of lane `src` (its radius r),
// added to its sums by the wave.
template <int PREC, bool FREC>
__device__ inline void shared_round(const StepArgs& a, WaveRows& w, int at, int n, int src, double r, double* F,
                                    double* T)
{
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const uint32_t u = lane < n ? glb<const uint32_t>(a.rows.ent)[at + lane] : 0u;
    const bool use = (u & kRealBit) != 0u && (u & kPairMask) < (uint32_t)a.npairs;
    if (use) {
        double f[kForceWords];
        pair_force<PREC, FREC>(a, u & kPairMask, f);
        for (int q = 0; q < kForceWords; ++q) w.f[q][lane] = f[q];
    }
    const unsigned long long neg = __ballot(u & kNegSign);
    wave_lds_sync();
    // lane q adds component q: the forces with their sign, the torques with
    // the lever arm
    const double sum[kForceWords] = {F[0], F[1], F[2], T[0], T[1], T[2]};
    const double lever = -__shfl(r, src, 64);
    double acc = 0.0;
    for (int q = 0; q < kForceWords; ++q) {
        const double v = __shfl(sum[q], src, 64);
        if (lane == q) acc = v;
    }
    const double* const comp = w.f[lane < kForceWords ? lane : 0];
    for (unsigned long long left = __ballot(use); left; left &= left - 1ull) {
        const int j = __builtin_ctzll(left);
        const double v = comp[j];
        if (lane < 3)
            acc += (neg >> j & 1ull) ? -v : v;
        else
            acc += lever * v;
    }
    for (int q = 0; q < kForceWords; ++q) {
        const double v = __shfl(acc, q, 64);
        if (lane == src) (q < 3 ? F[q] : T[q - 3]) = v;
    }
    wave_lds_sync();
}

template <int PREC, bool FREC, bool QUAD>
__device__ inline void body_sum_wave(const StepArgs& a, int beg, int end, double r, double* F, double* T,
                                     WaveRows& w)
{
    constexpr int kB = FREC ? 4 : QUAD ? 2 : 3;
    F[0] = F[1] = F[2] = 0.0;
    T[0] = T[1] = T[2] = 0.0;
    const int lane = threadIdx.x & 63;
    int next = beg;
    int share = INT32_MAX;  // a row with more left than this is shared
    while (__any(next < end)) {
        const unsigned long long longs = __ballot(end - next > share);
        if (longs) {
            const int src = __builtin_ctzll(longs);
            const int at = __shfl(next, src, 64), n = min(__shfl(end, src, 64) - at, 64);
            shared_round<PREC, FREC>(a, w, at, n, src, r, F, T);
            if (lane == src) next += n;
        } else {
            const int n = min(end - next, kSpan);
            const gptr<const Entries> from = (gptr<const Entries>)(glb<const uint32_t>(a.rows.ent) + next);
            Entries e[kSpan / 4] = {};
            for (int j = 0; j < kSpan / 4; ++j)
                if (j < 2 || __any(n > 4 * j)) e[j] = from[j];
            int count = 0;
            for (int j = 0; j < kSpan; ++j) {
                const uint32_t u = e[j / 4][j % 4];
                if (j < n && (u & kRealBit) != 0u && (u & kPairMask) < (uint32_t)a.npairs) w.list[count++][lane] = u;
            }
            next += n;
            for (int c = 0; __any(c < count); c += kB) {
                // an entry that does not count is 0 and reads pair 0's record
                // (always cached), which is then ignored
                uint32_t u[kB];
                for (int j = 0; j < kB; ++j) u[j] = c + j < count ? w.list[c + j][lane] : 0u;
                Record<PREC, FREC, QUAD> rec[kB];
                for (int j = 0; j < kB; ++j) rec[j].fetch(a, u[j] & kPairMask);
                for (int j = 0; j < kB; ++j) {
                    double f[kForceWords];
                    rec[j].force(f);
                    if (u[j]) add_entry(u[j], f, r, F, T);
                }
            }
            wave_lds_sync();  // the list and a shared round's forces lie in the same place
        }
        share = 4 * __popcll(__ballot(next < end));
    }
}

__device__ inline void matvec(const double* M, double x, double y, double z, double* o)
{
    o[0] = (M[0] * x + M[1] * y) + M[2] * z;
    o[1] = (M[3] * x + M[4] * y) + M[5] * z;
    o[2] = (M[6] * x + M[7] * y) + M[8] * z;
}

typedef double Quat __attribute__((ext_vector_type(4)));

struct IntPartial {
    double kin, rot, grav, damp, fsum, fcnt;
};

template <int PREC, bool BATCHED, bool PERIODIC, bool FREC, bool LARGE>
__global__ void __launch_bounds__(kMaxBlock) k_integrate(const StepArgs* __restrict__ args, int parity)
{
    const StepArgs& a = *args;
    int slot;
    const int i = logical_block(gridDim.x, &slot) * blockDim.x + threadIdx.x;
    const bool live = i < a.nslots;
    const gptr<double4> bxr = glb(a.bod.xr), bvm = glb(a.bod.vm), bw = glb(a.bod.w);
    const gptr<Quat> bq = glb(reinterpret_cast<Quat*>(a.bod.q));
    // the previous step's stall flag is read first and tested only after the
    // body's loads are issued (they are in bounds, and nothing is stored
    // before the test), so that its latency overlaps theirs; the row bounds
    // before the body state: the row's loads wait for them
    const int32_t stalled = a.ctr->stall[parity ^ 1];
    int beg = 0, end = 0;
    double4 xr0 = make_double4(0.0, 0.0, 0.0, 0.0), vm0 = xr0, w0 = xr0;
    uint16_t mi = 0;
    uint8_t blocked = 0;
    if (live) {
        beg = glb<const int32_t>(a.rows.start)[i];
        end = glb<const int32_t>(a.rows.start)[i + 1];
        xr0 = bxr[i];
        vm0 = bvm[i];
        w0 = bw[i];
        mi = glb<const uint16_t>(a.bod.mat)[i];
        blocked = glb<const uint8_t>(a.bod.blocked)[i];
    }
    if (stalled) {
        // not run: keep every later step of this launch chain stopped too
        if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->stall[parity] = 1;
        return;
    }
    // this step ends an update period of the controlled cell: also sum the
    // dynamic spheres' |resultant contact force| (unbalanced force)
    const bool measure = a.ctr->measure != 0;
    IntPartial part = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    bool bad = false;
    bool over = false;
    // the contact force sum, by every lane of the wave (a lane past the last
    // body has an empty row)
    extern __shared__ __align__(16) char s_rows[];
    double F[3], T[3];
    body_sum_wave<PREC, FREC, LARGE && !FREC>(a, beg, end, xr0.w, F, T,
                                              reinterpret_cast<WaveRows*>(s_rows)[threadIdx.x >> 6]);
    if (live) {
        const int s = BATCHED ? (int)glb<const uint16_t>(a.bod.scene)[i] : 0;
        // an unbatched scene (periodic included) reads the descriptor's own
        // copy of its parameters: uniform, read-only here, so scalar loads
        const SceneParams& S = BATCHED ? a.scenes[s] : a.scene0;
        const double dt = S.dt;
        const double lam = S.damping;
        const double rho = glb<const Material>(a.mats)[mi].density;
        const double r = xr0.w, m = sphere_mass(r, rho);
        const double I = 2.0 * m * r * r / 5.0;
        // FP64 division costs about ten FP64 instructions: the step divides
        // by m and by I once and multiplies after that
        const double inv_m = 1.0 / m, inv_I = 1.0 / I;
        if (measure && blocked != 63u) {
            part.fsum = sqrt(F[0] * F[0] + F[1] * F[1] + F[2] * F[2]);
            part.fcnt = 1.0;
        }

        const double x0[3] = {xr0.x, xr0.y, xr0.z};
        const double v0[3] = {vm0.x, vm0.y, vm0.z};
        double w[3] = {w0.x, w0.y, w0.z};
        double f[3], t[3];
        for (int k = 0; k < 3; ++k) {
            f[k] = F[k] + m * S.gravity[k];
            t[k] = T[k];
        }
        part.kin = 0.5 * m * ((v0[0] * v0[0] + v0[1] * v0[1]) + v0[2] * v0[2]);
        part.rot = 0.5 * I * ((w[0] * w[0] + w[1] * w[1]) + w[2] * w[2]);

        double homo[3] = {0.0, 0.0, 0.0};
        if (PERIODIC && S.homo_deform > 0) {
            double dL[9], a1[3], a2[3];
            for (int k = 0; k < 9; ++k) dL[k] = S.L[k] - S.Lprev[k];
            matvec(dL, x0[0], x0[1], x0[2], a1);
            matvec(S.L, v0[0], v0[1], v0[2], a2);
            for (int k = 0; k < 3; ++k) homo[k] = a1[k] + (S.homo_deform == 2 ? a2[k] * dt : 0.0);
        }
        double v[3];
        for (int k = 0; k < 3; ++k) {
            if (blocked & (1u << k)) {
                v[k] = v0[k];
                continue;
            }
            part.grav += -m * S.gravity[k] * v0[k] * dt;
            if (lam > 0.0) {
                const double acc = f[k] * inv_m;
                const double df = -lam * sgn(f[k] * (v0[k] + acc * dt / 2.0)) * f[k];
                part.damp += -df * v0[k] * dt;
                f[k] += df;
            }
            v[k] = v0[k] + f[k] * inv_m * dt + homo[k];
        }
        const double x1[3] = {x0[0] + v[0] * dt, x0[1] + v[1] * dt, x0[2] + v[2] * dt};

        for (int k = 0; k < 3; ++k) {
            if (blocked & (8u << k)) continue;
            if (lam > 0.0 && S.damp_rot) {
                // the torque's share of the damping work uses the mid-step spin
                const double acc = t[k] * inv_I;
                const double dtq = -lam * sgn(t[k] * (w[k] + acc * dt / 2.0)) * t[k];
                part.damp += -dtq * w[k] * dt;
                t[k] += dtq;
            }
            w[k] = w[k] + t[k] * inv_I * dt;
        }
        const double ww = (w[0] * w[0] + w[1] * w[1]) + w[2] * w[2];
        if (ww > 0.0) {
            // the orientation only changes (and is only read) for a spinning body
            const double wn = sqrt(ww);
            const Quat q0 = load_once<LARGE, Quat>(bq + i);
            double q[4] = {q0.x, q0.y, q0.z, q0.w};
            const double half = 0.5 * wn * dt;
            double sn, cs;
            sincos(half, &sn, &cs);
            const double sh = sn / wn;
            const double d0 = cs, d1 = w[0] * sh, d2 = w[1] * sh, d3 = w[2] * sh;
            const double n0 = d0 * q[0] - d1 * q[1] - d2 * q[2] - d3 * q[3];
            const double n1 = d0 * q[1] + d1 * q[0] + d2 * q[3] - d3 * q[2];
            const double n2 = d0 * q[2] - d1 * q[3] + d2 * q[0] + d3 * q[1];
            const double n3 = d0 * q[3] + d1 * q[2] - d2 * q[1] + d3 * q[0];
            const double inv_qn = 1.0 / sqrt(n0 * n0 + n1 * n1 + n2 * n2 + n3 * n3);
            q[0] = n0 * inv_qn;
            q[1] = n1 * inv_qn;
            q[2] = n2 * inv_qn;
            q[3] = n3 * inv_qn;
            const Quat q1 = {q[0], q[1], q[2], q[3]};
            if constexpr (LARGE)
                __builtin_nontemporal_store(q1, bq + i);
            else
                bq[i] = q1;
        }
        bxr[i] = make_double4(x1[0], x1[1], x1[2], r);
        // the Verlet account (fourth word of vm): non-affine displacement of
        // this step (eq. 2.3); the cell's mean field uses its own share
        double u[3] = {v[0], v[1], v[2]};
        if (PERIODIC) {
            double Lx[3];
            matvec(S.L, x0[0], x0[1], x0[2], Lx);
            for (int k = 0; k < 3; ++k) u[k] -= Lx[k];
        }
        const double d = vm0.w + sqrt((u[0] * u[0] + u[1] * u[1]) + u[2] * u[2]) * dt + a.ctr->verlet_cell_step;
        bvm[i] = make_double4(v[0], v[1], v[2], d);
        // an unchanged spin (no torque, or blocked) is not stored again
        if (w[0] != w0.x || w[1] != w0.y || w[2] != w0.z) bw[i] = make_double4(w[0], w[1], w[2], 0.0);

        over = d > a.ctr->verlet_limit;
        bad = !(isfinite(x1[0]) && isfinite(x1[1]) && isfinite(x1[2]) && isfinite(v[0]) && isfinite(v[1]) &&
                isfinite(v[2]));
    }
    // eq. 2.4: some body may now have left its enlarged bound: the next step
    // needs a broad-phase run (plain stores of the same value)
    if (__any(over) && (threadIdx.x & 63) == 0) a.ctr->stall[parity] = 1;
    if (__any(bad) && (threadIdx.x & 63) == 0) a.ctr->nonfinite = 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->steps_done += 1;
    const bool energy = a.track_energy != 0;
    if (!energy && !measure) return;

    // ---- energies and the controlled cell's force sums into this block's
    // slot (fixed-order wave/block sums)
    __shared__ IntPartial s_p[kMaxBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    for (int off = 32; off > 0; off >>= 1) {
        if (energy) {
            part.kin += __shfl_down(part.kin, off, 64);
            part.rot += __shfl_down(part.rot, off, 64);
            part.grav += __shfl_down(part.grav, off, 64);
            part.damp += __shfl_down(part.damp, off, 64);
        }
        if (measure) {
            part.fsum += __shfl_down(part.fsum, off, 64);
            part.fcnt += __shfl_down(part.fcnt, off, 64);
        }
    }
    if (lane == 0) s_p[wave] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        IntPartial p = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int w = 0; w < nwaves; ++w) {
            p.kin += s_p[w].kin;
            p.rot += s_p[w].rot;
            p.grav += s_p[w].grav;
            p.damp += s_p[w].damp;
            p.fsum += s_p[w].fsum;
            p.fcnt += s_p[w].fcnt;
        }
        IntAcc& acc = a.acc_integrate[slot];
        if (energy) {
            acc.kin = p.kin;
            acc.rot = p.rot;
            acc.grav += p.grav;
            acc.damp += p.damp;
        }
        if (measure) {
            acc.fsum = p.fsum;
            acc.fcnt = p.fcnt;
        }
    }
}

// The controlled cell's first reduction level (update steps only): block g
// of kCtrlReduceGrid sums, in a fixed order, a fixed contiguous share of the
// contact kernel's per-block terms (term-major in acc_ctrl) and of the
// integrate kernel's slots, into kCtrlWords values at acc_ctrl2[g].
constexpr int kCtrlWords = kNetworkWords + 2;
constexpr int kCtrlReduceBlock = 256;

__global__ void __launch_bounds__(kCtrlReduceBlock) k_ctrl_reduce(const StepArgs* __restrict__ args, int parity)
{
    const StepArgs& a = *args;
    if (a.ctr->stall[parity ^ 1] || !a.ctr->measure) return;
    const int g = blockIdx.x, G = gridDim.x;
    const int nb = a.nblocks_contact, ni = a.nblocks_integrate;
    const int b0 = (int)(((int64_t)g * nb) / G), b1 = (int)(((int64_t)(g + 1) * nb) / G);
    const int i0 = (int)(((int64_t)g * ni) / G), i1 = (int)(((int64_t)(g + 1) * ni) / G);
    double t[kCtrlWords];
    for (int q = 0; q < kCtrlWords; ++q) t[q] = 0.0;
    for (int b = b0 + (int)threadIdx.x; b < b1; b += blockDim.x)
        for (int q = 0; q < kNetworkWords; ++q) t[q] += a.acc_ctrl[(size_t)q * nb + b];
    for (int i = i0 + (int)threadIdx.x; i < i1; i += blockDim.x) {
        t[kNetworkWords] += a.acc_integrate[i].fsum;
        t[kNetworkWords + 1] += a.acc_integrate[i].fcnt;
    }
    __shared__ double sh[kCtrlReduceBlock / 64][kCtrlWords];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int q = 0; q < kCtrlWords; ++q)
        for (int off = 32; off > 0; off >>= 1) t[q] += __shfl_down(t[q], off, 64);
    if (lane == 0)
        for (int q = 0; q < kCtrlWords; ++q) sh[wave][q] = t[q];
    __syncthreads();
    if (threadIdx.x < kCtrlWords) {
        double v = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) v += sh[w][threadIdx.x];
        a.acc_ctrl2[(size_t)kCtrlWords * g + threadIdx.x] = v;
    }
}

// Periodic cell (section 2.1.6), once per step after the bodies: H+ =
// (I + L dt) H and the same for trsf; H - H_prev is kept for the image
// velocity of the next step's contacts; L becomes L_prev.  Then, on the
// steps that end an update period of the controlled cell, the controller
// (PeriTriaxController driven by the packing stiffness) sets the velocity
// gradient of the next steps from the partial sums of the contact kernel's
// measuring instantiation and of the integrate kernel's slots (first reduced
// by k_ctrl_reduce): per stress axis (1 - grow_damping)(goal - sigma_ii)/(M_i T),
// M_i = (1/V) sum k_n (d_i n_i)^2 and T = glob_update dt (the full rate
// towards the goal's sign while M_i = 0), per strain axis
// (goal - log trsf_ii)/T, capped at max_rate; zero once the goal is reached
// (every stress axis within max(abs_tol, rel_tol |goal|), every strain axis
// within 1e-6, unbalanced force at most max_unbalanced), and with
// stop_when_done the launch chain halts.  One block; the partial sums are
// combined in a fixed order (a fixed range per thread, then a fixed tree).
constexpr int kCellBlock = 256;

// What bounds it is the chain of dependent accesses of one thread: it reads
// the cell from the descriptor, all at once and beside the flags, and writes
// the fields that change to the descriptor and to the scene table (which hold
// the same cell between steps).  Reading and writing the table field by field
// and copying it whole to the descriptor afterwards took 1.1 us longer (32,000
// dense spheres: 23.5 us per step, now 22.4).
__global__ void __launch_bounds__(kCellBlock) k_cell_update(StepArgs* args, int parity)
{
    const StepArgs& a = *args;
    const int32_t stalled = a.ctr->stall[parity ^ 1];
    const bool measure = a.ctrl->active && a.ctr->measure;
    SceneParams* const cells[2] = {&a.scenes[0], &args->scene0};
    const double dt = a.scene0.dt;
    double H0[9], T0[9], L[9], H[9], trsf[9];
    for (int k = 0; k < 9; ++k) {
        H0[k] = a.scene0.H[k];
        T0[k] = a.scene0.trsf[k];
        L[k] = a.scene0.L[k];
    }
    if (stalled) return;
    {
        double M[9], Hinv[9], dH[9];
        for (int k = 0; k < 9; ++k) M[k] = ((k % 4 == 0) ? 1.0 : 0.0) + L[k] * dt;
        for (int r = 0; r < 3; ++r)
            for (int q = 0; q < 3; ++q) {
                H[3 * r + q] = (M[3 * r + 0] * H0[q] + M[3 * r + 1] * H0[3 + q]) + M[3 * r + 2] * H0[6 + q];
                trsf[3 * r + q] = (M[3 * r + 0] * T0[q] + M[3 * r + 1] * T0[3 + q]) + M[3 * r + 2] * T0[6 + q];
            }
        for (int k = 0; k < 9; ++k) dH[k] = H[k] - H0[k];
        const double a0 = H[0], a1 = H[1], a2 = H[2], a3 = H[3], a4 = H[4], a5 = H[5], a6 = H[6], a7 = H[7],
                     a8 = H[8];
        const double C0 = a4 * a8 - a5 * a7, C1 = -(a3 * a8 - a5 * a6), C2 = a3 * a7 - a4 * a6;
        const double det = a0 * C0 + a1 * C1 + a2 * C2;
        Hinv[0] = C0 / det;
        Hinv[1] = -(a1 * a8 - a2 * a7) / det;
        Hinv[2] = (a1 * a5 - a2 * a4) / det;
        Hinv[3] = C1 / det;
        Hinv[4] = (a0 * a8 - a2 * a6) / det;
        Hinv[5] = -(a0 * a5 - a2 * a3) / det;
        Hinv[6] = C2 / det;
        Hinv[7] = -(a0 * a7 - a1 * a6) / det;
        Hinv[8] = (a0 * a4 - a1 * a3) / det;
        if (threadIdx.x == 0)
            for (SceneParams* S : cells)
                for (int k = 0; k < 9; ++k) {
                    S->dH[k] = dH[k];
                    S->H[k] = H[k];
                    S->trsf[k] = trsf[k];
                    S->Lprev[k] = L[k];
                    S->Hinv[k] = Hinv[k];
                }
    }
    if (measure) {
        const CtrlConfig& c = *a.ctrl;
        // fixed-order sum of the partials: thread t takes the blocks t,
        // t + blockDim, ... in order; then a fixed pairwise tree over threads
        constexpr int W = kCtrlWords;
        double t[W];
        for (int q = 0; q < W; ++q) t[q] = 0.0;
        for (int g = threadIdx.x; g < kCtrlReduceGrid; g += blockDim.x)
            for (int q = 0; q < W; ++q) t[q] += a.acc_ctrl2[(size_t)W * g + q];
        __shared__ double sh[kCellBlock][W];
        for (int q = 0; q < W; ++q) sh[threadIdx.x][q] = t[q];
        __syncthreads();
        for (int half = kCellBlock / 2; half > 0; half >>= 1) {
            if ((int)threadIdx.x < half)
                for (int q = 0; q < W; ++q) sh[threadIdx.x][q] += sh[threadIdx.x + half][q];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const double* sum = sh[0];
            CtrlState& st = *a.ctrl_state;
            const double V = fabs(H[0] * (H[4] * H[8] - H[5] * H[7]) - H[1] * (H[3] * H[8] - H[5] * H[6]) +
                                  H[2] * (H[3] * H[7] - H[4] * H[6]));
            const double T = (double)c.glob_update * dt;
            double rates[3];
            bool reached = true;
            const double ncont = sum[13], ndyn = sum[kNetworkWords + 1];
            st.unbalanced = (ncont > 0.0 && ndyn > 0.0) ? (sum[kNetworkWords] / ndyn) / (sum[12] / ncont) : NAN;
            for (int i = 0; i < 3; ++i) {
                st.stress[i] = sum[4 * i] / V;
                st.strain[i] = log(trsf[4 * i]);
                st.stiff[i] = sum[9 + i] / V;
            }
            if (c.iso) {
                // the isotropic compressor: mean stress and mean modulus, one
                // rate; a reached stress (balanced packing) hands over to the
                // next of the series in the same update
                const double sm = (st.stress[0] + st.stress[1] + st.stress[2]) / 3.0;
                const double Mm = (st.stiff[0] + st.stiff[1] + st.stiff[2]) / 3.0;
                double goal = c.series[st.series_index];
                auto at_goal = [&](double g) {
                    return fabs(g - sm) <= fmax(c.abs_tol, c.rel_tol * fabs(g)) && st.unbalanced <= c.max_unbalanced;
                };
                reached = at_goal(goal);
                if (reached && st.series_index + 1 < c.n_series) {
                    st.series_index += 1;
                    goal = c.series[st.series_index];
                    reached = false;
                }
                const double err = goal - sm;
                double rate;
                if (Mm > 0.0)
                    rate = (1.0 - c.grow_damping) * err / (Mm * T);
                else
                    rate = err != 0.0 ? copysign(c.max_rate[0], err) : 0.0;
                rate = fmax(-c.max_rate[0], fmin(c.max_rate[0], rate));
                rates[0] = rates[1] = rates[2] = rate;
            }
            for (int i = 0; i < 3 && !c.iso; ++i) {
                double rate;
                if (c.stress_mask & (1 << i)) {
                    const double err = c.goal[i] - st.stress[i];
                    if (st.stiff[i] > 0.0)
                        rate = (1.0 - c.grow_damping) * err / (st.stiff[i] * T);
                    else
                        rate = err != 0.0 ? copysign(c.max_rate[i], err) : 0.0;
                    if (fabs(err) > fmax(c.abs_tol, c.rel_tol * fabs(c.goal[i]))) reached = false;
                } else {
                    const double err = c.goal[i] - st.strain[i];
                    rate = err / T;
                    if (fabs(err) > 1e-6) reached = false;
                }
                rates[i] = fmax(-c.max_rate[i], fmin(c.max_rate[i], rate));
            }
            if (!c.iso && !(st.unbalanced <= c.max_unbalanced)) reached = false;
            st.done = reached ? 1 : 0;
            if (reached) rates[0] = rates[1] = rates[2] = 0.0;
            double lf = 0.0;
            for (int i = 0; i < 3; ++i) {
                st.rate[i] = rates[i];
                lf += rates[i] * rates[i];
            }
            st.updates += 1;
            // the mean field's share of the Verlet budget follows the new gradient
            const double cell_rate = 0.5 * sqrt(lf) * (2.0 * a.scene0.rmax + 4.0 * a.scene0.verlet);
            a.ctr->verlet_cell_step = cell_rate * dt;
            for (SceneParams* S : cells) {
                for (int k = 0; k < 9; ++k) S->L[k] = k % 4 == 0 ? rates[k / 4] : 0.0;
                S->verlet_cell_rate = cell_rate;
            }
            if (reached && c.stop_when_done) {
                a.ctr->halt = 1;
                a.ctr->stall[parity] = 1;  // the remaining steps of the chain do not run
            }
        }
    }
}

// Resultant force/torque per slot (for reporting), same sum as the step.
template <int PREC, bool FREC>
__global__ void k_body_forces(StepArgs a, double* __restrict__ f3, double* __restrict__ t3)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.nslots) return;
    double F[3], T[3];
    body_sum<PREC, FREC>(a, a.rows.start[i], a.rows.start[i + 1], a.bod.xr[i].w, F, T);
    for (int k = 0; k < 3; ++k) {
        f3[3 * i + k] = F[k];
        t3[3 * i + k] = T[k];
    }
}

// Per-body measures of one scene for the unbalanced force and the stiffness
// timestepper (reporting, not in the step), kBodyWords doubles per block:
// sum and largest |resultant contact force| over the dynamic spheres (not
// all six DOFs blocked), their number, and the smallest critical timestep
// sqrt(2) sqrt(m / K_ii) over their unblocked DOFs (eq. 2.12), with the
// translational stiffness K_ii = sum of (k_n - k_s) n_i^2 + k_s over the
// body's contacts (eq. 2.14) and the rotational one R_ii = sum of
// k_s r^2 (1 - n_i^2) against the inertia (+inf without contacts).
constexpr int kMeasureBlock = 256;

template <int PREC, bool BATCHED, bool FREC>
__global__ void __launch_bounds__(kMeasureBlock) k_body_measures(StepArgs a, int scene, double* __restrict__ part)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double fsum = 0.0, fmaxv = 0.0, cnt = 0.0, dtmin = INFINITY;
    if (i < a.nslots && (!BATCHED || (int)a.bod.scene[i] == scene) && a.bod.blocked[i] != 63u) {
        const unsigned blocked = a.bod.blocked[i];
        const double4 xr = a.bod.xr[i];
        const double r = xr.w, m = sphere_mass(r, a.mats[a.bod.mat[i]].density);
        const double I = 2.0 * m * r * r / 5.0;
        const int beg = a.rows.start[i], end = a.rows.start[i + 1];
        double F[3], T[3];
        body_sum<PREC, FREC>(a, beg, end, r, F, T);
        const double fa = sqrt(F[0] * F[0] + F[1] * F[1] + F[2] * F[2]);
        fsum = fa;
        fmaxv = fa;
        cnt = 1.0;
        double K[3] = {0.0, 0.0, 0.0}, Rr[3] = {0.0, 0.0, 0.0};
        for (int e = beg; e < end; ++e) {
            const uint32_t k = a.rows.ent[e] & kPairMask;
            if (!a.pr.real[k]) continue;
            const HistRec h = hist_load<PREC>(a.pr.h, k);
            const double n[3] = {h.nx, h.ny, h.nz};
            const int sa = a.pr.a[k], sb = a.pr.b[k];
            const bool wall = sa < 0;
            const double r2 = a.bod.xr[sb].w;
            const double r1 = wall ? (a.walls[-1 - sa].kind == kFacet ? 2.0 * r2 : r2) : a.bod.xr[sa].w;
            const int m1 = wall ? a.walls[-1 - sa].mat : (int)a.bod.mat[sa];
            const Material M1 = a.mats[m1], M2 = a.mats[a.bod.mat[sb]];
            const double k1 = M1.young * (2.0 * r1), k2 = M2.young * (2.0 * r2);
            const double kn = k1 * k2 / (k1 + k2);
            const double q1 = M1.young_poisson * (2.0 * r1), q2 = M2.young_poisson * (2.0 * r2);
            const double ks = q1 * q2 / (q1 + q2);
            for (int c = 0; c < 3; ++c) {
                K[c] += (kn - ks) * n[c] * n[c] + ks;
                Rr[c] += ks * r * r * (1.0 - n[c] * n[c]);
            }
        }
        for (int c = 0; c < 3; ++c) {
            if (!(blocked & (1u << c)) && K[c] > 0.0) dtmin = fmin(dtmin, sqrt(2.0) * sqrt(m / K[c]));
            if (!(blocked & (8u << c)) && Rr[c] > 0.0) dtmin = fmin(dtmin, sqrt(2.0) * sqrt(I / Rr[c]));
        }
    }
    __shared__ double sh[kMeasureBlock / 64][kBodyWords];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int off = 32; off > 0; off >>= 1) {
        fsum += __shfl_down(fsum, off, 64);
        fmaxv = fmax(fmaxv, __shfl_down(fmaxv, off, 64));
        cnt += __shfl_down(cnt, off, 64);
        dtmin = fmin(dtmin, __shfl_down(dtmin, off, 64));
    }
    if (lane == 0) {
        sh[wave][0] = fsum;
        sh[wave][1] = fmaxv;
        sh[wave][2] = cnt;
        sh[wave][3] = dtmin;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t[kBodyWords] = {0.0, 0.0, 0.0, INFINITY};
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            t[0] += sh[w][0];
            t[1] = fmax(t[1], sh[w][1]);
            t[2] += sh[w][2];
            t[3] = fmin(t[3], sh[w][3]);
        }
        for (int q = 0; q < kBodyWords; ++q) part[kBodyWords * (size_t)blockIdx.x + q] = t[q];
    }
}

template <int PREC, bool BATCHED, bool PERIODIC, bool FREC, bool LARGE>
void launch_t(const StepArgs* args, int parity, int grid, int block, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1)
{
    const dim3 g(grid > 0 ? grid : 1), b(block);
    // each wave's list and shared rounds
    const size_t lds = sizeof(WaveRows) * (size_t)((block + 63) / 64);
    if (ev0)
        hipExtLaunchKernelGGL((k_integrate<PREC, BATCHED, PERIODIC, FREC, LARGE>), g, b, lds, st, ev0, ev1, 0, args,
                              parity);
    else
        hipLaunchKernelGGL((k_integrate<PREC, BATCHED, PERIODIC, FREC, LARGE>), g, b, lds, st, args, parity);
}

template <int PREC, bool FREC, bool LARGE>
void launch_kind(const StepArgs* args, int parity, int grid, bool batched, bool periodic, int block, hipStream_t st,
                 hipEvent_t ev0, hipEvent_t ev1)
{
    if (batched) launch_t<PREC, true, false, FREC, LARGE>(args, parity, grid, block, st, ev0, ev1);
    else if (periodic) launch_t<PREC, false, true, FREC, LARGE>(args, parity, grid, block, st, ev0, ev1);
    else launch_t<PREC, false, false, FREC, LARGE>(args, parity, grid, block, st, ev0, ev1);
}

template <int PREC, bool FREC>
void launch_sized(const StepArgs* args, int parity, int grid, bool batched, bool periodic, bool large, int block,
                  hipStream_t st, hipEvent_t ev0, hipEvent_t ev1)
{
    if (large) launch_kind<PREC, FREC, true>(args, parity, grid, batched, periodic, block, st, ev0, ev1);
    else launch_kind<PREC, FREC, false>(args, parity, grid, batched, periodic, block, st, ev0, ev1);
}

// f(precision, force records) with both as types
template <typename F>
void by_records(int precision, bool frec, F&& f)
{
    using Fp32 = std::integral_constant<int, DEM_FP32_MIXED>;
    using Fp64 = std::integral_constant<int, DEM_FP64>;
    if (precision == DEM_FP32_MIXED)
        frec ? f(Fp32{}, std::true_type{}) : f(Fp32{}, std::false_type{});
    else
        frec ? f(Fp64{}, std::true_type{}) : f(Fp64{}, std::false_type{});
}

}  // namespace

void launch_integrate(const StepArgs* args, int parity, int grid, int precision, bool batched, bool periodic,
                      bool frec, bool large, int block, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1)
{
    by_records(precision, frec, [&](auto prec, auto rec) {
        launch_sized<decltype(prec)::value, decltype(rec)::value>(args, parity, grid, batched, periodic, large, block,
                                                                  st, ev0, ev1);
    });
}

// Largest Verlet account (non-affine displacement since the last broad-phase
// run, the fourth word of vm) over the bodies: wave maxima, then an integer
// maximum on the bits (non-negative doubles order like their bits).
__global__ void __launch_bounds__(256) k_max_account(Bodies b, int n, unsigned long long* __restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double v = i < n ? b.vm[i].w : 0.0;
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(out, (unsigned long long)__double_as_longlong(v));
}

void launch_max_account(const Bodies& b, int n, unsigned long long* out, hipStream_t st)
{
    if (n > 0) hipLaunchKernelGGL(k_max_account, dim3((n + 255) / 256), dim3(256), 0, st, b, n, out);
}

__global__ void __launch_bounds__(256) k_publish(StepArgs a, Counters c, StepArgs* __restrict__ dst, int nc, int ni)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    for (int i = t; i < nc; i += stride) a.acc_contact[i] = ContactAcc{};
    for (int i = t; i < ni; i += stride) a.acc_integrate[i] = IntAcc{};
    if (t == 0) {
        *dst = a;
        *a.ctr = c;
    }
}

// One wave: the counters' words, then the number that the host waits for.
// After a failed step (non-finite or unstable) the chain behind finds the
// stall flag raised and does nothing, so that the state the host hears of is
// no more than this chain past the failure; the report has the flag as the
// steps left it, and the host puts it back (run_steps).
__global__ void __launch_bounds__(64) k_report(const StepArgs* __restrict__ args, Report* __restrict__ ring, int last)
{
    Counters* const ctr = args->ctr;
    const uint32_t seq = ctr->reports + 1u;
    Report& r = ring[seq % kReports];
    constexpr int kWords = sizeof(Counters) / 4;
    uint32_t word = 0u;
    if (threadIdx.x < kWords) {
        word = reinterpret_cast<const uint32_t*>(ctr)[threadIdx.x];
        reinterpret_cast<uint32_t*>(&r.c)[threadIdx.x] = word;
    }
    const bool failed = __any(word != 0u && (threadIdx.x == offsetof(Counters, nonfinite) / 4 ||
                                             threadIdx.x == offsetof(Counters, unstable) / 4));
    __threadfence_system();
    __builtin_amdgcn_wave_barrier();
    if (threadIdx.x == 0) {
        ctr->reports = seq;
        __hip_atomic_store(&r.seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        if (failed) ctr->stall[last] = 1;
    }
}

void launch_report(const StepArgs* args, Report* ring, int last, hipStream_t st)
{
    hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, st, args, ring, last);
}

void launch_publish(const StepArgs& a, const Counters& c, StepArgs* dst, int nslots_contact, int nslots_integrate,
                    hipStream_t st)
{
    const int n = std::max({nslots_contact, nslots_integrate, 1});
    hipLaunchKernelGGL(k_publish, dim3(std::min((n + 255) / 256, 1024)), dim3(256), 0, st, a, c, dst, nslots_contact,
                       nslots_integrate);
}

void launch_ctrl_reduce(const StepArgs* args, int parity, hipStream_t st)
{
    hipLaunchKernelGGL(k_ctrl_reduce, dim3(kCtrlReduceGrid), dim3(kCtrlReduceBlock), 0, st, args, parity);
}

void launch_cell_update(const StepArgs* args, int parity, hipStream_t st)
{
    hipLaunchKernelGGL(k_cell_update, dim3(1), dim3(kCellBlock), 0, st, const_cast<StepArgs*>(args), parity);
}


int body_blocks(int nslots) { return nslots > 0 ? (nslots + kMeasureBlock - 1) / kMeasureBlock : 0; }

void launch_body_measures(const StepArgs& a, int precision, bool batched, int scene, double* part, hipStream_t st)
{
    const int grid = body_blocks(a.nslots);
    if (grid == 0) return;
    const dim3 g(grid), b(kMeasureBlock);
    auto launch = [&](auto prec, auto frec) {
        constexpr int P = decltype(prec)::value;
        constexpr bool F = decltype(frec)::value;
        if (batched) hipLaunchKernelGGL((k_body_measures<P, true, F>), g, b, 0, st, a, scene, part);
        else hipLaunchKernelGGL((k_body_measures<P, false, F>), g, b, 0, st, a, scene, part);
    };
    by_records(precision, a.use_frec != 0, launch);
}

void launch_body_forces(const StepArgs& a, int precision, double* f3, double* t3, hipStream_t st)
{
    if (a.nslots <= 0) return;
    const int grid = (a.nslots + 255) / 256;
    by_records(precision, a.use_frec != 0, [&](auto prec, auto frec) {
        hipLaunchKernelGGL((k_body_forces<decltype(prec)::value, decltype(frec)::value>), dim3(grid), dim3(256), 0, st,
                           a, f3, t3);
    });
}

}  // namespace dem
