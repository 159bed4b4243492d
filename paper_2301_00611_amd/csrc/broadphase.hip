// broadphase.hip -- the collider's role (section 2.1.1, InsertionSortCollider)
// rebuilt for the GPU: bodies are binned in cells no smaller than the largest
// candidate distance (2 r_max + 2 Delta L), put in cell order by a counting
// sort (cells are numbered along Morton bricks, a cell's bodies keep their
// order), and each body sweeps the 27 cells around its own for candidates
// whose enlarged spheres overlap (distance < r_i + r_j + 2 Delta L).  The run
// is needed only when some body may have moved farther than Delta L since the
// last one (eq. 2.3-2.4).  Candidate pairs are stored once (owner = #1 of the
// contact); every body keeps a row of its candidate pairs sorted by partner
// id, and the shear history of surviving pairs is carried over by id.
#include "dem_internal.hpp"

#include <algorithm>
#include <cfloat>

namespace dem {

namespace {

constexpr int kBlock = 256;

// the low 10 bits of v, two zero bits after each
__device__ inline uint32_t spread3(uint32_t v)
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Pack an integer image shift (each component in [-512, 511]) so that
// unsigned comparison orders shifts lexicographically.
__device__ inline int32_t pack_cell(int cx, int cy, int cz)
{
    return (int32_t)(((uint32_t)(cx + 512) << 20) | ((uint32_t)(cy + 512) << 10) | (uint32_t)(cz + 512));
}
__device__ inline void unpack_cell(int32_t p, int* c)
{
    uint32_t u = (uint32_t)p;
    c[0] = (int)((u >> 20) & 1023u) - 512;
    c[1] = (int)((u >> 10) & 1023u) - 512;
    c[2] = (int)(u & 1023u) - 512;
}
// packed (0, 0, 0): the shift of every aperiodic pair and every wall pair
constexpr int32_t kCellZero = (int32_t)((512u << 20) | (512u << 10) | 512u);
__device__ inline int32_t neg_cell(int32_t p)
{
    int c[3];
    unpack_cell(p, c);
    return pack_cell(-c[0], -c[1], -c[2]);
}

// One level of a scene's grid (level 1 exists only when r_split > 0).
struct Level {
    const double* origin;
    const double* inv_h;
    const double* cellw;
    const int32_t* dims;
    int32_t offset;
    int32_t bits;
};
__device__ inline Level level_of(const SceneParams& P, int lv)
{
    return lv == 0 ? Level{P.origin, P.inv_h, P.cellw, P.dims, P.cell_offset, P.brick_bits}
                   : Level{P.origin2, P.inv_h2, P.cellw2, P.dims2, P.cell_offset2, P.brick_bits2};
}
// A cell's number: bricks of 2^bits cells a side, x fastest, Morton order
// inside (the host picks the largest bricks that pad the grid little: see
// brick_bits).  The part of y and z and the part of x add up.
__device__ inline uint32_t cell_index_yz(const Level& V, int y, int z)
{
    const int m = V.bits, mask = (1 << m) - 1;
    const uint32_t hx = (uint32_t)(V.dims[0] + mask) >> m, hy = (uint32_t)(V.dims[1] + mask) >> m;
    const uint32_t brick = (((uint32_t)z >> m) * hy + ((uint32_t)y >> m)) * hx;
    return (uint32_t)V.offset + (brick << (3 * m)) + (spread3(y & mask) << 1) + (spread3(z & mask) << 2);
}
__device__ inline uint32_t cell_index_x(const Level& V, int x)
{
    const int m = V.bits, mask = (1 << m) - 1;
    return (((uint32_t)x >> m) << (3 * m)) + spread3(x & mask);
}
// the level a sphere of radius r is binned on
__device__ inline int level_of_radius(const SceneParams& P, double r) { return (P.r_split > 0.0 && r > P.r_split) ? 1 : 0; }

// Cell of a body on one level and, in a periodic cell, its integer period.
template <bool PERIODIC>
__device__ inline void cell_of(const SceneParams& P, const Level& V, double x, double y, double z, int* c, int* per)
{
    if (!PERIODIC) {
        c[0] = clampi((int)floor((x - V.origin[0]) * V.inv_h[0]), 0, V.dims[0] - 1);
        c[1] = clampi((int)floor((y - V.origin[1]) * V.inv_h[1]), 0, V.dims[1] - 1);
        c[2] = clampi((int)floor((z - V.origin[2]) * V.inv_h[2]), 0, V.dims[2] - 1);
        per[0] = per[1] = per[2] = 0;
        return;
    }
    const double* M = P.Hinv;
    double f[3] = {M[0] * x + M[1] * y + M[2] * z, M[3] * x + M[4] * y + M[5] * z, M[6] * x + M[7] * y + M[8] * z};
    for (int k = 0; k < 3; ++k) {
        double p = floor(f[k]);
        per[k] = (int)p;
        c[k] = clampi((int)floor((f[k] - p) * V.inv_h[k]), 0, V.dims[k] - 1);
    }
}

__device__ inline unsigned long long ord_bits(double v)
{
    unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

// ------------------------------------------------------------------ bounds

__global__ void __launch_bounds__(kBlock) k_bounds(Bodies b, int nslots, int batched,
                                                   unsigned long long* __restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < nslots;
    const int s = valid && batched ? (int)b.scene[i] : 0;
    unsigned long long v[6];
    if (valid) {
        const double4 p = b.xr[i];
        v[0] = ~ord_bits(p.x);
        v[1] = ~ord_bits(p.y);
        v[2] = ~ord_bits(p.z);
        v[3] = ord_bits(p.x);
        v[4] = ord_bits(p.y);
        v[5] = ord_bits(p.z);
    } else {
        for (int k = 0; k < 6; ++k) v[k] = 0ull;
    }
    // every value is reduced as a maximum (minima are stored complemented)
    const int s0 = __shfl(s, 0, 64);
    const bool uniform = __all(!valid || s == s0);
    if (uniform) {
        for (int k = 0; k < 6; ++k)
            for (int off = 32; off > 0; off >>= 1) {
                unsigned long long o = __shfl_xor(v[k], off, 64);
                v[k] = o > v[k] ? o : v[k];
            }
        if ((threadIdx.x & 63) == 0 && __any(valid))
            for (int k = 0; k < 6; ++k) atomicMax(&out[s0 * 6 + k], v[k]);
    } else if (valid) {
        for (int k = 0; k < 6; ++k) atomicMax(&out[s * 6 + k], v[k]);
    }
}

__device__ inline double unord_bits(unsigned long long v)
{
    return __longlong_as_double((long long)((v & 0x8000000000000000ull) ? (v & 0x7fffffffffffffffull) : ~v));
}

// Block maximum of the six ordered values; the first six threads get it.
__device__ inline unsigned long long bounds_block_max(unsigned long long* v)
{
    for (int k = 0; k < 6; ++k)
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(v[k], off, 64);
            v[k] = o > v[k] ? o : v[k];
        }
    __shared__ unsigned long long s[kBlock / 64][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
        for (int k = 0; k < 6; ++k) s[wave][k] = v[k];
    __syncthreads();
    unsigned long long m = 0ull;
    if (threadIdx.x < 6)
        for (int w = 0; w < kBlock / 64; ++w) m = s[w][threadIdx.x] > m ? s[w][threadIdx.x] : m;
    return m;
}

// the six words as doubles: lower corner (stored complemented), upper corner
__device__ inline void bounds_store(unsigned long long m, double* __restrict__ out)
{
    if (threadIdx.x < 6) out[threadIdx.x] = unord_bits(threadIdx.x < 3 ? ~m : m);
}

// Single scene: block maxima of the six ordered values, then one block
// combines them (no contended atomics); a scene that one block covers is
// done in one launch.
constexpr int kBoundsBlocks = 512;

__global__ void __launch_bounds__(kBlock) k_bounds_block(Bodies b, int nslots, unsigned long long* __restrict__ part,
                                                         double* __restrict__ out)
{
    unsigned long long v[6] = {0ull, 0ull, 0ull, 0ull, 0ull, 0ull};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nslots; i += gridDim.x * blockDim.x) {
        const double4 p = b.xr[i];
        const double x[3] = {p.x, p.y, p.z};
        for (int k = 0; k < 3; ++k) {
            const unsigned long long u = ord_bits(x[k]);
            v[k] = ~u > v[k] ? ~u : v[k];
            v[3 + k] = u > v[3 + k] ? u : v[3 + k];
        }
    }
    const unsigned long long m = bounds_block_max(v);
    if (gridDim.x == 1)
        bounds_store(m, out);
    else if (threadIdx.x < 6)
        part[(long)blockIdx.x * 6 + threadIdx.x] = m;
}

__global__ void __launch_bounds__(kBlock) k_bounds_final(const unsigned long long* __restrict__ part, int nblk,
                                                         double* __restrict__ out)
{
    unsigned long long v[6] = {0ull, 0ull, 0ull, 0ull, 0ull, 0ull};
    for (int b = threadIdx.x; b < nblk; b += blockDim.x)
        for (int k = 0; k < 6; ++k) {
            const unsigned long long o = part[(long)b * 6 + k];
            v[k] = o > v[k] ? o : v[k];
        }
    bounds_store(bounds_block_max(v), out);
}

__global__ void k_bounds_decode(unsigned long long* __restrict__ bits, double* __restrict__ out, int n6)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n6) return;
    const unsigned long long v = bits[i];
    out[i] = unord_bits(i % 6 < 3 ? ~v : v);
}

// ----------------------------------------------------------- counting sort
//
// The bodies go to cell order in three passes around a scan of the cells'
// counts: every body counts itself in its cell (and a large one in its
// level-1 cell), takes a place in the cell in the order of arrival, and is
// moved to its rank by its old slot among the bodies of its cell (a stable
// sort).  The order of arrival depends on the atomics, the final order does
// not.  The level-1
// index array keeps the order of arrival: only the order in which a search
// meets its candidates depends on it, and rows are sorted.  Against a radix
// sort of 64-bit keys (five launches per 8 bits, twice with two levels) the
// sort takes five to seven launches whatever the grid.  A whole run, start to
// first step, with the counts read back once: 1,000 spheres 400 -> 141 us,
// 9,262 408 -> 271, 200,000 (size ratio 3) 1.4 ms -> 281 us.

template <bool BATCHED, bool PERIODIC>
__global__ void __launch_bounds__(kBlock) k_cell_count(GridArgs g, CellSortArgs c)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.nslots) return;
    const int s = BATCHED ? (int)g.bod.scene[i] : 0;
    const SceneParams& P = BATCHED ? g.scenes[s] : g.scene0;
    int cc[3], per[3];
    const double4 p = g.bod.xr[i];
    const Level V = level_of(P, 0);
    cell_of<PERIODIC>(P, V, p.x, p.y, p.z, cc, per);
    const uint32_t lin = cell_index_yz(V, cc[1], cc[2]) + cell_index_x(V, cc[0]);
    c.cell[i] = lin;
    c.arrival[i] = atomicAdd(&c.count[lin], 1u);
    if (PERIODIC) {
        // a period is packed in 10 bits per axis: farther than 512 periods
        // from the origin it would wrap, so the run is refused instead
        bool out = false;
        for (int k = 0; k < 3; ++k) out = out || per[k] < -512 || per[k] > 511;
        if (out) *g.period_range = 1;
        g.bod.period[i] = pack_cell(per[0], per[1], per[2]);
    }
    if (c.nlarge > 0 && level_of_radius(P, p.w) == 1) {
        const Level V1 = level_of(P, 1);
        cell_of<PERIODIC>(P, V1, p.x, p.y, p.z, cc, per);
        const uint32_t lin1 = cell_index_yz(V1, cc[1], cc[2]) + cell_index_x(V1, cc[0]);
        c.cell1[i] = lin1;
        c.arrival1[i] = atomicAdd(&c.count[lin1], 1u);
    }
}

// How crowded it is around a scene's bodies, for the choice of its grid
// levels: the number of bodies in each body's cube of cells (consecutive in
// their brick, so two reads of the scan), summed.  A block adds its sum once
// where there is one scene; a batch's waves add theirs to their scene's word.
constexpr int kCrowdBlocks = 512;
template <bool BATCHED>
__global__ void __launch_bounds__(kBlock) k_crowd(GridArgs g, CellSortArgs c, unsigned long long* __restrict__ out)
{
    unsigned long long sum = 0ull;
    for (int i0 = blockIdx.x * blockDim.x; i0 < g.nslots; i0 += gridDim.x * blockDim.x) {
        const int i = i0 + threadIdx.x;
        const bool valid = i < g.nslots;
        const int s = BATCHED && valid ? (int)g.bod.scene[i] : 0;
        unsigned long long n = 0ull;
        if (valid) {
            const SceneParams& P = BATCHED ? g.scenes[s] : g.scene0;
            const int m = 3 * P.crowd_bits;
            const uint32_t off = (uint32_t)P.cell_offset;
            const uint32_t cube = off + (((c.cell[i] - off) >> m) << m);
            n = c.start[cube + (1u << m)] - c.start[cube];
        }
        if (!BATCHED) {
            sum += n;
            continue;
        }
        const int s0 = __shfl(s, 0, 64);
        if (__all(!valid || s == s0)) {
            for (int w = 32; w > 0; w >>= 1) n += __shfl_down(n, w, 64);
            if ((threadIdx.x & 63) == 0 && valid) atomicAdd(&out[s], n);
        } else if (valid) {
            atomicAdd(&out[s], n);
        }
    }
    if (BATCHED) return;
    for (int w = 32; w > 0; w >>= 1) sum += __shfl_down(sum, w, 64);
    __shared__ unsigned long long sh[kBlock / 64];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) sum += sh[w];
        atomicAdd(out, sum);
    }
}

__global__ void __launch_bounds__(kBlock) k_cell_bucket(GridArgs g, CellSortArgs c)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.nslots) return;
    c.bucket[c.start[c.cell[i]] + c.arrival[i]] = (uint32_t)i;
}

// ----------------------------------------------------------------- permute

// One thread per place of the bucket order: the body there moves to its rank
// by old slot in its cell.  Also clears the next pair list's range of every body
// (a body without pairs keeps the empty one).
template <bool BATCHED>
__global__ void __launch_bounds__(kBlock) k_permute(GridArgs g, CellSortArgs c, Bodies dst, int periodic,
                                                    int32_t* __restrict__ slot_of_id, int32_t* __restrict__ own_begin,
                                                    int32_t* __restrict__ own_count)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= g.nslots) return;
    const Bodies& src = g.bod;
    const uint32_t o = c.bucket[t];
    const int32_t id = src.id[o];
    const uint32_t lin = c.cell[o];
    const uint32_t beg = c.start[lin], end = c.start[lin + 1];
    const double4 xr = src.xr[o];
    uint32_t i = beg;
    for (uint32_t q = beg; q < end; ++q) i += c.bucket[q] < o ? 1u : 0u;
    dst.xr[i] = xr;
    const double4 v = src.vm[o];
    dst.vm[i] = make_double4(v.x, v.y, v.z, 0.0);  // a fresh Verlet account after every broad-phase run
    dst.w[i] = src.w[o];
    dst.q[i] = src.q[o];
    dst.mat[i] = src.mat[o];
    dst.blocked[i] = src.blocked[o];
    dst.id[i] = id;
    if (BATCHED) dst.scene[i] = src.scene[o];
    if (periodic) dst.period[i] = src.period[o];
    slot_of_id[id] = (int32_t)i;
    own_begin[id] = 0;
    own_count[id] = 0;
    if (c.nlarge > 0) {
        const SceneParams& P = BATCHED ? g.scenes[src.scene[o]] : g.scene0;
        if (level_of_radius(P, xr.w) == 1)
            c.large_slot[c.start[c.cell1[o]] - (uint32_t)g.nslots + c.arrival1[o]] = i;
    }
}

// ------------------------------------------------------------------- sweep

// A neighbour cell's index along one axis, wrapped into [0, dim) with the
// period crossed in w; outside an aperiodic grid the cell does not exist.
template <bool PERIODIC>
__device__ inline void wrap_axis(int& n, int dim, int& w, bool& skip)
{
    if (n < 0) {
        if (!PERIODIC) skip = true;
        n += dim;
        w = -1;
    } else if (n >= dim) {
        if (!PERIODIC) skip = true;
        n -= dim;
        w = 1;
    }
}

// Visit every candidate of home slot i (27 cells, then the scene's walls).
// f(partner_slot_or_wall, partner_id, packed_cell) is called per candidate.
// LANES lanes of a wave share one sphere's search: lane `part` visits every
// LANES-th group of cells, and every LANES-th wall.
template <bool BATCHED, bool PERIODIC, int LANES = 1, typename F>
__device__ inline void for_each_candidate(const SweepArgs& a, int i, F&& f, int part = 0)
{
    const GridArgs& g = a.g;
    const Bodies& B = g.bod;
    const int s = BATCHED ? (int)B.scene[i] : 0;
    const SceneParams& P = BATCHED ? g.scenes[s] : g.scene0;
    const double4 pi = B.xr[i];
    const double xi = pi.x, yi = pi.y, zi = pi.z, ri = pi.w;
    const int32_t myid = B.id[i];
    const double reach = 2.0 * P.verlet;
    // level 0 holds every sphere; with two levels a sphere takes its
    // partners up to r_split there and the larger ones from level 1
    const bool two = P.r_split > 0.0;
    const int nlev = two ? 2 : 1;
    for (int lv = 0; lv < nlev; ++lv) {
    const Level V = level_of(P, lv);
    int c[3], per_i[3];
    cell_of<PERIODIC>(P, V, xi, yi, zi, c, per_i);
    // cells of this level within reach of this body's largest possible
    // candidate distance on it (the largest radius it takes there)
    const double far = (ri + (lv == 0 && two ? P.r_split : P.rmax)) + reach;
    int kk[3];
    for (int q = 0; q < 3; ++q) kk[q] = max(1, (int)ceil(far / V.cellw[q]));
    // test one sphere j (position and radius pj, packed period perj, id idj)
    // found across the periods (w0, w1, w2) of the home cell's neighbourhood
    auto visit = [&](uint32_t j, const double4& pj, int32_t perj_packed, int32_t idj, int w0, int w1, int w2) {
        if ((int)j == i) return;
        const double rj = pj.w;
        if (lv == 0 && two && rj > P.r_split) return;  // found on level 1
        const double sc = (ri + rj) + reach;
        double ddx, ddy, ddz;
        int32_t packed = kCellZero;
        if (PERIODIC) {
            int perj[3];
            unpack_cell(perj_packed, perj);
            const int cc[3] = {per_i[0] - perj[0] + w0, per_i[1] - perj[1] + w1, per_i[2] - perj[2] + w2};
            packed = pack_cell(cc[0], cc[1], cc[2]);
            // evaluate from the lower id's side so that both bodies of
            // a pair take the same decision
            const bool from_i = myid < idj;
            const int sg = from_i ? 1 : -1;
            const double* H = P.H;
            const double sx = (H[0] * (sg * cc[0]) + H[1] * (sg * cc[1])) + H[2] * (sg * cc[2]);
            const double sy = (H[3] * (sg * cc[0]) + H[4] * (sg * cc[1])) + H[5] * (sg * cc[2]);
            const double sz = (H[6] * (sg * cc[0]) + H[7] * (sg * cc[1])) + H[8] * (sg * cc[2]);
            const double ax = from_i ? xi : pj.x, ay = from_i ? yi : pj.y, az = from_i ? zi : pj.z;
            const double bx = from_i ? pj.x : xi, by = from_i ? pj.y : yi, bz = from_i ? pj.z : zi;
            ddx = (bx + sx) - ax;
            ddy = (by + sy) - ay;
            ddz = (bz + sz) - az;
        } else {
            ddx = pj.x - xi;
            ddy = pj.y - yi;
            ddz = pj.z - zi;
        }
        const double dd = (ddx * ddx + ddy * ddy) + ddz * ddz;
        if (dd < sc * sc) f((int32_t)j, idj, packed);
    };
    // one group of cells: up to three along x from (dx0, dy, dz); their
    // ranges are loaded together, then their spheres are visited as one
    // sequence, two at a time (the loads of both are issued before either
    // is tested); of `of` lanes that share the group, lane `mine` takes every
    // of-th two
    auto group = [&](int dz, int dy, int dx0, int mine, int of) {
        int ny = c[1] + dy, nz = c[2] + dz, wy = 0, wz = 0;
        bool skip_row = false;
        wrap_axis<PERIODIC>(ny, V.dims[1], wy, skip_row);
        wrap_axis<PERIODIC>(nz, V.dims[2], wz, skip_row);
        if (skip_row) return;
        const uint32_t row = cell_index_yz(V, ny, nz);
        uint32_t st[3], en[3];
        int wx[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            int nx = c[0] + dx0 + t;
            bool skip = dx0 + t > kk[0];
            wx[t] = 0;
            wrap_axis<PERIODIC>(nx, V.dims[0], wx[t], skip);
            st[t] = en[t] = 0;
            if (!skip) {
                const uint32_t lin = row + cell_index_x(V, nx);
                st[t] = a.cell_start[lin];
                en[t] = a.cell_start[lin + 1];
            }
        }
        const uint32_t c0 = en[0] - st[0], c1 = en[1] - st[1], c2 = en[2] - st[2];
        const uint32_t tot = c0 + c1 + c2;
        auto at = [&](uint32_t k, int& wk) -> uint32_t {
            uint32_t q;
            if (k < c0) {
                q = st[0] + k;
                wk = wx[0];
            } else if (k < c0 + c1) {
                q = st[1] + (k - c0);
                wk = wx[1];
            } else {
                q = st[2] + (k - c0 - c1);
                wk = wx[2];
            }
            return lv == 0 ? q : g.large_slot[q - (uint32_t)g.nslots];
        };
        for (uint32_t k = 2u * mine; k < tot; k += 2u * of) {
            const bool two_here = k + 1 < tot;
            int wa, wb;
            const uint32_t ja = at(k, wa);
            const uint32_t jb = at(two_here ? k + 1 : k, wb);
            const double4 pa = B.xr[ja], pb = B.xr[jb];
            const int32_t pera = PERIODIC ? B.period[ja] : 0, perb = PERIODIC ? B.period[jb] : 0;
            const int32_t ida = B.id[ja], idb = B.id[jb];
            visit(ja, pa, pera, ida, wa, wy, wz);
            if (two_here) visit(jb, pb, perb, idb, wb, wy, wz);
        }
    };
    if (LANES > 1) {
        // group gi = ((dz * ndy) + dy) * nch + chunk, lane `part` taking
        // every LANES-th, so that the lanes search at the same time.  The
        // groups left when there are fewer than lanes are shared in turn: with
        // nine groups on four lanes the ninth alone would make three rounds of
        // two and a quarter, and where cells are crowded the time is in the
        // tests, not in the chain of reads (185,000 spheres, 240 in a cell:
        // 9.5 -> 8.4 ms per run)
        const int nch = (2 * kk[0] + 3) / 3, ndy = 2 * kk[1] + 1, ng = nch * ndy * (2 * kk[2] + 1);
        const int left = ng % LANES, whole = ng - left;
        auto nth = [&](int gi, int mine, int of) {
            const int ch = gi % nch, r = gi / nch;
            group(r / ndy - kk[2], r % ndy - kk[1], 3 * ch - kk[0], mine, of);
        };
        for (int gi = part; gi < whole; gi += LANES) nth(gi, 0, 1);
        if (left) {
            const int of = LANES / left, gi = whole + part / of;
            if (gi < ng) nth(gi, part % of, of);
        }
    } else {
        for (int dz = -kk[2]; dz <= kk[2]; ++dz)
            for (int dy = -kk[1]; dy <= kk[1]; ++dy)
                for (int dx0 = -kk[0]; dx0 <= kk[0]; dx0 += 3) group(dz, dy, dx0, 0, 1);
    }
    }
    for (int k = part; k < P.wall_count; k += LANES) {
        const int wi = P.wall_begin + k;
        const Wall W = a.walls[wi];
        if (W.kind == kPlane) {
            const double xa = W.axis == 0 ? xi : (W.axis == 1 ? yi : zi);
            const double delta = xa - W.pos;
            if (fabs(delta) < ri + reach) f(-1 - wi, W.id, kCellZero);
        } else {
            // box or facet: closer than r + 2 Delta L to the primitive
            const double x[3] = {xi, yi, zi};
            if (boundary_distance(W, x) < ri + reach) f(-1 - wi, W.id, kCellZero);
        }
    }
}

// The sweeps run in two passes when a scene has two levels: the spheres of
// level 0 first (a large sphere's lanes return at once), then the large ones
// through their index array, one per wave (a large sphere searches many more
// cells, which the wave's lanes share).  On level 0 a sphere takes LANES
// lanes: the search is a chain of dependent loads, nine groups of cells long
// in the plain grid, so a scene too small to fill the chip with a sphere per
// lane shares each search among as many lanes as fill it (sweep_lanes).
template <bool BATCHED, int LANES>
__device__ inline int sweep_body(const SweepArgs& a)
{
    const int t = (blockIdx.x * blockDim.x + threadIdx.x) / LANES;
    if (t >= a.g.nslots) return -1;
    if (a.nlarge > 0) {
        const int s = BATCHED ? (int)a.g.bod.scene[t] : 0;
        const SceneParams& P = BATCHED ? a.g.scenes[s] : a.g.scene0;
        if (level_of_radius(P, a.g.bod.xr[t].w) == 1) return -1;
    }
    return t;
}

template <bool BATCHED, bool PERIODIC, int LANES>
__global__ void __launch_bounds__(kBlock) k_sweep_count(SweepArgs a)
{
    const int i = sweep_body<BATCHED, LANES>(a);
    if (i < 0) return;
    const int part = threadIdx.x % LANES;
    uint32_t n = 0;
    for_each_candidate<BATCHED, PERIODIC, LANES>(a, i, [&](int32_t, int32_t, int32_t) { ++n; }, part);
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1) n += __shfl_down(n, off, LANES);
    if (part == 0) a.count[i] = n;
}

// The level-1 sphere of a wave (-1 past the last: the whole wave returns).
__device__ inline int large_sphere_of_wave(const SweepArgs& a)
{
    const int t = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    return t < a.nlarge ? (int)a.g.large_slot[t] : -1;
}

template <bool BATCHED, bool PERIODIC>
__global__ void __launch_bounds__(kBlock) k_sweep_count_large(SweepArgs a)
{
    const int i = large_sphere_of_wave(a);
    if (i < 0) return;
    const int lane = threadIdx.x & 63;
    uint32_t n = 0;
    for_each_candidate<BATCHED, PERIODIC, 64>(a, i, [&](int32_t, int32_t, int32_t) { ++n; }, lane);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n += __shfl_down(n, off, 64);
    if (lane == 0) a.count[i] = n;
}

// How each row was left by the fill, kept in `count` (the counts are spent
// once the rows are laid out): already sorted, in the order found (sorted by
// the rank pass), or a level-1 row in the order found (sorted by the wave
// rank pass).
constexpr uint32_t kRowSorted = 0, kRowFound = 1, kRowLarge = 2;

// LDS pool of the level-0 fill: 8 entries per sphere of the block on
// average (24 KB, so that the six blocks per CU its registers allow fit).
constexpr int kStageEntries = 8 * kBlock;

// (partner id, packed image as unsigned) as one unsigned key
__device__ inline uint64_t row_key(int32_t pid, int32_t cell)
{
    return ((uint64_t)((uint32_t)pid ^ 0x80000000u) << 32) | (uint32_t)cell;
}

// Whether this run's entries (and pairs) fit what the host sized the buffers
// and launches for; if not, every later kernel of the run returns at once
// and the host runs them again with the sizes it reads back.
__device__ inline bool entries_fit(const SweepArgs& a) { return *a.nent_dev <= (uint32_t)a.lim_ent; }

// The level-0 fill.  The rows of a block's spheres are contiguous, and the
// block takes them, in slot order, into its LDS pool while they fit: such a
// sweep stores nothing to memory (a store inside its loop would hold every
// later load until the store is done), then ranks its row in LDS and writes
// it sorted.  A row beyond the pool is written in the order found and
// sorted by the rank pass.  The lanes that share a sphere take the next
// place of its row from a counter in LDS (the order found does not matter).
template <bool BATCHED, bool PERIODIC, int LANES>
__global__ void __launch_bounds__(kBlock) k_sweep_fill_staged(SweepArgs a)
{
    __shared__ int32_t s_slot[kStageEntries];
    __shared__ int32_t s_pid[kStageEntries];
    __shared__ int32_t s_cell[kStageEntries];
    __shared__ uint32_t s_wave[kBlock / 64];
    __shared__ int32_t s_found[kBlock / LANES];
    if (!entries_fit(a)) return;
    const int i = sweep_body<BATCHED, LANES>(a);
    const int part = threadIdx.x % LANES, own = threadIdx.x / LANES;
    int beg = 0, len = 0;
    if (i >= 0) {
        beg = a.row_start[i];
        len = a.row_start[i + 1] - beg;
    }
    // the block's exclusive scan of the row lengths, in slot order (a
    // sphere's first lane brings its length)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = part == 0 ? (uint32_t)len : 0u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    if (lane == 63) s_wave[wave] = inc;
    if (part == 0) s_found[own] = 0;
    __syncthreads();
    uint32_t base = 0;
    for (int w = 0; w < wave; ++w) base += s_wave[w];
    if (i < 0) return;
    const uint32_t off = base + inc - (uint32_t)len;
    const bool staged = off + (uint32_t)len <= (uint32_t)kStageEntries;
    int mine = 0;
    for_each_candidate<BATCHED, PERIODIC, LANES>(a, i, [&](int32_t slot, int32_t pid, int32_t cell) {
        const int n = LANES == 1 ? mine++ : atomicAdd(&s_found[own], 1);
        if (n < len) {
            if (staged) {
                s_slot[off + n] = slot;
                s_pid[off + n] = pid;
                s_cell[off + n] = cell;
            } else {
                a.raw_slot[beg + n] = slot;
                a.raw_pid[beg + n] = pid;
                a.raw_cell[beg + n] = cell;
            }
        }
    }, part);
    for (int e = part; e < len; e += LANES) a.ent_body[beg + e] = i;
    if (part == 0) a.count[i] = staged ? kRowSorted : kRowFound;
    if (!staged) return;
    if (LANES > 1) {
        // the sphere's lanes are in one wave: their LDS writes are complete
        // before any of them ranks the row
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    const int32_t myid = a.g.bod.id[i];
    for (int e = part; e < len; e += LANES) {
        const int32_t slot = s_slot[off + e], pid = s_pid[off + e], cell = s_cell[off + e];
        const uint64_t ke = row_key(pid, cell);
        int rank = 0;
        for (int f = 0; f < len; ++f) {
            const uint64_t kf = row_key(s_pid[off + f], s_cell[off + f]);
            rank += (kf < ke || (kf == ke && f < e)) ? 1 : 0;
        }
        const int dst = beg + rank;
        a.ent_slot[dst] = slot;
        a.ent_pid[dst] = pid;
        a.ent_cell[dst] = cell;
        a.ent_own[dst] = (slot < 0 || myid < pid) ? 1u : 0u;
    }
}

// The level-1 fill, one wave per sphere: each lane counts the candidates
// of its groups of cells, then writes them after those of the lanes before
// it (the row is sorted afterwards, so this order only has to be complete).
template <bool BATCHED, bool PERIODIC>
__global__ void __launch_bounds__(kBlock) k_sweep_fill_large(SweepArgs a)
{
    if (!entries_fit(a)) return;
    const int i = large_sphere_of_wave(a);
    if (i < 0) return;
    const int lane = threadIdx.x & 63;
    uint32_t mine = 0;
    for_each_candidate<BATCHED, PERIODIC, 64>(a, i, [&](int32_t, int32_t, int32_t) { ++mine; }, lane);
    uint32_t inc = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    const int beg = a.row_start[i];
    const int cap = a.row_start[i + 1] - beg;
    int n = (int)(inc - mine);
    for_each_candidate<BATCHED, PERIODIC, 64>(a, i, [&](int32_t slot, int32_t pid, int32_t cell) {
        if (n < cap) {
            a.raw_slot[beg + n] = slot;
            a.raw_pid[beg + n] = pid;
            a.raw_cell[beg + n] = cell;
            a.ent_body[beg + n] = i;
        }
        ++n;
    }, lane);
    if (lane == 0) a.count[i] = kRowLarge;
}

// One thread per entry of a level-0 row that the fill left in the order
// found: its place in its row sorted by (partner id, image as unsigned; ties
// by the order found, which cannot happen for distinct candidates) is the
// number of the row's entries before it in that order.  This order fixes the
// order of the force sum.
__global__ void __launch_bounds__(kBlock) k_row_rank(SweepArgs a)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (!entries_fit(a) || (uint32_t)e >= *a.nent_dev) return;
    const int i = a.ent_body[e];
    if (a.count[i] != kRowFound) return;
    const int beg = a.row_start[i], end = a.row_start[i + 1];
    const int32_t pid = a.raw_pid[e];
    const uint32_t cell = (uint32_t)a.raw_cell[e];
    int rank = 0;
    for (int f = beg; f < end; ++f) {
        const int32_t pf = a.raw_pid[f];
        const uint32_t cf = (uint32_t)a.raw_cell[f];
        rank += (pf < pid || (pf == pid && (cf < cell || (cf == cell && f < e)))) ? 1 : 0;
    }
    const int dst = beg + rank;
    const int32_t slot = a.raw_slot[e];
    a.ent_slot[dst] = slot;
    a.ent_pid[dst] = pid;
    a.ent_cell[dst] = (int32_t)cell;
    a.ent_own[dst] = (slot < 0 || a.g.bod.id[i] < pid) ? 1u : 0u;
}

// One wave per level-1 sphere: its row, the longest kind, ranked as above
// with the row's keys in LDS (a row longer than the wave's share is ranked
// from memory).
constexpr int kLargeRowLds = 1024;

__global__ void __launch_bounds__(kBlock) k_row_rank_large(SweepArgs a)
{
    __shared__ uint64_t s_key[kBlock / 64][kLargeRowLds];
    if (!entries_fit(a)) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int t = blockIdx.x * (kBlock / 64) + wave;
    if (t >= a.nlarge) return;  // the whole wave
    const int i = (int)a.g.large_slot[t];
    const int beg = a.row_start[i], len = a.row_start[i + 1] - beg;
    const bool in_lds = len <= kLargeRowLds;
    if (in_lds) {
        for (int f = lane; f < len; f += 64) s_key[wave][f] = row_key(a.raw_pid[beg + f], a.raw_cell[beg + f]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    const int32_t myid = a.g.bod.id[i];
    for (int e = lane; e < len; e += 64) {
        const int32_t slot = a.raw_slot[beg + e], pid = a.raw_pid[beg + e], cell = a.raw_cell[beg + e];
        const uint64_t ke = row_key(pid, cell);
        int rank = 0;
        if (in_lds) {
            for (int f = 0; f < len; ++f) {
                const uint64_t kf = s_key[wave][f];
                rank += (kf < ke || (kf == ke && f < e)) ? 1 : 0;
            }
        } else {
            for (int f = 0; f < len; ++f) {
                const uint64_t kf = row_key(a.raw_pid[beg + f], a.raw_cell[beg + f]);
                rank += (kf < ke || (kf == ke && f < e)) ? 1 : 0;
            }
        }
        const int dst = beg + rank;
        a.ent_slot[dst] = slot;
        a.ent_pid[dst] = pid;
        a.ent_cell[dst] = cell;
        a.ent_own[dst] = (slot < 0 || myid < pid) ? 1u : 0u;
    }
}

// -------------------------------------------------------- pairs and history

__device__ inline bool pairs_fit(const PairBuildArgs& a)
{
    return *a.nent_dev <= (uint32_t)a.lim_ent && *a.npairs_dev <= (uint32_t)a.lim_pairs;
}

// One thread per row entry: an owning entry writes its pair (canonical
// index = the scan of the owner flags) and its row entry; the other finds
// its pair by binary search in the partner's sorted row.  The first entry of
// a row also writes the body's range of owned pairs.
__global__ void __launch_bounds__(kBlock) k_pair_build(PairBuildArgs a)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (!pairs_fit(a) || (uint32_t)e >= *a.nent_dev) return;
    const int i = a.ent_body[e];
    const int32_t myid = a.bod.id[i];
    const int32_t slot = a.ent_slot[e];
    if (a.ent_own[e]) {
        const uint32_t k = a.own_scan[e];
        if (slot < 0) {
            // a wall pair: the wall is #1 and has no row
            a.ca[k] = slot;
            a.cb[k] = i;
            a.rows.ent[e] = k;
        } else {
            a.ca[k] = i;
            a.cb[k] = slot;
            a.rows.ent[e] = k | kNegSign;
        }
        a.hist_new.cell[k] = a.ent_cell[e];
        a.hist_new.pid[k] = a.ent_pid[e];
    } else {
        // the pair is owned by the partner: find this body in its row,
        // which is sorted by (partner id, packed image as unsigned)
        const uint32_t want = (uint32_t)neg_cell(a.ent_cell[e]);
        int lo = a.row_start[slot], hi = a.row_start[slot + 1];
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            const int32_t pm = a.ent_pid[mid];
            const uint32_t cm = (uint32_t)a.ent_cell[mid];
            if (pm < myid || (pm == myid && cm < want))
                lo = mid + 1;
            else
                hi = mid;
        }
        uint32_t k = kPairMask;
        if (lo < a.row_start[slot + 1] && a.ent_pid[lo] == myid && (uint32_t)a.ent_cell[lo] == want &&
            a.ent_own[lo])
            k = a.own_scan[lo];
        a.rows.ent[e] = k;
    }
    const int beg = a.row_start[i];
    if (e == beg) {
        const int end = a.row_start[i + 1];
        a.hist_new.own_begin[myid] = (int32_t)a.own_scan[beg];
        a.hist_new.own_count[myid] = (int32_t)(a.own_scan[end] - a.own_scan[beg]);
    }
}

// Per canonical pair: where its history sits in the previous list, and
// whether that history says the pair touched (a carried normal is a unit
// vector; a new pair starts with zero shear force and no normal).
__global__ void __launch_bounds__(kBlock) k_carry_find(PairBuildArgs a, int old_nbodies)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (!pairs_fit(a) || (uint32_t)k >= *a.npairs_dev) return;
    const int32_t sa = a.ca[k], sb = a.cb[k];
    const int32_t owner = sa >= 0 ? a.bod.id[sa] : a.bod.id[sb];
    const int32_t partner = a.hist_new.pid[k];
    const int32_t cell = a.hist_new.cell[k];
    int32_t found = -1;
    if (a.has_old && owner < old_nbodies) {
        const int lo = a.hist_old.own_begin[owner];
        const int cnt = a.hist_old.own_count[owner];
        for (int q = lo; q < lo + cnt; ++q) {
            if (a.hist_old.pid[q] == partner && a.hist_old.cell[q] == cell) {
                found = a.hist_old.map[q];
                break;
            }
        }
    }
    bool touched = false;
    if (found >= 0) {
        const HistRec h = a.hist_f32 ? widen(reinterpret_cast<const HistRec32*>(a.hist_old.h)[found])
                                     : a.hist_old.h[found];
        touched = h.nx != 0.0 || h.ny != 0.0 || h.nz != 0.0;
    }
    a.found[k] = found;
    a.flag[k] = touched ? 1u : 0u;
}

// The stable partition, within each eighth [P_x, P_x+1) of the pairs
// (P_x = x npairs / 8, the segment one XCD takes in the contact kernel) and
// within each chunk of kPartitionChunk pairs of it: touching pairs first,
// then the others, each group in canonical order; the history moves with its
// pair, and the canonical -> final map is kept for the next run.  Chunks keep
// a body's touching and non-touching pairs close in time in the contact
// kernel, so the positions the second group gathers are still cached.
__device__ inline uint32_t segment_start(int x, int npairs) { return (uint32_t)(((int64_t)x * npairs) >> 3); }
constexpr uint32_t kPartitionChunk = 1u << 14;

__global__ void __launch_bounds__(kBlock) k_partition(PairBuildArgs a)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (!pairs_fit(a) || (uint32_t)k >= *a.npairs_dev) return;
    const int npairs = (int)*a.npairs_dev;
    int x = (int)(((int64_t)k * 8) / npairs);
    if (x > 7) x = 7;
    while (x < 7 && (uint32_t)k >= segment_start(x + 1, npairs)) ++x;
    while (x > 0 && (uint32_t)k < segment_start(x, npairs)) --x;
    const uint32_t x0 = segment_start(x, npairs), x1 = segment_start(x + 1, npairs);
    const uint32_t p0 = x0 + (((uint32_t)k - x0) / kPartitionChunk) * kPartitionChunk;
    const uint32_t p1 = min(p0 + kPartitionChunk, x1);
    const uint32_t s0 = a.flag_scan[p0];
    const uint32_t ntouch = a.flag_scan[p1] - s0;
    const uint32_t r = a.flag_scan[k] - s0;
    const bool touched = a.flag[k] != 0u;
    const uint32_t pos = p0 + (touched ? r : ntouch + (((uint32_t)k - p0) - r));
    a.pr.a[pos] = a.ca[k];
    a.pr.b[pos] = a.cb[k];
    a.pr.cell[pos] = a.hist_new.cell[k];
    a.pr.pid[pos] = a.hist_new.pid[k];
    const int32_t f = a.found[k];
    if (a.hist_f32)
        reinterpret_cast<HistRec32*>(a.pr.h)[pos] =
            f >= 0 ? reinterpret_cast<const HistRec32*>(a.hist_old.h)[f] : HistRec32{};
    else
        a.pr.h[pos] = f >= 0 ? a.hist_old.h[f] : HistRec{};
    // the force of a pair that touched, for reports before the next step
    if (a.carry_frec && f >= 0) {
        for (int q = 0; q < kForceWords; ++q)
            if (a.hist_f32)
                a.pr.frecf[kForceWords * (size_t)pos + q] = static_cast<const float*>(a.hist_old.frec)[kForceWords * (size_t)f + q];
            else
                a.pr.frec[kForceWords * (size_t)pos + q] = static_cast<const double*>(a.hist_old.frec)[kForceWords * (size_t)f + q];
    }
    a.pr.real[pos] = touched ? 1 : 0;
    a.pr.ea[pos] = -1;  // set below from the rows (stays -1 for a boundary pair)
    a.pr.eb[pos] = -1;
    a.hist_new.map[k] = (int32_t)pos;
}

// Row entries: canonical pair index -> partitioned index (the side bit kept,
// the touched bit from the carried history); each pair learns where its
// entries sit, so that the contact kernel can update their touched bits.
__global__ void __launch_bounds__(kBlock) k_remap_rows(PairBuildArgs a)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (!pairs_fit(a) || (uint32_t)e >= *a.nent_dev) return;
    const uint32_t u = a.rows.ent[e];
    const uint32_t k = u & kPairMask;
    if (k < *a.npairs_dev) {
        const uint32_t pos = (uint32_t)a.hist_new.map[k];
        a.rows.ent[e] = (u & kNegSign) | (a.flag[k] ? kRealBit : 0u) | pos;
        if (u & kNegSign)
            a.pr.ea[pos] = e;
        else
            a.pr.eb[pos] = e;
    }
}

inline int nblocks(long n) { return (int)((n + kBlock - 1) / kBlock); }

}  // namespace

size_t bounds_temp_bytes() { return sizeof(unsigned long long) * 6 * kBoundsBlocks; }

void launch_bounds(const Bodies& b, int nslots, int nscenes, double* out6, void* temp, hipStream_t st)
{
    if (nslots > 0 && nscenes == 1) {
        // a block takes up to eight bodies per thread
        unsigned long long* part = static_cast<unsigned long long*>(temp);
        const int nblk = std::min(nblocks((nslots + 7L) / 8), kBoundsBlocks);
        hipLaunchKernelGGL(k_bounds_block, dim3(nblk), dim3(kBlock), 0, st, b, nslots, part, out6);
        if (nblk > 1) hipLaunchKernelGGL(k_bounds_final, dim3(1), dim3(kBlock), 0, st, part, nblk, out6);
        return;
    }
    // out6 doubles as the buffer of ordered bits (same size)
    unsigned long long* bits = reinterpret_cast<unsigned long long*>(out6);
    (void)hipMemsetAsync(bits, 0, sizeof(unsigned long long) * 6 * nscenes, st);
    // bodies are grouped by scene after the first run, so nearly every
    // wave is uniform and the atomics spread over the scenes
    if (nslots > 0) hipLaunchKernelGGL(k_bounds, dim3(nblocks(nslots)), dim3(kBlock), 0, st, b, nslots, 1, bits);
    hipLaunchKernelGGL(k_bounds_decode, dim3(nblocks(6 * nscenes)), dim3(kBlock), 0, st, bits, out6, 6 * nscenes);
}

void launch_cell_count(const GridArgs& g, const CellSortArgs& c, bool periodic, void* scan_temp, hipStream_t st)
{
    if (g.nslots <= 0) return;
    const bool batched = g.nscenes > 1;
    const dim3 grid(nblocks(g.nslots)), blk(kBlock);
    (void)hipMemsetAsync(c.count, 0, sizeof(uint32_t) * (size_t)c.ncells, st);
    if (batched)
        hipLaunchKernelGGL((k_cell_count<true, false>), grid, blk, 0, st, g, c);
    else if (periodic)
        hipLaunchKernelGGL((k_cell_count<false, true>), grid, blk, 0, st, g, c);
    else
        hipLaunchKernelGGL((k_cell_count<false, false>), grid, blk, 0, st, g, c);
    exclusive_scan_u32(c.count, c.start, c.ncells, nullptr, scan_temp, nullptr, st);
}

void launch_crowd(const GridArgs& g, const CellSortArgs& c, unsigned long long* crowd, hipStream_t st)
{
    if (g.nslots <= 0) return;
    const int nblk = nblocks(g.nslots);
    if (g.nscenes > 1)
        hipLaunchKernelGGL((k_crowd<true>), dim3(nblk), dim3(kBlock), 0, st, g, c, crowd);
    else
        hipLaunchKernelGGL((k_crowd<false>), dim3(std::min(nblk, kCrowdBlocks)), dim3(kBlock), 0, st, g, c, crowd);
}

void launch_cell_place(const GridArgs& g, const CellSortArgs& c, const Bodies& dst, bool periodic, int32_t* slot_of_id,
                       int32_t* own_begin, int32_t* own_count, hipStream_t st)
{
    if (g.nslots <= 0) return;
    const bool batched = g.nscenes > 1;
    const dim3 grid(nblocks(g.nslots)), blk(kBlock);
    hipLaunchKernelGGL(k_cell_bucket, grid, blk, 0, st, g, c);
    if (batched)
        hipLaunchKernelGGL((k_permute<true>), grid, blk, 0, st, g, c, dst, 0, slot_of_id, own_begin, own_count);
    else
        hipLaunchKernelGGL((k_permute<false>), grid, blk, 0, st, g, c, dst, periodic ? 1 : 0, slot_of_id, own_begin,
                           own_count);
}

// Lanes per sphere of the level-0 sweeps: as many as keep the launch within
// about the threads the chip holds at once (256 CUs x 2,048).  Measured
// (count + fill) with 1 lane and with the choice: 1,000 spheres 44 + 63 us ->
// 8.7 + 12.9 on 16 lanes, 200,000 72 + 87 -> 52 + 65 on 4; 8 M keep 1.
inline int sweep_lanes(int nslots) { return nslots <= 32768 ? 16 : (nslots <= 262144 ? 4 : 1); }

// The level-0 pass and, with two levels, the level-1 pass (one sphere per
// wave) of a sweep kernel pair.
#define DEM_SWEEP_SMALL(K, B, P, A, ST)                                                                        \
    do {                                                                                                      \
        const int lanes_ = sweep_lanes((A).g.nslots);                                                         \
        const dim3 g0_(nblocks((long)(A).g.nslots * lanes_)), b0_(kBlock);                                    \
        if (lanes_ == 16)                                                                                     \
            hipLaunchKernelGGL((K<B, P, 16>), g0_, b0_, 0, ST, A);                                            \
        else if (lanes_ == 4)                                                                                 \
            hipLaunchKernelGGL((K<B, P, 4>), g0_, b0_, 0, ST, A);                                             \
        else                                                                                                  \
            hipLaunchKernelGGL((K<B, P, 1>), g0_, b0_, 0, ST, A);                                             \
    } while (0)
#define DEM_SWEEP_LAUNCH(SMALL, LARGE_K, A, ST)                                                                \
    do {                                                                                                      \
        const dim3 blk(kBlock);                                                                               \
        const dim3 g1(((A).nlarge + kBlock / 64 - 1) / (kBlock / 64));                                        \
        if ((A).g.nscenes > 1) {                                                                              \
            DEM_SWEEP_SMALL(SMALL, true, false, A, ST);                                                       \
            if ((A).nlarge > 0) hipLaunchKernelGGL((LARGE_K<true, false>), g1, blk, 0, ST, A);                \
        } else if ((A).g.scene0.periodic) {                                                                   \
            DEM_SWEEP_SMALL(SMALL, false, true, A, ST);                                                       \
            if ((A).nlarge > 0) hipLaunchKernelGGL((LARGE_K<false, true>), g1, blk, 0, ST, A);                \
        } else {                                                                                              \
            DEM_SWEEP_SMALL(SMALL, false, false, A, ST);                                                      \
            if ((A).nlarge > 0) hipLaunchKernelGGL((LARGE_K<false, false>), g1, blk, 0, ST, A);               \
        }                                                                                                     \
    } while (0)

void launch_sweep_count(const SweepArgs& a, hipStream_t st)
{
    if (a.g.nslots <= 0) return;
    DEM_SWEEP_LAUNCH(k_sweep_count, k_sweep_count_large, a, st);
}

void launch_sweep_fill(const SweepArgs& a, hipStream_t st)
{
    if (a.g.nslots <= 0) return;
    DEM_SWEEP_LAUNCH(k_sweep_fill_staged, k_sweep_fill_large, a, st);
    if (a.lim_ent > 0) hipLaunchKernelGGL(k_row_rank, dim3(nblocks(a.lim_ent)), dim3(kBlock), 0, st, a);
    if (a.nlarge > 0)
        hipLaunchKernelGGL(k_row_rank_large, dim3((a.nlarge + kBlock / 64 - 1) / (kBlock / 64)), dim3(kBlock), 0, st,
                           a);
}

void launch_pair_build(const PairBuildArgs& a, hipStream_t st)
{
    if (a.lim_ent > 0) hipLaunchKernelGGL(k_pair_build, dim3(nblocks(a.lim_ent)), dim3(kBlock), 0, st, a);
}

void launch_carry_find(const PairBuildArgs& a, hipStream_t st, int old_nbodies)
{
    if (a.lim_pairs > 0)
        hipLaunchKernelGGL(k_carry_find, dim3(nblocks(a.lim_pairs)), dim3(kBlock), 0, st, a, old_nbodies);
}

void launch_partition(const PairBuildArgs& a, hipStream_t st)
{
    if (a.lim_pairs > 0) hipLaunchKernelGGL(k_partition, dim3(nblocks(a.lim_pairs)), dim3(kBlock), 0, st, a);
    if (a.lim_ent > 0) hipLaunchKernelGGL(k_remap_rows, dim3(nblocks(a.lim_ent)), dim3(kBlock), 0, st, a);
}

}  // namespace dem
