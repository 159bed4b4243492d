// state.hip -- the bodies' state between the library's order and the
// caller's: reports in id order (dem_get_state, dem_get_state_device), the
// state a caller sets, and the boundary pairs' forces for the reaction on
// each boundary.
//
// One thread per body of the caller's range.  The reads are gathers of one
// aligned 32-byte vector per quantity through the id -> slot map, the writes
// are contiguous over the wave.  Bound by memory: 128 bytes gathered and 104
// written per body.  Measured (one MI355X) as a pass of steps with one
// read-back into device tensors, against copying the four arrays to the host,
// sorting there and copying back: 30 steps of 8 M bodies 741 -> 75 ms, 200
// steps of 24 scenes (each reading the whole batch before) 64.6 -> 6.0 ms.
#include "dem_internal.hpp"

#include <algorithm>

namespace dem {

namespace {

constexpr int kBlock = 256;

// Reported position of a boundary along axis k: a plane's coordinate on its
// axis (0 elsewhere), a box's centre, a facet's centroid.
__device__ inline double boundary_position(const Wall& W, int k)
{
#pragma clang fp contract(off)
    if (W.kind == kPlane) return k == W.axis ? W.pos : 0.0;
    if (W.kind == kBox) return 0.5 * (W.g[k] + W.g[3 + k]);
    return (W.g[k] + W.g[3 + k] + W.g[6 + k]) / 3.0;
}

__device__ inline void store3(double* p, long i, double x, double y, double z)
{
    p[3 * i] = x;
    p[3 * i + 1] = y;
    p[3 * i + 2] = z;
}

__global__ void __launch_bounds__(kBlock) k_gather_state(StateArgs a, StateOut o)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.count) return;
    const int32_t gid = a.gids ? a.gids[a.first + i] : a.first + i;
    const int32_t s = a.slot_of_id[gid];
    if (s < 0) {
        // a boundary: it does not move; its reaction is the host's to fill in
        const Wall& W = a.walls[-1 - s];
        if (o.pos3) store3(o.pos3, i, boundary_position(W, 0), boundary_position(W, 1), boundary_position(W, 2));
        if (o.vel3) store3(o.vel3, i, 0.0, 0.0, 0.0);
        if (o.angvel3) store3(o.angvel3, i, 0.0, 0.0, 0.0);
        if (o.force3) store3(o.force3, i, 0.0, 0.0, 0.0);
        if (o.torque3) store3(o.torque3, i, 0.0, 0.0, 0.0);
        if (o.ori4) {
            o.ori4[4 * (long)i] = 1.0;
            store3(o.ori4 + 4 * (long)i + 1, 0, 0.0, 0.0, 0.0);
        }
        return;
    }
    if (o.pos3) {
        const double4 v = a.bod.xr[s];
        store3(o.pos3, i, v.x, v.y, v.z);
    }
    if (o.vel3) {
        const double4 v = a.bod.vm[s];
        store3(o.vel3, i, v.x, v.y, v.z);
    }
    if (o.angvel3) {
        const double4 v = a.bod.w[s];
        store3(o.angvel3, i, v.x, v.y, v.z);
    }
    if (o.ori4) {
        const double4 v = a.bod.q[s];
        double* p = o.ori4 + 4 * (long)i;
        p[0] = v.x;
        p[1] = v.y;
        p[2] = v.z;
        p[3] = v.w;
    }
    if (o.force3) {
        const double* f = a.slot_force3 + 3 * (long)s;
        store3(o.force3, i, a.slot_force3 ? f[0] : 0.0, a.slot_force3 ? f[1] : 0.0, a.slot_force3 ? f[2] : 0.0);
    }
    if (o.torque3) {
        const double* t = a.slot_torque3 + 3 * (long)s;
        store3(o.torque3, i, a.slot_torque3 ? t[0] : 0.0, a.slot_torque3 ? t[1] : 0.0, a.slot_torque3 ? t[2] : 0.0);
    }
}

// The other way: the radius and the Verlet account stay; boundaries are
// skipped.
__global__ void __launch_bounds__(kBlock) k_scatter_state(StateArgs a, StateIn in)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.count) return;
    const int32_t gid = a.gids ? a.gids[a.first + i] : a.first + i;
    const int32_t s = a.slot_of_id[gid];
    if (s < 0) return;
    const long j = 3 * (long)i;
    if (in.pos3) a.bod.xr[s] = make_double4(in.pos3[j], in.pos3[j + 1], in.pos3[j + 2], a.bod.xr[s].w);
    if (in.vel3) a.bod.vm[s] = make_double4(in.vel3[j], in.vel3[j + 1], in.vel3[j + 2], a.bod.vm[s].w);
    if (in.angvel3) a.bod.w[s] = make_double4(in.angvel3[j], in.angvel3[j + 1], in.angvel3[j + 2], 0.0);
    if (in.ori4) {
        const double* q = in.ori4 + 4 * (long)i;
        a.bod.q[s] = make_double4(q[0], q[1], q[2], q[3]);
    }
}

// New bodies (or all of them, after some were added): one thread per record
// as the host holds it, 144 bytes of which are read here and 142 written;
// bound by the copy that brings them.  A pass of steps on new bodies,
// against arrays picked apart on the host: 8 M 427 -> 127 ms, 1 M 67 -> 29,
// 500,000 33 -> 20.
__global__ void __launch_bounds__(kBlock) k_unpack_bodies(const HostBody* __restrict__ raw, int first, int n,
                                                          const int32_t* __restrict__ fixed, int nfixed, Bodies out,
                                                          int32_t* __restrict__ slot_of_id)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const HostBody& b = raw[i];
    const int32_t gid = first + i;
    if (b.kind != 0) {
        slot_of_id[gid] = -1 - b.wall;
        return;
    }
    int lo = 0, hi = nfixed;  // boundaries before it
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (fixed[mid] < gid)
            lo = mid + 1;
        else
            hi = mid;
    }
    const int s = gid - lo;
    slot_of_id[gid] = s;
    out.xr[s] = make_double4(b.x[0], b.x[1], b.x[2], b.r);
    out.vm[s] = make_double4(b.v[0], b.v[1], b.v[2], 0.0);  // fresh Verlet account
    out.w[s] = make_double4(b.w[0], b.w[1], b.w[2], 0.0);
    out.q[s] = make_double4(b.q[0], b.q[1], b.q[2], b.q[3]);
    out.mat[s] = (uint16_t)b.mat;
    out.blocked[s] = b.blocked;
    out.id[s] = gid;
    out.scene[s] = (uint16_t)b.scene;
}

// A read-back of a few kilobytes: one block copies them and posts that they
// are there.  With a copy for each array and a wait for the stream a broad-phase
// run took some 35 us longer (a column of 71,000 spheres, 500 steps with about
// 5 runs: 7.70 ms, now 7.54).
constexpr int kPostBlock = 1024;
__global__ void __launch_bounds__(kPostBlock) k_post(PostArgs p, uint32_t* __restrict__ flag, uint32_t seq)
{
    for (int q = 0; q < 3; ++q)
        for (uint32_t i = threadIdx.x; i < p.words[q]; i += blockDim.x)
            static_cast<uint2*>(p.dst[q])[i] = static_cast<const uint2*>(p.src[q])[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// flag[k] = 1 for a boundary pair that touched at the last step, 0 at k =
// npairs (the scan's extra entry)
template <int PREC>
__global__ void __launch_bounds__(kBlock) k_wall_flags(StepArgs a, uint32_t* __restrict__ flag)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > a.npairs) return;
    bool touched = false;
    if (k < a.npairs && a.pr.a[k] < 0) {
        const HistRec h = hist_load<PREC>(a.pr.h, k);
        touched = h.nx != 0.0 || h.ny != 0.0 || h.nz != 0.0;
    }
    flag[k] = touched ? 1u : 0u;
}

// the flagged pairs' boundary and force, in pair order (4 doubles each)
__global__ void __launch_bounds__(kBlock) k_wall_pack(StepArgs a, const uint32_t* __restrict__ flag,
                                                      const uint32_t* __restrict__ scan,
                                                      const double* __restrict__ f3, double* __restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.npairs || !flag[k]) return;
    double* o = out + 4 * (size_t)scan[k];
    o[0] = (double)(-1 - a.pr.a[k]);
    for (int q = 0; q < 3; ++q) o[1 + q] = f3[3 * (size_t)k + q];
}

inline dim3 blocks(long n) { return dim3((unsigned)((n + kBlock - 1) / kBlock)); }

}  // namespace

void launch_unpack_bodies(const HostBody* raw, int first, int n, const int32_t* fixed, int nfixed, const Bodies& b,
                          int32_t* slot_of_id, hipStream_t st)
{
    if (n > 0)
        hipLaunchKernelGGL(k_unpack_bodies, blocks(n), dim3(kBlock), 0, st, raw, first, n, fixed, nfixed, b, slot_of_id);
}

void launch_post(const PostArgs& p, uint32_t* flag, uint32_t seq, hipStream_t st)
{
    const uint32_t most = std::max({p.words[0], p.words[1], p.words[2]});
    const int block = most <= 64 ? 64 : kPostBlock;
    hipLaunchKernelGGL(k_post, dim3(1), dim3(block), 0, st, p, flag, seq);
}

void launch_gather_state(const StateArgs& a, const StateOut& o, hipStream_t st)
{
    if (a.count > 0) hipLaunchKernelGGL(k_gather_state, blocks(a.count), dim3(kBlock), 0, st, a, o);
}

void launch_scatter_state(const StateArgs& a, const StateIn& in, hipStream_t st)
{
    if (a.count > 0) hipLaunchKernelGGL(k_scatter_state, blocks(a.count), dim3(kBlock), 0, st, a, in);
}

void launch_wall_flags(const StepArgs& a, int precision, uint32_t* flag, hipStream_t st)
{
    if (precision == DEM_FP32_MIXED)
        hipLaunchKernelGGL(k_wall_flags<DEM_FP32_MIXED>, blocks((long)a.npairs + 1), dim3(kBlock), 0, st, a, flag);
    else
        hipLaunchKernelGGL(k_wall_flags<DEM_FP64>, blocks((long)a.npairs + 1), dim3(kBlock), 0, st, a, flag);
}

void launch_wall_pack(const StepArgs& a, const uint32_t* flag, const uint32_t* scan, const double* f3, double* out,
                      hipStream_t st)
{
    if (a.npairs > 0) hipLaunchKernelGGL(k_wall_pack, blocks(a.npairs), dim3(kBlock), 0, st, a, flag, scan, f3, out);
}

}  // namespace dem
