// prim.hip -- device primitive for gfx950 (wave64): exclusive scan of u32,
// over a count the host knows or one that is still on the device.
//
// Up to kOneBlock elements take one launch of one block; more take three:
// the tiles' sums, their scan by one block, the tiles' scans.  Threads read
// and write eight consecutive elements as two 16-byte vectors.
#include "dem_internal.hpp"

namespace dem {

namespace {

constexpr int kBlock = 256;           // 4 wavefronts of 64
constexpr int kTopBlock = 1024;       // the one-block kernels
constexpr int kItems = 8;             // consecutive elements per thread
constexpr int kTile = kBlock * kItems;
constexpr int kOneBlock = 2 * kTopBlock * kItems;

// Sums saturate, so that a total past 2^32 - 1 is not taken for a small one:
// the caller abandons the run then, and the places scanned are not used.
__device__ inline uint32_t sat_add(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }

__device__ inline uint32_t wave_inclusive_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t y = __shfl_up(v, off, 64);
        if (lane >= off) v = sat_add(v, y);
    }
    return v;
}

// Exclusive scan of one value per thread over the block; returns the block total in *total.
template <int BLOCK>
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* total)
{
    __shared__ uint32_t wave_tot[BLOCK / 64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    uint32_t inc = wave_inclusive_scan(v);
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) {
        uint32_t t = wave_tot[w];
        if (w < wave) before = sat_add(before, t);
        all = sat_add(all, t);
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

// n = *n_dev where it is given and does not exceed n_max (a larger one means
// that the run is abandoned: nothing is scanned), else n_max
__device__ inline int scan_length(int n_max, const uint32_t* n_dev)
{
    if (!n_dev) return n_max;
    const uint32_t n = *n_dev;
    return n <= (uint32_t)n_max ? (int)n : 0;
}

// the kItems elements from i on (0 past the end); arrays are 16-byte aligned
__device__ inline uint32_t load_items(const uint32_t* __restrict__ in, long i, int n, uint32_t* v)
{
    if (i + kItems <= n) {
        const uint4 a = *reinterpret_cast<const uint4*>(in + i), b = *reinterpret_cast<const uint4*>(in + i + 4);
        v[0] = a.x;
        v[1] = a.y;
        v[2] = a.z;
        v[3] = a.w;
        v[4] = b.x;
        v[5] = b.y;
        v[6] = b.z;
        v[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < kItems; ++k) v[k] = i + k < n ? in[i + k] : 0u;
    }
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) s = sat_add(s, v[k]);
    return s;
}

// their exclusive scan from `run` on; the thread holding the last element
// also writes the total at out[n]
__device__ inline void store_items(uint32_t* __restrict__ out, long i, int n, uint32_t run, const uint32_t* v)
{
    uint32_t o[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        o[k] = run;
        run += v[k];
    }
    if (i + kItems <= n) {
        *reinterpret_cast<uint4*>(out + i) = make_uint4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<uint4*>(out + i + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
        for (int k = 0; k < kItems; ++k)
            if (i + k < n) out[i + k] = o[k];
    }
    if (i < n && i + kItems >= n) out[n] = run;
}

__global__ void __launch_bounds__(kTopBlock) k_scan_one(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                        int n_max, const uint32_t* __restrict__ n_dev,
                                                        uint32_t* __restrict__ total_dev)
{
    const int n = scan_length(n_max, n_dev);
    uint32_t carry = 0;
    for (int c = 0; c < n; c += kTopBlock * kItems) {
        const long i = c + (long)threadIdx.x * kItems;
        uint32_t v[kItems], tot;
        const uint32_t s = load_items(in, i, n, v);
        const uint32_t ex = block_exclusive_scan<kTopBlock>(s, &tot);
        store_items(out, i, n, carry + ex, v);
        carry = sat_add(carry, tot);
    }
    if (threadIdx.x == 0) {
        if (n == 0) out[0] = 0u;
        if (total_dev) *total_dev = carry;
    }
}

__global__ void __launch_bounds__(kBlock) k_scan_reduce(const uint32_t* __restrict__ in, int n_max,
                                                        const uint32_t* __restrict__ n_dev,
                                                        uint32_t* __restrict__ sums)
{
    const int n = scan_length(n_max, n_dev);
    uint32_t v[kItems], total;
    block_exclusive_scan<kBlock>(load_items(in, (long)blockIdx.x * kTile + (long)threadIdx.x * kItems, n, v), &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// One block scans the tiles' sums in place.
__global__ void __launch_bounds__(kTopBlock) k_scan_top(uint32_t* __restrict__ sums, int nsums,
                                                        uint32_t* __restrict__ out,
                                                        int n_max, const uint32_t* __restrict__ n_dev,
                                                        uint32_t* __restrict__ total_dev)
{
    uint32_t carry = 0;
    for (int c = 0; c < nsums; c += kTopBlock) {
        const int i = c + (int)threadIdx.x;
        const uint32_t v = i < nsums ? sums[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan<kTopBlock>(v, &tot);
        if (i < nsums) sums[i] = carry + ex;
        carry = sat_add(carry, tot);
    }
    if (threadIdx.x == 0) {
        if (scan_length(n_max, n_dev) == 0) out[0] = 0u;
        if (total_dev) *total_dev = carry;
    }
}

__global__ void __launch_bounds__(kBlock) k_scan_down(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                      int n_max, const uint32_t* __restrict__ n_dev,
                                                      const uint32_t* __restrict__ sums)
{
    const int n = scan_length(n_max, n_dev);
    const long i = (long)blockIdx.x * kTile + (long)threadIdx.x * kItems;
    uint32_t v[kItems], total;
    const uint32_t s = load_items(in, i, n, v);
    const uint32_t ex = block_exclusive_scan<kBlock>(s, &total);
    store_items(out, i, n, sums[blockIdx.x] + ex, v);
}

inline int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

}  // namespace

size_t scan_temp_bytes(int n) { return sizeof(uint32_t) * (size_t)(ceil_div(n, kTile) + 1); }

void exclusive_scan_u32(const uint32_t* in, uint32_t* out, int n_max, const uint32_t* n_dev, void* temp,
                        uint32_t* total_dev, hipStream_t st)
{
    if (n_max <= kOneBlock) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kTopBlock), 0, st, in, out, n_max, n_dev, total_dev);
        return;
    }
    const int nblk = ceil_div(n_max, kTile);
    uint32_t* sums = static_cast<uint32_t*>(temp);
    hipLaunchKernelGGL(k_scan_reduce, dim3(nblk), dim3(kBlock), 0, st, in, n_max, n_dev, sums);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kTopBlock), 0, st, sums, nblk, out, n_max, n_dev, total_dev);
    hipLaunchKernelGGL(k_scan_down, dim3(nblk), dim3(kBlock), 0, st, in, out, n_max, n_dev, sums);
}

}  // namespace dem
