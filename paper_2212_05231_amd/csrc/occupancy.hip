// Occupancy grid and ray marcher (arXiv 2212.05231, supplement Sec. E.3 "Ray Marching
// Acceleration"; the grid is kept as in the publication that passage cites: a density value per
// cell, decayed, raised at candidate cells, thresholded into one bit per cell, cells numbered
// along the Morton curve).
//
// Which lattice points of a ray become samples is an integer decision taken from binary32
// arithmetic.  Every operation that feeds it is a single rounded operation in a fixed order
// (no fused multiply-add anywhere in this file), so that the kept set can be reproduced bit for
// bit by any IEEE implementation.
#include <algorithm>

#include "common.h"

#pragma clang fp contract(off)

namespace neus2 {
namespace {

constexpr int kThreads = 256;
constexpr int kScanThreads = 1024;

// 8 coordinate bits -> bits 0, 3, 6, ..., 21
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v = (v | (v << 8)) & 0x00F00Fu;
    v = (v | (v << 4)) & 0x0C30C3u;
    v = (v | (v << 2)) & 0x249249u;
    return v;
}

__device__ __forceinline__ uint32_t gather3(uint32_t v) {
    v &= 0x249249u;
    v = (v | (v >> 2)) & 0x0C30C3u;
    v = (v | (v >> 4)) & 0x00F00Fu;
    v = (v | (v >> 8)) & 0xFFu;
    return v;
}

// Sample point of a candidate cell: (cell coordinate + jitter) / G.
__global__ __launch_bounds__(kThreads) void cell_points_kernel(int log2_res, const int32_t* __restrict__ cells,
                                                               const float* __restrict__ jitter, int64_t m,
                                                               float* __restrict__ pos) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= m) return;
    const uint32_t mask = (1u << (3 * log2_res)) - 1u;
    const uint32_t code = (uint32_t)cells[i] & mask;
    const float inv = 1.0f / (float)(1 << log2_res);           // a power of two: exact
    pos[3 * i + 0] = ((float)gather3(code) + jitter[3 * i + 0]) * inv;
    pos[3 * i + 1] = ((float)gather3(code >> 1) + jitter[3 * i + 1]) * inv;
    pos[3 * i + 2] = ((float)gather3(code >> 2) + jitter[3 * i + 2]) * inv;
}

__global__ __launch_bounds__(kThreads) void decay_kernel(float* __restrict__ density, int64_t count, float decay) {
    const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
    if (i + 3 < count) {
        float4 v = *reinterpret_cast<float4*>(density + i);
        v.x *= decay, v.y *= decay, v.z *= decay, v.w *= decay;
        *reinterpret_cast<float4*>(density + i) = v;
    }
}

__device__ __forceinline__ float logistic_density(float sdf, float s) {
    const float e = expf(-s * fabsf(sdf));
    return s * e / ((1.0f + e) * (1.0f + e));
}

// density[cell] = max(density[cell], phi_s(sdf)).  Densities are never negative, so their bit
// patterns order like unsigned integers and one integer atomic maximum does it.
__global__ __launch_bounds__(kThreads) void raise_kernel(float* __restrict__ density, int64_t count,
                                                         const int32_t* __restrict__ cells,
                                                         const float* __restrict__ sdf, int64_t stride, int64_t m,
                                                         const float* __restrict__ s_dev, float s_fixed) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= m) return;
    const int64_t c = cells[i];
    if (c < 0 || c >= count) return;
    const float s = s_dev ? s_dev[0] : s_fixed;
    const float phi = logistic_density(sdf[i * stride], s);
    if (!(phi > 0.0f) || phi > 3.0e38f) return;                 // NaN, zero, overflow: nothing to raise
    atomicMax(reinterpret_cast<unsigned int*>(density) + c, __float_as_uint(phi));
}

// One bit per cell: set where the density exceeds the threshold.  A wavefront covers 64
// consecutive cells, i.e. two words.
__global__ __launch_bounds__(kThreads) void bits_kernel(const float* __restrict__ density, int64_t count,
                                                        float threshold, uint32_t* __restrict__ bitfield) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool on = i < count && density[i] > threshold;
    const uint64_t mask = __ballot(on);
    const int lane = threadIdx.x & 63;
    if (i < count && (lane & 31) == 0) bitfield[i >> 5] = (uint32_t)(mask >> lane);
}

// The numbers of the cells whose bit is set, ascending.  A thread takes a word of 32 cells, a workgroup kThreads of them:
// first every workgroup's count, then each adds up the counts in front of it (2048 at most) and writes its part of the list.
// counts[0] = their total, counts[1 + b] = those of workgroup b.  Bound by launch latency: the bitfield is 2 MB at most.
// (Unpacking the bits to a byte a cell and compacting those took five passes over 2 to 16 bytes a cell.)
__global__ __launch_bounds__(kThreads) void count_cells_kernel(const uint32_t* __restrict__ bitfield, int words, int32_t* __restrict__ counts) {
    __shared__ int part[kThreads / 64];
    const int w = blockIdx.x * kThreads + threadIdx.x;
    int v = w < words ? __popc(bitfield[w]) : 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) v += __shfl_xor(v, step);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int k = 0; k < kThreads / 64; ++k) sum += part[k];
        counts[1 + blockIdx.x] = sum;
    }
}

__global__ __launch_bounds__(kThreads) void list_cells_kernel(const uint32_t* __restrict__ bitfield, int words, int32_t* __restrict__ counts,
                                                              int32_t* __restrict__ cells) {
    __shared__ int before[kThreads / 64], own[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int w = blockIdx.x * kThreads + threadIdx.x;
    uint32_t bits = w < words ? bitfield[w] : 0u;
    int front = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kThreads) front += counts[1 + b];
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) front += __shfl_xor(front, step);
    const int count = __popc(bits);
    int upto = count;
#pragma unroll
    for (int step = 1; step < 64; step <<= 1) {
        const int up = __shfl_up(upto, step);
        if (lane >= step) upto += up;
    }
    if (lane == 63) { before[wave] = front; own[wave] = upto; }
    __syncthreads();
    int at = upto - count;
    for (int k = 0; k < kThreads / 64; ++k) at += before[k] + (k < wave ? own[k] : 0);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kThreads - 1) counts[0] = at + count;
    // two words at a time, a lane a bit: stores of consecutive lanes side by side (a lane a word was 11 us at 128^3 cells)
    const int half = lane >> 5, bit = lane & 31;
#pragma unroll 4
    for (int k = 0; k < 64; k += 2) {
        const uint32_t word = (uint32_t)__shfl((int)bits, k + half);
        const int first = __shfl(at, k + half);
        if ((word >> bit) & 1u) cells[first + __popc(word & ((1u << bit) - 1u))] = 32 * (w - lane + k + half) + bit;
    }
}

// ---- candidates in order of where they lie -----------------------------------------------------
//
// Drawn candidates come in random order: the gathers of the encoding then find nothing of a neighbour's in a cache, on
// the coarse levels either, and every atomic maximum is a request of its own.  Three kernels put them in order: counts
// and places by kBuckets blocks of consecutive Morton numbers (a block is a cube of cells), then the order inside every
// kSortItems of them.  A workgroup lays its candidates out in LDS and writes them with consecutive threads, so runs of one
// bucket leave together (a random store a candidate would touch a line each): 512 buckets are eight candidates a run.
// 2^20 candidates of a 128^3 grid: 7 + 15 + 12 us, for which the encoding takes 259 instead of 324 (the levels finer than the
// grid are left: their cells are nobody else's, and four cache lines a point and level are what the L2s can deliver) and the
// refresh of the cells 8 instead of 52.
constexpr int kBuckets = 512;
constexpr int kSortThreads = 1024;
constexpr int kSortItems = 4 * kSortThreads;
constexpr int kSortEach = kSortItems / kSortThreads;

__device__ __forceinline__ uint32_t bucket_of(int log2_res, int32_t cell) {      // log2_res >= 3
    return ((uint32_t)cell & ((1u << (3 * log2_res)) - 1u)) >> (3 * log2_res - 9);
}

// Exclusive prefix sums of a value a thread, by the whole workgroup.
__device__ __forceinline__ int bucket_scan(int v, int* wave_total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int upto = v;
#pragma unroll
    for (int step = 1; step < 64; step <<= 1) {
        const int up = __shfl_up(upto, step);
        if (lane >= step) upto += up;
    }
    if (lane == 63) wave_total[wave] = upto;
    __syncthreads();
    for (int k = 0; k < wave; ++k) upto += wave_total[k];
    return upto - v;
}

// counts[b] += the candidates of bucket b
__global__ __launch_bounds__(kSortThreads) void count_buckets_kernel(int log2_res, const int32_t* __restrict__ cells, int64_t m,
                                                                     int32_t* __restrict__ counts) {
    __shared__ int hist[kBuckets];
    if (threadIdx.x < kBuckets) hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kSortItems + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        const int64_t i = first + k * kSortThreads;
        if (i < m) atomicAdd(&hist[bucket_of(log2_res, cells[i])], 1);
    }
    __syncthreads();
    if (threadIdx.x < kBuckets && hist[threadIdx.x] > 0) atomicAdd(counts + threadIdx.x, hist[threadIdx.x]);
}

struct SortItems {
    int cell[kSortItems];
    float jitter[3][kSortItems];
};

// counts[0 .. kBuckets) as counted, counts[kBuckets ..) cursors that start at zero.
__global__ __launch_bounds__(kSortThreads) void place_cells_kernel(int log2_res, const int32_t* __restrict__ cells, const float* __restrict__ jitter,
                                                                   int64_t m, int32_t* __restrict__ counts, int32_t* __restrict__ cells_out,
                                                                   float* __restrict__ jitter_out) {
    __shared__ int hist[kBuckets];               // candidates of this workgroup, then the place of its first one minus its place in LDS
    __shared__ int front[kBuckets];              // places in LDS
    __shared__ int totals[2][kSortThreads / 64];
    __shared__ SortItems items;
    const int t = threadIdx.x;
    if (t < kBuckets) hist[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortItems;
    const int here = (int)min((int64_t)kSortItems, m - base);
    int cell[kSortEach], rank[kSortEach];
    float j[kSortEach][3];
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        const int i = k * kSortThreads + t;
        if (i >= here) continue;
        cell[k] = cells[base + i];
#pragma unroll
        for (int a = 0; a < 3; ++a) j[k][a] = fminf(jitter[3 * (base + i) + a], 0x1.fffffep-1f);
        rank[k] = atomicAdd(&hist[bucket_of(log2_res, cell[k])], 1);
    }
    __syncthreads();
    const int start = bucket_scan(t < kBuckets ? counts[t] : 0, totals[0]);
    const int own = t < kBuckets ? hist[t] : 0;
    const int place = bucket_scan(own, totals[1]);
    if (t < kBuckets) {
        front[t] = place;
        hist[t] = start + (own > 0 ? atomicAdd(counts + kBuckets + t, own) : 0) - place;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        if (k * kSortThreads + t >= here) continue;
        const int at = front[bucket_of(log2_res, cell[k])] + rank[k];
        items.cell[at] = cell[k];
#pragma unroll
        for (int a = 0; a < 3; ++a) items.jitter[a][at] = j[k][a];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        const int i = k * kSortThreads + t;
        if (i >= here) continue;
        const int c = items.cell[i];
        const int64_t dst = (int64_t)hist[bucket_of(log2_res, c)] + i;
        if (dst < 0 || dst >= m) continue;                     // cells changed between the two kernels: stay inside
        cells_out[dst] = c;
#pragma unroll
        for (int a = 0; a < 3; ++a) jitter_out[3 * dst + a] = items.jitter[a][i];
    }
}

// The candidates of a workgroup, consecutive ones of the list, in order of kSortThreads equal pieces of the numbers they
// span (about eight cells a piece at 2^20 candidates of a 128^3 grid), in place, and their points.  Neighbouring lanes of
// the encoding then share cells and cache lines on levels up to the grid's resolution, also hashed ones.
__global__ __launch_bounds__(kSortThreads) void order_cells_kernel(int log2_res, int64_t m, int32_t* __restrict__ cells, float* __restrict__ jitter,
                                                                   float* __restrict__ pos) {
    __shared__ int hist[kSortThreads];
    __shared__ int totals[kSortThreads / 64];
    __shared__ uint32_t low, high;
    __shared__ SortItems items;
    const int t = threadIdx.x;
    const uint32_t mask = (1u << (3 * log2_res)) - 1u;
    hist[t] = 0;
    if (t == 0) { low = mask; high = 0u; }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortItems;
    const int here = (int)min((int64_t)kSortItems, m - base);
    int cell[kSortEach], rank[kSortEach];
    float j[kSortEach][3];
    uint32_t least = mask, most = 0u;
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        const int i = k * kSortThreads + t;
        if (i >= here) continue;
        cell[k] = cells[base + i];
#pragma unroll
        for (int a = 0; a < 3; ++a) j[k][a] = jitter[3 * (base + i) + a];
        const uint32_t code = (uint32_t)cell[k] & mask;
        least = min(least, code);
        most = max(most, code);
    }
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        least = min(least, (uint32_t)__shfl_xor((int)least, step));
        most = max(most, (uint32_t)__shfl_xor((int)most, step));
    }
    if ((t & 63) == 0) { atomicMin(&low, least); atomicMax(&high, most); }
    __syncthreads();
    // pieces are aligned, so none holds cells of two buckets: at most kSortThreads + 1 of them by the first guess
    int shift = max(0, 22 - __clz((int)((high - low) | 1u)));
    if ((high >> shift) - (low >> shift) >= kSortThreads) ++shift;
    const uint32_t first = low >> shift;
#pragma unroll
    for (int k = 0; k < kSortEach; ++k)
        if (k * kSortThreads + t < here) rank[k] = atomicAdd(&hist[(((uint32_t)cell[k] & mask) >> shift) - first], 1);
    __syncthreads();
    const int place = bucket_scan(hist[t], totals);
    hist[t] = place;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        if (k * kSortThreads + t >= here) continue;
        const int at = hist[(((uint32_t)cell[k] & mask) >> shift) - first] + rank[k];
        items.cell[at] = cell[k];
#pragma unroll
        for (int a = 0; a < 3; ++a) items.jitter[a][at] = j[k][a];
    }
    __syncthreads();
    const float inv = 1.0f / (float)(1 << log2_res);           // a power of two: exact
#pragma unroll
    for (int k = 0; k < kSortEach; ++k) {
        const int i = k * kSortThreads + t;
        if (i >= here) continue;
        const int c = items.cell[i];
        const uint32_t code = (uint32_t)c & mask;
        cells[base + i] = c;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float ja = items.jitter[a][i];
            jitter[3 * (base + i) + a] = ja;
            pos[3 * (base + i) + a] = ((float)gather3(code >> a) + ja) * inv;
        }
    }
}

// Decay, raise and threshold in one pass over the cells, for candidates in order of their buckets: a workgroup owns
// `own_cells` consecutive cells (a bucket, or a part of one: it then reads the whole bucket), takes the maxima of its
// candidates in LDS and writes each density and bit once.  Atomic maxima in memory were 42 us at 2^20 candidates (a
// request each, whatever their order), decay and bits another pass over the cells each.
// Where the occupied cells lie in few buckets, half of the candidates are theirs: from `share` on a bucket's candidates are left to
// crowded_cells_kernel, which spreads them over the chip.
constexpr int kOwnCells = 4096;

__global__ __launch_bounds__(kSortThreads) void update_cells_kernel(int log2_res, float* __restrict__ density, const int32_t* __restrict__ cells,
                                                                    const float* __restrict__ sdf, int64_t m, const int32_t* __restrict__ counts,
                                                                    const float* __restrict__ s_dev, float s_fixed, float decay, float threshold,
                                                                    uint32_t* __restrict__ bitfield, int own_cells, int64_t share) {
    __shared__ uint32_t top[kOwnCells];
    __shared__ int totals[kSortThreads / 64];
    __shared__ int span[2];
    const int t = threadIdx.x;
    for (int c = t; c < own_cells; c += kSortThreads) top[c] = 0u;
    const uint32_t first = blockIdx.x * (uint32_t)own_cells;
    const int bucket = (int)bucket_of(log2_res, (int32_t)first);
    const int count = t < kBuckets ? counts[t] : 0;
    const int start = bucket_scan(count, totals);
    if (t == bucket) { span[0] = start; span[1] = start + count; }
    __syncthreads();
    const float s = s_dev ? s_dev[0] : s_fixed;
    const int64_t end = min(min((int64_t)span[1], span[0] + share), m);
    for (int64_t i = max(span[0], 0) + t; i < end; i += kSortThreads) {
        const uint32_t c = (uint32_t)cells[i] - first;
        if (c >= (uint32_t)own_cells) continue;                // another part of the bucket, or outside the grid
        const float phi = logistic_density(sdf[i], s);
        if (!(phi > 0.0f) || phi > 3.0e38f) continue;           // NaN, zero, overflow: nothing to raise
        atomicMax(&top[c], __float_as_uint(phi));
    }
    __syncthreads();
    for (int c = t; c < own_cells; c += kSortThreads) {         // own_cells is a multiple of 64: whole wavefronts
        const float old = density[first + c] * decay;
        // the bit patterns of values that are never negative order like unsigned integers
        const float v = __uint_as_float(max(__float_as_uint(old), top[c]));
        density[first + c] = v;
        const uint64_t mask = __ballot(v > threshold);
        const int lane = t & 63;
        if ((lane & 31) == 0) bitfield[(first + c) >> 5] = (uint32_t)(mask >> lane);
    }
}

// What update_cells_kernel left of crowded buckets, after it: a workgroup takes the ones among kSortItems consecutive
// candidates, which are one bucket's (share >= kSortItems), merges those of one cell in LDS and raises density and bit where
// they are larger than what is there.  Exact: neither ever falls here, so the order does not matter.
__global__ __launch_bounds__(kSortThreads) void crowded_cells_kernel(int log2_res, float* __restrict__ density, const int32_t* __restrict__ cells,
                                                                     const float* __restrict__ sdf, int64_t m, const int32_t* __restrict__ counts,
                                                                     const float* __restrict__ s_dev, float s_fixed, float threshold,
                                                                     uint32_t* __restrict__ bitfield, int64_t share) {
    constexpr int kSlots = 4096;
    __shared__ int totals[kSortThreads / 64];
    __shared__ int span[2];
    __shared__ int owner[kSlots];
    __shared__ uint32_t top[kSlots];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kSortItems;
    if (t == 0) { span[0] = 0; span[1] = 0; }
    const int count = t < kBuckets ? counts[t] : 0;
    const int start = bucket_scan(count, totals);               // a barrier inside
    const int64_t low = max((int64_t)start + share, base), high = min(min((int64_t)start + count, m), base + kSortItems);
    if (t < kBuckets && low < high) { span[0] = (int)(low - base); span[1] = (int)(high - base); }
    __syncthreads();
    const int first = max(span[0], 0), last = span[1];
    if (first >= last) return;                                  // the same for the workgroup
    for (int k = t; k < kSlots; k += kSortThreads) { owner[k] = -1; top[k] = 0u; }
    __syncthreads();
    const int64_t total = (int64_t)1 << (3 * log2_res);
    const float s = s_dev ? s_dev[0] : s_fixed;
    auto raise = [&](int c, uint32_t bits) {
        if (bits > __float_as_uint(density[c])) atomicMax(reinterpret_cast<unsigned int*>(density) + c, bits);
        const uint32_t bit = 1u << (c & 31);
        if (__uint_as_float(bits) > threshold && !(bitfield[c >> 5] & bit)) atomicOr(bitfield + (c >> 5), bit);
    };
    for (int k = first + t; k < last; k += kSortThreads) {
        const int c = cells[base + k];
        if (c < 0 || c >= total) continue;
        const float phi = logistic_density(sdf[base + k], s);
        if (!(phi > 0.0f) || phi > 3.0e38f) continue;           // NaN, zero, overflow: nothing to raise
        const int slot = c & (kSlots - 1);
        const int other = atomicCAS(&owner[slot], -1, c);
        if (other == -1 || other == c) atomicMax(&top[slot], __float_as_uint(phi));
        else raise(c, __float_as_uint(phi));                    // grids beyond 128^3: another cell has the slot
    }
    __syncthreads();
    for (int k = t; k < kSlots; k += kSortThreads)
        if (owner[k] >= 0) raise(owner[k], top[k]);
}

// ---- marching ---------------------------------------------------------------------------------

struct Chord {
    float t0, far;     // first lattice parameter, exit parameter
    bool hit;
};

// Slab test against [0,1]^3; every lane of the wavefront computes the same values.
__device__ __forceinline__ Chord clip_ray(const float o[3], const float d[3], float jitter, float dt) {
    float near = 0.0f, far = INFINITY;
    bool hit = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (d[a] == 0.0f) {
            hit = hit && (o[a] >= 0.0f && o[a] < 1.0f);
        } else {
            const float inv = 1.0f / d[a];
            const float t1 = (0.0f - o[a]) * inv;
            const float t2 = (1.0f - o[a]) * inv;
            near = fmaxf(near, fminf(t1, t2));
            far = fminf(far, fmaxf(t1, t2));
        }
    }
    Chord c;
    c.hit = hit && near < far;
    c.far = far;
    c.t0 = near + jitter * dt;
    return c;
}

// One wavefront per ray; lane j of pass b looks at lattice point k = 64 b + j:
//   t_k = t0 + k dt, point = o + t_k d, cell = clamp(floor(point G)), kept if t_k < far and the
//   cell's bit is set.
// WRITE = false: ray_offsets[r+1] = number of kept points.  WRITE = true: ray_offsets holds the
// scanned, capacity-clamped offsets and the kept points are written in order.
template <bool WRITE>
__global__ __launch_bounds__(kThreads) void march_kernel(int log2_res, const uint32_t* __restrict__ bitfield,
                                                         const float* __restrict__ origins,
                                                         const float* __restrict__ dirs,
                                                         const float* __restrict__ jitter, int64_t rays, float dt,
                                                         int max_steps, int32_t* __restrict__ ray_offsets,
                                                         float* __restrict__ pos, int32_t* __restrict__ sample_ray,
                                                         float* __restrict__ t_out) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (r >= rays) return;
    const float o[3] = {origins[3 * r], origins[3 * r + 1], origins[3 * r + 2]};
    const float d[3] = {dirs[3 * r], dirs[3 * r + 1], dirs[3 * r + 2]};
    const Chord ch = clip_ray(o, d, jitter[r], dt);
    const int G = 1 << log2_res;
    const float Gf = (float)G;
    int64_t begin = 0, end = 0;
    if (WRITE) {
        begin = ray_offsets[r];
        end = ray_offsets[r + 1];
    }
    int64_t kept = 0;
    if (ch.hit && (!WRITE || end > begin)) {
        for (int base = 0; base < max_steps; base += 64) {
            if (!(ch.t0 + (float)base * dt < ch.far)) break;            // t_k does not decrease with k
            const int k = base + lane;
            const float t = ch.t0 + (float)k * dt;
            float p[3];
            uint32_t code = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                p[a] = o[a] + t * d[a];
                int c = (int)floorf(p[a] * Gf);
                c = c < 0 ? 0 : (c > G - 1 ? G - 1 : c);
                code |= spread3((uint32_t)c) << a;
            }
            bool on = k < max_steps && t < ch.far;
            if (on) on = (bitfield[code >> 5] >> (code & 31u)) & 1u;
            const uint64_t mask = __ballot(on);
            if (WRITE) {
                const int64_t dst = begin + kept + __popcll(mask & ((1ull << lane) - 1ull));
                if (on && dst < end) {
                    pos[3 * dst + 0] = p[0];
                    pos[3 * dst + 1] = p[1];
                    pos[3 * dst + 2] = p[2];
                    sample_ray[dst] = (int32_t)r;
                    if (t_out) t_out[dst] = t;
                }
            }
            kept += __popcll(mask);
            if (WRITE && begin + kept >= end) break;
        }
    }
    if (!WRITE && lane == 0) ray_offsets[r + 1] = (int32_t)kept;
}

// In place: ray_offsets[0] = 0, ray_offsets[r+1] = min(count_0 + ... + count_r, capacity).
// One workgroup walks the array in tiles of kScanThreads.
__global__ __launch_bounds__(kScanThreads) void scan_offsets_kernel(int32_t* __restrict__ ray_offsets, int64_t rays,
                                                                    int64_t capacity) {
    __shared__ int64_t wave_total[kScanThreads / 64];
    __shared__ int64_t carry_s;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) {
        ray_offsets[0] = 0;
        carry_s = 0;
    }
    __syncthreads();
    for (int64_t tile = 0; tile < rays; tile += kScanThreads) {
        const int64_t i = tile + threadIdx.x;
        int64_t v = i < rays ? ray_offsets[i + 1] : 0;
#pragma unroll
        for (int step = 1; step < 64; step <<= 1) {
            const int64_t up = __shfl_up(v, step);
            if (lane >= step) v += up;
        }
        if (lane == 63) wave_total[wave] = v;
        __syncthreads();
        int64_t before = carry_s;
        for (int w = 0; w < wave; ++w) before += wave_total[w];
        v += before;
        if (i < rays) ray_offsets[i + 1] = (int32_t)(v < capacity ? v : capacity);
        __syncthreads();
        if (threadIdx.x == kScanThreads - 1) carry_s = v;
        __syncthreads();
    }
}

int check_grid(int log2_res) {
    if (log2_res < 2 || log2_res > 8) return fail(NEUS2_ERR_SHAPE, "log2_res %d outside 2..8", log2_res);
    return NEUS2_OK;
}

int check_m(int64_t m, const char* name) {
    if (m < 0 || m > ((int64_t)1 << 30)) return fail(NEUS2_ERR_SHAPE, "%s = %lld outside 0..2^30", name, (long long)m);
    return NEUS2_OK;
}

}  // namespace
}  // namespace neus2

using namespace neus2;

extern "C" int neus2_occupancy_points(int log2_res, const int32_t* cells, const float* jitter, int64_t m,
                                      float* pos, void* stream) {
    NEUS2_TRY(check_grid(log2_res));
    NEUS2_TRY(check_m(m, "m"));
    NEUS2_TRY(check_ptr(cells, "cells"));
    NEUS2_TRY(check_ptr(jitter, "jitter"));
    NEUS2_TRY(check_ptr(pos, "pos"));
    if (m == 0) return NEUS2_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    cell_points_kernel<<<(unsigned)((m + kThreads - 1) / kThreads), kThreads, 0, st>>>(log2_res, cells, jitter, m, pos);
    return check_launch("cell_points_kernel");
}

extern "C" int neus2_occupancy_list(int log2_res, const uint32_t* bitfield, int32_t* counts, int32_t* cells, void* stream) {
    NEUS2_TRY(check_grid(log2_res));
    NEUS2_TRY(check_ptr(bitfield, "bitfield"));
    NEUS2_TRY(check_ptr(counts, "counts"));
    NEUS2_TRY(check_ptr(cells, "cells"));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int words = 1 << (3 * log2_res - 5);
    const unsigned blocks = (unsigned)((words + kThreads - 1) / kThreads);
    count_cells_kernel<<<blocks, kThreads, 0, st>>>(bitfield, words, counts);
    NEUS2_TRY(check_launch("count_cells_kernel"));
    list_cells_kernel<<<blocks, kThreads, 0, st>>>(bitfield, words, counts, cells);
    return check_launch("list_cells_kernel");
}

static int check_sorted(int log2_res, int64_t m) {
    NEUS2_TRY(check_grid(log2_res));
    NEUS2_TRY(check_m(m, "m"));
    if (log2_res < 5) return fail(NEUS2_ERR_SHAPE, "log2_res %d: candidates are put in order from 5 on", log2_res);
    return NEUS2_OK;
}

extern "C" int neus2_occupancy_points_ordered(int log2_res, const int32_t* cells, const float* jitter, int64_t m, int32_t* counts,
                                              int32_t* cells_out, float* jitter_out, float* pos, void* stream) {
    NEUS2_TRY(check_sorted(log2_res, m));
    NEUS2_TRY(check_ptr(cells, "cells"));
    NEUS2_TRY(check_ptr(jitter, "jitter"));
    NEUS2_TRY(check_ptr(counts, "counts"));
    NEUS2_TRY(check_ptr(cells_out, "cells_out"));
    NEUS2_TRY(check_ptr(jitter_out, "jitter_out"));
    NEUS2_TRY(check_ptr(pos, "pos"));
    hipStream_t st = static_cast<hipStream_t>(stream);
    NEUS2_TRY(launch_zero(reinterpret_cast<float*>(counts), 2 * kBuckets, st));
    if (m == 0) return NEUS2_OK;
    const unsigned blocks = (unsigned)((m + kSortItems - 1) / kSortItems);
    count_buckets_kernel<<<blocks, kSortThreads, 0, st>>>(log2_res, cells, m, counts);
    NEUS2_TRY(check_launch("count_buckets_kernel"));
    place_cells_kernel<<<blocks, kSortThreads, 0, st>>>(log2_res, cells, jitter, m, counts, cells_out, jitter_out);
    NEUS2_TRY(check_launch("place_cells_kernel"));
    order_cells_kernel<<<blocks, kSortThreads, 0, st>>>(log2_res, m, cells_out, jitter_out, pos);
    return check_launch("order_cells_kernel");
}

static int check_refresh(const float* density, const uint32_t* bitfield, const float* s_dev, float s, float decay, float threshold) {
    NEUS2_TRY(check_ptr(density, "density"));
    NEUS2_TRY(check_ptr(bitfield, "bitfield"));
    NEUS2_TRY(check_ptr(s_dev, "s_dev", false));
    if (!(decay >= 0.0f && decay <= 1.0f)) return fail(NEUS2_ERR_CONFIG, "decay %g outside [0,1]", (double)decay);
    if (!(threshold >= 0.0f)) return fail(NEUS2_ERR_CONFIG, "threshold %g is negative or NaN", (double)threshold);
    if (!s_dev && !(s > 0.0f)) return fail(NEUS2_ERR_CONFIG, "s %g is not positive", (double)s);
    return NEUS2_OK;
}

extern "C" int neus2_occupancy_update_ordered(int log2_res, float* density, const int32_t* cells, const float* sdf, int64_t m,
                                              const int32_t* counts, const float* s_dev, float s, float decay, float threshold,
                                              uint32_t* bitfield, void* stream) {
    NEUS2_TRY(check_sorted(log2_res, m));
    NEUS2_TRY(check_refresh(density, bitfield, s_dev, s, decay, threshold));
    NEUS2_TRY(check_ptr(cells, "cells"));
    NEUS2_TRY(check_ptr(sdf, "sdf"));
    NEUS2_TRY(check_ptr(counts, "counts"));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int total = 1 << (3 * log2_res);
    const int own = std::min(kOwnCells, total / kBuckets);
    // two workgroups' worth, and four times the mean: evenly spread candidates and those of a shell stay below it
    const int64_t share = std::max((int64_t)2 * kSortItems, 4 * (m / kBuckets));
    update_cells_kernel<<<total / own, kSortThreads, 0, st>>>(log2_res, density, cells, sdf, m, counts, s_dev, s, decay, threshold,
                                                              bitfield, own, share);
    NEUS2_TRY(check_launch("update_cells_kernel"));
    if (m <= share) return NEUS2_OK;
    crowded_cells_kernel<<<(unsigned)((m + kSortItems - 1) / kSortItems), kSortThreads, 0, st>>>(
        log2_res, density, cells, sdf, m, counts, s_dev, s, threshold, bitfield, share);
    return check_launch("crowded_cells_kernel");
}

extern "C" int neus2_occupancy_update(int log2_res, float* density, const int32_t* cells, const float* sdf,
                                      int64_t sdf_stride, int64_t m, const float* s_dev, float s, float decay,
                                      float threshold, uint32_t* bitfield, void* stream) {
    NEUS2_TRY(check_grid(log2_res));
    NEUS2_TRY(check_m(m, "m"));
    if (m > 0) {
        NEUS2_TRY(check_ptr(cells, "cells"));
        NEUS2_TRY(check_ptr(sdf, "sdf"));
        if (sdf_stride < 1) return fail(NEUS2_ERR_SHAPE, "sdf_stride %lld < 1", (long long)sdf_stride);
    }
    NEUS2_TRY(check_refresh(density, bitfield, s_dev, s, decay, threshold));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t count = (int64_t)1 << (3 * log2_res);
    decay_kernel<<<(unsigned)((count / 4 + kThreads - 1) / kThreads), kThreads, 0, st>>>(
        density, count, decay);
    NEUS2_TRY(check_launch("decay_kernel"));
    if (m > 0) {
        raise_kernel<<<(unsigned)((m + kThreads - 1) / kThreads), kThreads, 0, st>>>(density, count, cells, sdf,
                                                                                      sdf_stride, m, s_dev, s);
        NEUS2_TRY(check_launch("raise_kernel"));
    }
    bits_kernel<<<(unsigned)((count + kThreads - 1) / kThreads), kThreads, 0, st>>>(density, count, threshold, bitfield);
    return check_launch("bits_kernel");
}

extern "C" int neus2_march_rays(int log2_res, const uint32_t* bitfield, const float* origins, const float* dirs,
                                const float* jitter, int64_t rays, float dt, int32_t max_steps, int64_t capacity,
                                int32_t* ray_offsets, float* pos, int32_t* sample_ray, float* t, void* stream) {
    NEUS2_TRY(check_grid(log2_res));
    if (rays < 0 || rays > ((int64_t)1 << 24)) return fail(NEUS2_ERR_SHAPE, "rays = %lld outside 0..2^24", (long long)rays);
    if (capacity < 0 || capacity > 0x7fffffffLL)
        return fail(NEUS2_ERR_SHAPE, "capacity = %lld outside 0..2^31-1", (long long)capacity);
    if (max_steps < 1 || max_steps > (1 << 20)) return fail(NEUS2_ERR_SHAPE, "max_steps = %d outside 1..2^20", max_steps);
    if (!(dt > 0.0f) || !(dt < 1e30f)) return fail(NEUS2_ERR_CONFIG, "dt %g is not a positive finite step", (double)dt);
    NEUS2_TRY(check_ptr(bitfield, "bitfield"));
    NEUS2_TRY(check_ptr(ray_offsets, "ray_offsets"));
    NEUS2_TRY(check_ptr(t, "t", false));
    if (rays > 0) {
        NEUS2_TRY(check_ptr(origins, "origins"));
        NEUS2_TRY(check_ptr(dirs, "dirs"));
        NEUS2_TRY(check_ptr(jitter, "jitter"));
    }
    if (capacity > 0) {
        NEUS2_TRY(check_ptr(pos, "pos"));
        NEUS2_TRY(check_ptr(sample_ray, "sample_ray"));
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const unsigned blocks = (unsigned)((rays + kThreads / 64 - 1) / (kThreads / 64));
    if (rays > 0) {
        march_kernel<false><<<blocks, kThreads, 0, st>>>(log2_res, bitfield, origins, dirs, jitter, rays, dt, max_steps,
                                                         ray_offsets, nullptr, nullptr, nullptr);
        NEUS2_TRY(check_launch("march_kernel<count>"));
    }
    scan_offsets_kernel<<<1, kScanThreads, 0, st>>>(ray_offsets, rays, capacity);
    NEUS2_TRY(check_launch("scan_offsets_kernel"));
    if (rays > 0 && capacity > 0) {
        march_kernel<true><<<blocks, kThreads, 0, st>>>(log2_res, bitfield, origins, dirs, jitter, rays, dt, max_steps,
                                                        ray_offsets, pos, sample_ray, t);
        NEUS2_TRY(check_launch("march_kernel<write>"));
    }
    return NEUS2_OK;
}
