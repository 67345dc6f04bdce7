// Device-side pieces of the backward pass that both kernel families use (internal): the list of query
// regions that attend to a key region, and the reduction of per-workgroup partial sums.
#pragma once

#include "bra_mfma_dev.h"

namespace bra {
namespace bwd {

using mfma::kWave;

// ---------------------------------------------------------------------------
// The entries of rows `irb` (D.R x D.k of one image) with value j among entries [e0, e0 + kListChunk), in
// ascending order, to `list`; returns how many.  Called by all 256 threads; ends with a barrier.  The order is
// that of the entry numbers, so sums over the list come out the same every time.
constexpr int kListChunk = 1024;

__device__ __forceinline__ int collect_entries(const int32_t *__restrict__ irb, int entries, int e0, int j, int R,
                                               int *list, int *counts)
{
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    unsigned long long votes[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = e0 + 256 * u + (int)threadIdx.x;
        votes[u] = __ballot(e < entries && region_index(irb[e < entries ? e : 0], R) == j);
        if (lane == 0) counts[4 * u + wave] = __popcll(votes[u]);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == wave && (votes[u] >> lane & 1))
                list[total + __popcll(votes[u] & ((1ull << lane) - 1))] = e0 + 256 * u + (int)threadIdx.x;
            total += counts[4 * u + w];
        }
    __syncthreads();
    return total;
}

// ---------------------------------------------------------------------------
// out[e] = sum_p part[p][e], p in a fixed order, for up to three arrays in one launch.  A thread sums 4 elements (16
// bytes) of one of `slices` slices of p (a power of two up to 16, about a quarter of the number of partial arrays or less), the
// slices are summed through LDS.  Counts are multiples of 4 and arrays 16-byte aligned, else VEC = false: single elements.
// 256 consecutive bytes of an array at a time, eight arrays' on their way (64 slices of 64 bytes, four on their way: 64 x 56 x 56 x 64, 224
// arrays of 64 KB, whole gradient 210.3 -> 208.3 us; 8 images 69.2 -> 66.4; 2 x 56 x 56 x 64 float32 58.9 -> 57.2).
struct ReduceJob {
    const float *part;
    float *out;
    int nparts, count, slices, blocks;
    int vec;
};

inline ReduceJob reduce_job(const float *part, float *out, int nparts, int count)
{
    int slices = 1;
    while (slices < 16 && 4 * slices <= nparts) slices *= 2;
    const int vec = count % 4 == 0 && (uintptr_t)part % 16 == 0 && (uintptr_t)out % 16 == 0;
    const int elems = 256 / slices * (vec ? 4 : 1);
    return ReduceJob{part, out, nparts, count, slices, (count + elems - 1) / elems, vec};
}

template <typename V>
__device__ __forceinline__ void reduce_block(const ReduceJob &job, int bi, V *red)
{
    const int per = 256 / job.slices, x = threadIdx.x % per, y = threadIdx.x / per, n = job.count / (int)(sizeof(V) / 4);
    const int e = bi * per + x;
    const V *part = (const V *)job.part;
    V sum = V{};
    if (e < n) {
#pragma unroll 8
        for (int p = y; p < job.nparts; p += job.slices) sum += part[(size_t)p * n + e];
    }
    red[y * per + x] = sum;
    __syncthreads();
    if (y == 0 && e < n) {
        V total = V{};
        for (int u = 0; u < job.slices; ++u) total += red[u * per + x];
        ((V *)job.out)[e] = total;
    }
}

[[maybe_unused]] static __global__ __launch_bounds__(256) void k_reduce_parts(ReduceJob j0, ReduceJob j1, ReduceJob j2)
{
    __shared__ mfma::f32x4 red[256];
    int bi = blockIdx.x;
    ReduceJob job = j0;
    if (bi >= j0.blocks) {
        bi -= j0.blocks;
        job = j1;
        if (bi >= j1.blocks) {
            bi -= j1.blocks;
            job = j2;
        }
    }
    if (job.vec) reduce_block<mfma::f32x4>(job, bi, red);
    else reduce_block<float>(job, bi, (float *)red);
}

}  // namespace bwd
}  // namespace bra
