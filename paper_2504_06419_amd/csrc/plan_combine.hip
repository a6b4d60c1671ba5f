// plan_combine.hip -- work partition (plan) and split-segment merge (combine).
//
// The plan reads the per-sequence lengths on the device, clamps them to what
// the cache descriptors can address, cuts every sequence into key tiles (plus
// the phantom positions of each segment) and assigns each worker an equal
// share of all positions (see spire_internal.h).  It runs as one workgroup
// ahead of the LDS-staged and generic kernels; the register-staged kernel
// computes the same partition itself (plan_in_kernel, mfma_common.h).
// Everything it produces stays in the caller's workspace.
//
// The combine merges the partial results of a segment that several workers
// shared: with partials (o_p, lse_p) in base 2,
//   M = max_p lse_p,  w_p = 2^(lse_p - M),  out = sum_p w_p o_p / sum_p w_p,
//   lse = (M + log2 sum_p w_p) * ln 2,
// the log-sum-exp identity that makes attention over a union of disjoint key
// sets equal to a weighted merge of attention over each set.  A NaN partial
// (a NaN key or a +inf score in that part) makes the merged row NaN.
#include "combine.h"

namespace spire {

constexpr int kPlanThreads = 1024;

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(Problem p, Plan pl) {
    __shared__ int32_t prefix[kPlanMaxB + 1];
    __shared__ int32_t sums[kPlanThreads];
    const int tid = threadIdx.x;
    const int B = p.B;
    const int per = (B + kPlanThreads - 1) / kPlanThreads;
    const int b0 = tid * per;
    const int b1 = b0 + per < B ? b0 + per : B;
    int local = 0;
    for (int b = b0; b < b1; ++b) {
        const int n = effective_keys(p, b);
        pl.nkeys[b] = n;
        const int tiles = (n > 0 ? (n + pl.tile - 1) / pl.tile : 1) + pl.seg_cost;
        prefix[b] = tiles;  // temporarily the position count
        local += tiles;
    }
    sums[tid] = local;
    __syncthreads();
    for (int off = 1; off < kPlanThreads; off <<= 1) {  // inclusive scan
        const int v = tid >= off ? sums[tid - off] : 0;
        __syncthreads();
        sums[tid] += v;
        __syncthreads();
    }
    int run = sums[tid] - local;
    for (int b = b0; b < b1; ++b) {
        const int tiles = prefix[b];
        prefix[b] = run;
        pl.prefix[b] = run;
        run += tiles;
    }
    if (tid == kPlanThreads - 1) {
        prefix[B] = sums[kPlanThreads - 1];
        pl.prefix[B] = sums[kPlanThreads - 1];
    }
    __syncthreads();
    const int64_t T = (int64_t)prefix[B] * pl.units;
    for (int w = tid; w < pl.workers; w += kPlanThreads) {
        const int64_t x = worker_begin(w, T, pl.workers);
        if (x >= worker_begin(w + 1, T, pl.workers)) {  // empty range
            pl.wstart[2 * w] = -1;
            pl.wstart[2 * w + 1] = 0;
            continue;
        }
        int lo = 0, hi = B - 1;  // last b with units * prefix[b] <= x
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if ((int64_t)prefix[mid] * pl.units <= x) lo = mid; else hi = mid - 1;
        }
        const int tiles = prefix[lo + 1] - prefix[lo];
        const int64_t rel = x - (int64_t)prefix[lo] * pl.units;
        const int q = (int)div_floor((double)rel, (double)tiles);
        pl.wstart[2 * w] = lo * pl.units + q;
        pl.wstart[2 * w + 1] = (int)(rel - (int64_t)q * tiles);
    }
}

hipError_t launch_plan(const Problem &p, const Plan &pl, hipStream_t st) {
    if (p.B > kPlanMaxB) return hipErrorInvalidValue;
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, st, p, pl);
    return hipGetLastError();
}

template <bool PER_WORKER, bool GROUPED>
__global__ __launch_bounds__(kCombineThreads) void combine_kernel(Problem p, Plan pl) {
    CombineLds *lds = nullptr;
    if constexpr (GROUPED) {
        __shared__ CombineLds mem;
        lds = &mem;
    }
    combine_block<PER_WORKER, GROUPED>(p, pl, blockIdx.x, blockIdx.y, gridDim.y, lds, [](int, int) {
        if constexpr (GROUPED) __syncthreads();
        return false;
    });
}

hipError_t launch_combine(const Problem &p, const Plan &pl, hipStream_t st) {
    if ((int64_t)p.B * pl.units == 0) return hipSuccess;
    if (pl.workers > kCombineMaxWorkers) return hipErrorInvalidValue;
    const dim3 grid = combine_grid(p, pl), block(kCombineThreads);
    if (combine_per_worker(p, pl))
        hipLaunchKernelGGL((combine_kernel<true, false>), grid, block, 0, st, p, pl);
    else if (combine_grouped(p, pl))
        hipLaunchKernelGGL((combine_kernel<false, true>), grid, block, 0, st, p, pl);
    else
        hipLaunchKernelGGL((combine_kernel<false, false>), grid, block, 0, st, p, pl);
    return hipGetLastError();
}

}  // namespace spire
