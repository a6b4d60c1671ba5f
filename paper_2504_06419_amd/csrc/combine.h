// combine.h -- merge of the partial results of one split segment (device code
// shared by the combine kernel and the fp32 path's combine with value check).
//
// The grid is either one workgroup per (segment, row chunk) -- workgroups of
// segments one worker covered return at once -- or, when segments outnumber
// workers, one per (worker w, row chunk): w merges the segment it starts inside
// of when it is the first worker to start inside that segment's tiles (every
// split segment has exactly one such worker), so no workgroup is spent on
// unsplit segments.
//
// Few partials per segment (GROUPED false): a thread merges 4 outputs on its
// own, no LDS.  Many (GROUPED): a workgroup takes rc rows at a time, D/4 threads
// per row and partial, and G = 256 / (rc D/4) groups of threads share the
// partials of the rows, summed over the groups through LDS in a fixed order.
// What bounds it is latency: a small batch splits every segment over workers /
// segments partials (128 for one sequence of 8 KV heads), which single threads
// would walk one after the other.  There the log-sum-exps and the first four
// outputs of every group are requested together before the weights are formed.
// MI355X: 13 sequences x 8 KV heads (10 partials a segment) 8.5 -> 5.1 us; 4 x 2
// of 512 fp32 keys (38 partials, and as many workers without any position, no
// longer visited) about 43 -> 7 us.  With 2 partials a segment the grouped form
// lost (256 x 8, 20 rows: 17.6 us against 12.7 ungrouped; 512 x 8, 72 rows: 49.6
// against 33.5; those were 13.7 and 36.6 with the slots in an LDS list).
#pragma once
#include <algorithm>

#include "spire_internal.h"

namespace spire {

constexpr int kCombineThreads = 256;
struct CombineLds {
    float w[kCombineMaxWorkers];    // [m][rc] log-sum-exps, then weights
    float4 red[kCombineThreads];
    float M[32], L[32];             // of the rows in flight (rc <= 16)
};

// `skip(b, h)` is asked by every thread of a merging workgroup (GROUPED: after
// its first requests; its answer is the same for all, and it ends with a
// workgroup barrier there); true leaves the segment's rows alone.
template <bool PER_WORKER, bool GROUPED, class Skip>
__device__ __forceinline__ void combine_block(const Problem &p, const Plan &pl, int bx, int by, int ny,
                                              CombineLds *lds, Skip &&skip) {
    int seg = bx, tile0 = 0;
    if (PER_WORKER) {
        seg = pl.wstart[2 * bx];
        if (seg < 0) return;  // empty range
        tile0 = pl.wstart[2 * bx + 1];
    }
    const int b = seg / pl.units, u = seg - (seg / pl.units) * pl.units;
    const int span = pl.prefix[b + 1] - pl.prefix[b];  // tiles + phantom positions
    const int tiles = span - pl.seg_cost;
    if (PER_WORKER && (tile0 == 0 || tile0 >= tiles)) return;  // starts at the first tile or past the last
    const int64_t T = (int64_t)pl.prefix[p.B] * pl.units;
    const int64_t start = (int64_t)pl.prefix[b] * pl.units + (int64_t)u * span;
    // the workers whose ranges hold the segment's tiles (phantoms are not read)
    const int64_t wlo = worker_of(start, T, pl.workers);
    const int64_t whi = worker_of(start + tiles - 1, T, pl.workers);
    if (wlo == whi) return;
    // workers wlo+1 .. whi start inside the tiles; the first non-empty one merges
    if (PER_WORKER && worker_begin(bx, T, pl.workers) != worker_begin(wlo + 1, T, pl.workers)) return;
    const int nrb = pl.units / p.Hkv;  // units per KV head
    const int h = u / nrb;

    // Partial i of the segment.  With fewer positions than workers every
    // position has a worker of its own (others have empty ranges and wrote
    // nothing); otherwise no range is empty.
    const bool sparse = T < pl.workers;
    const int m = sparse ? tiles : (int)(whi - wlo + 1);  // <= workers <= kCombineMaxWorkers
    const bool tail0 = !sparse && worker_begin(wlo, T, pl.workers) < start;  // wlo's last segment, not its first
    auto slot = [&](int i) -> int64_t {
        return sparse ? 2 * worker_of(start + i, T, pl.workers) : 2 * (wlo + i) + (i == 0 && tail0 ? 1 : 0);
    };

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = (u - h * nrb) * pl.rows;
    const int nrows = p.R - r0 < pl.rows ? p.R - r0 : pl.rows;
    const int d4n = p.D >> 2;
    const int rpc = (pl.rows + ny - 1) / ny;  // rows per chunk
    const int rend = by * rpc + rpc < nrows ? by * rpc + rpc : nrows;
    constexpr int U = 4;                      // partials a thread requests together
    auto part = [&](int i, int r, int d4) {
        return *reinterpret_cast<const float4 *>(pl.part_o + (slot(i) * pl.rows + r) * (int64_t)p.D + 4 * d4);
    };
    auto add = [](float4 &acc, float wgt, const float4 &v) {
        acc.x += wgt * v.x; acc.y += wgt * v.y; acc.z += wgt * v.z; acc.w += wgt * v.w;
    };
    // L: the sum of the weights; 0: no visible key; NaN: a NaN partial (a NaN
    // key or a +inf score in that part) makes the row NaN
    auto write = [&](int r, int d4, float4 acc, float M, float L) {
        const float inv = L > 0.f ? 1.f / L : (L == 0.f ? 0.f : L);
        if (!(L > 0.f)) acc = make_float4(L, L, L, L);
        const int64_t off = row_offset(p, b, h, r0 + r) + 4 * d4;
        if (p.out_dtype == SPIRE_BF16) {
            uint16_t *q = reinterpret_cast<uint16_t *>(p.out) + off;
            const uint32_t lo = f32_to_bf16_rne(acc.x * inv) | ((uint32_t)f32_to_bf16_rne(acc.y * inv) << 16);
            const uint32_t hi = f32_to_bf16_rne(acc.z * inv) | ((uint32_t)f32_to_bf16_rne(acc.w * inv) << 16);
            *reinterpret_cast<uint2 *>(q) = make_uint2(lo, hi);
        } else {
            *reinterpret_cast<float4 *>(reinterpret_cast<float *>(p.out) + off) =
                make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
        }
        if (d4 == 0 && p.lse != nullptr)
            p.lse[lse_index(p, b, h, r0 + r)] = L > 0.f ? (M + log2f(L)) * 0.69314718055994531f
                                                         : (L == 0.f ? -INFINITY : L);
    };

    if constexpr (!GROUPED) {
        if (skip(b, h)) return;
        for (int idx = tid; idx < (rend - by * rpc) * d4n; idx += kCombineThreads) {
            const int rr = idx / d4n, d4 = idx - rr * d4n, r = by * rpc + rr;
            float M = -INFINITY, L = 0.f;
            for (int i = 0; i < m; ++i) {
                const float lp = pl.part_lse[slot(i) * pl.rows + r];
                if (lp != lp) L = lp;
                else M = fmaxf(M, lp);
            }
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            if (L == L && M != -INFINITY) {
                for (int i = 0; i < m; ++i) {
                    const float lp = pl.part_lse[slot(i) * pl.rows + r];
                    const float wgt = lp == -INFINITY ? 0.f : exp2f(lp - M);
                    L += wgt;
                    add(acc, wgt, part(i, r, d4));
                }
            }
            write(r, d4, acc, M, L);
        }
        return;
    } else {
        CombineLds &s = *lds;
        int most = kCombineMaxWorkers / m;  // rows whose weights fit
        if (most > kCombineThreads / d4n) most = kCombineThreads / d4n;
        for (int rlo = by * rpc; rlo < rend; rlo += most) {
            const int rc = rend - rlo < most ? rend - rlo : most;
            const int per = rc * d4n;             // threads of a group
            const int G = kCombineThreads / per;
            const int g = tid / per, e = tid - g * per;
            const int rr = e / d4n, d4 = e - rr * d4n;
            const bool on = g < G;
            float4 o[U];
#pragma unroll
            for (int x = 0; x < U; ++x)
                o[x] = on && g + G * x < m ? part(g + G * x, rlo + rr, d4) : make_float4(0.f, 0.f, 0.f, 0.f);
            for (int x = tid; x < rc * m; x += kCombineThreads) {
                const int i = x / rc;
                s.w[x] = pl.part_lse[slot(i) * pl.rows + rlo + (x - i * rc)];
            }
            if (skip(b, h)) return;
            // one wave per row: maximum, weights, their sum.  A NaN partial (a NaN
            // key or a +inf score in that part) makes the row NaN.
            for (int r = wave; r < rc; r += kCombineThreads / 64) {
                float M = -INFINITY;
                bool nan = false;
                for (int i = lane; i < m; i += 64) {
                    const float lp = s.w[i * rc + r];
                    if (lp != lp) nan = true;
                    else M = fmaxf(M, lp);
                }
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
                nan = __any(nan);
                float L = 0.f;
                for (int i = lane; i < m; i += 64) {
                    const float lp = s.w[i * rc + r];
                    const float wgt = lp == -INFINITY ? 0.f : exp2f(lp - M);
                    s.w[i * rc + r] = wgt;
                    L += wgt;
                }
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) L += __shfl_xor(L, d);
                if (lane == 0) {
                    s.M[r] = M;
                    s.L[r] = nan ? __builtin_nanf("") : L;
                }
            }
            __syncthreads();
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            const float L = s.L[on ? rr : 0];
            if (on && L > 0.f) {  // L == 0: no visible key; NaN: a NaN row
#pragma unroll
                for (int x = 0; x < U; ++x)
                    if (g + G * x < m) add(acc, s.w[(g + G * x) * rc + rr], o[x]);
                for (int i = g + G * U; i < m; i += G * U) {
#pragma unroll
                    for (int x = 0; x < U; ++x)
                        if (i + G * x < m) o[x] = part(i + G * x, rlo + rr, d4);
#pragma unroll
                    for (int x = 0; x < U; ++x)
                        if (i + G * x < m) add(acc, s.w[(i + G * x) * rc + rr], o[x]);
                }
            }
            if (G > 1) {
                s.red[tid] = acc;
                __syncthreads();
                for (int x = 1; x < G && g == 0; ++x) add(acc, 1.f, s.red[x * per + e]);
            }
            if (g == 0) write(rlo + rr, d4, acc, s.M[rr], L);
            __syncthreads();  // the next rows reuse the LDS
        }
    }
}

// Grid of the merge: x = workers or segments, y = row chunks.  With more
// segments than workers there is at most one split segment per worker start and
// about two partials each; up to a quarter as many segments, a thread per 4
// outputs walks them.  Below, a segment has about workers / segments partials:
// fewer rows per workgroup, so that up to 8 or 16 groups of threads share them,
// while that keeps the grid within ~4096 workgroups (more measured slower).
inline bool combine_per_worker(const Problem &p, const Plan &pl) { return (int64_t)p.B * pl.units > pl.workers; }
inline bool combine_grouped(const Problem &p, const Plan &pl) { return 4 * (int64_t)p.B * pl.units <= pl.workers; }
inline dim3 combine_grid(const Problem &p, const Plan &pl) {
    const int64_t segs = (int64_t)p.B * pl.units;
    int64_t rpw = kCombineThreads / (p.D / 4);
    if (combine_grouped(p, pl)) rpw /= std::min<int64_t>(rpw, pl.workers / (4 * segs));
    const int64_t want = (pl.rows + rpw - 1) / rpw;
    if (combine_per_worker(p, pl)) return dim3((unsigned)pl.workers, (unsigned)want);
    const int64_t room = segs >= 4096 ? 1 : 4096 / segs;
    return dim3((unsigned)segs, (unsigned)std::min(want, room));
}

}  // namespace spire
