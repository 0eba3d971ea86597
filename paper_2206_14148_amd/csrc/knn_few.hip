// gfx950 (CDNA4, MI355X) kNN search for small problems, squared-Euclidean metric, d > 8: so few
// pairs that evaluating each of them exactly (the key of exact_partial, knn_exact.h, the same bits)
// costs less than the rounded copies, norms, shared thresholds and list restarts of the matrix-core
// filters.  One pass over the points, no preparation.
//
// A wave owns 64 points at a time, one per lane, and NQ queries.  Pieces of 32 coordinates of the
// points go through LDS (read there with rows side by side, 128 bytes each; used with a lane per
// row, rows 33 words apart: conflicts in 1.5 % of the cycles), the queries' coordinates are the same for the whole
// wave and come through scalar loads, and every point value read feeds NQ queries.  Pairs under a
// query's current k-th key wait in a buffer of 64 and are merged into its list when that is full.
//
// What bounds it: 1000 x 1e4, d = 16, k = 10 3.1e7 vector instructions, of which the keys, two operations per pair and
// coordinate, are 5e6 and most others the lists' merges; vector units active in 39 % of the wave cycles, waits 35 %.  At 16
// queries x 1e5 points, d = 50, k = 10 the round trips of a wave's groups of points: 50 us here, 22 us for the merge of
// 391 lists a query.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "knn_config.h"
#include "knn_device.h"
#include "knn_kernels.h"

namespace knn {

namespace {

constexpr int kPiece = 32;            // coordinates staged at a time
constexpr int kStride = kPiece + 1;   // words per staged row
constexpr int kFewWaves = 4;

constexpr size_t few_lds_per_wave(int nq, int k) {
    return (size_t)(64 * kStride + nq * 2 * kWave + 2 * kWave + 2 * k) * 4;
}

// (ALIGNED: d % 4 == 0; rows begin at any multiple of 4 bytes)
template <int NQ, bool ALIGNED>
__global__ __launch_bounds__(64 * kFewWaves) void knn_few_kernel(
    const float* __restrict__ Q, int64_t ldq, const float* __restrict__ X, int64_t ldx, int rows, int n, int d,
    int k, int S, int split_len, float* __restrict__ lk, int* __restrict__ li) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // (uniform: scalar loads of the queries)
    float* const xt = reinterpret_cast<float*>(smem + (size_t)wave * few_lds_per_wave(NQ, k));  // [64][kStride]
    float* const ck = xt + 64 * kStride;                     // [NQ][64] keys of buffered pairs
    int* const ci = reinterpret_cast<int*>(ck + NQ * kWave);  // [NQ][64] their points
    MergeScratch sc;
    sc.cand_key = reinterpret_cast<float*>(ci + NQ * kWave);
    sc.cand_idx = reinterpret_cast<int*>(sc.cand_key + kWave);
    sc.list_key = reinterpret_cast<float*>(sc.cand_idx + kWave);
    sc.list_idx = reinterpret_cast<int*>(sc.list_key + k);

    // one (group of queries, range of points) per wave, the ranges of a group side by side
    const int id = (int)blockIdx.x * kFewWaves + wave;  // (few_applies keeps the number of waves small)
    const int s = __builtin_amdgcn_readfirstlane(id % S);
    const int r0 = __builtin_amdgcn_readfirstlane(id / S) * NQ;
    if (r0 >= rows) return;  // whole wave; no workgroup barrier below
    const int j0 = s * split_len;
    const int j1 = min(n, j0 + split_len);
    const float* qp[NQ];
    float tau[NQ];
    int cnt[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        qp[i] = Q + (int64_t)min(r0 + i, rows - 1) * ldq;
        tau[i] = r0 + i < rows ? kInf : -kInf;
        cnt[i] = 0;
        if (r0 + i < rows) {
            const size_t lb = ((size_t)(r0 + i) * S + s) * k;
            for (int p = lane; p < k; p += kWave) {
                lk[lb + p] = kInf;
                li[lb + p] = kNoIdx;
            }
        }
    }
    auto flush = [&](int i) {
        wave_sync();
        const size_t lb = ((size_t)(r0 + i) * S + s) * k;
        const float key = lane < cnt[i] ? ck[i * kWave + lane] : kInf;
        const int id = lane < cnt[i] ? ci[i * kWave + lane] : kNoIdx;
        tau[i] = wave_merge(lk + lb, li + lb, k, key, id, sc, lane, cnt[i]);
        cnt[i] = 0;
    };

    // staging: eight lanes per row, four coordinates each, eight rows an instruction
    const int srow = lane >> 3, scol = (lane & 7) * 4;
    f32x4 g[8];
    auto fetch = [&](int j, int t0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* row = X + (int64_t)min(j + 8 * u + srow, j1 - 1) * ldx;
            const int t = t0 + scol;
            if (ALIGNED)
                g[u] = load4(row + (t < d ? t : 0));
            else
                g[u] = load4(row + min(t, d - 4));  // (the last group begins earlier: see the stores)
        }
    };
    if (j0 < j1) fetch(j0, 0);
    for (int j = j0; j < j1; j += 64) {
        // the two chains of a key: coordinates in groups of four, even groups and odd groups
        float s0[NQ], s1[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) s0[i] = s1[i] = 0.f;
        for (int t0 = 0; t0 < d; t0 += kPiece) {
            wave_sync();
            // (where a lane's group begins earlier than its place, it stores what its neighbour does, the same values)
            const int to = ALIGNED ? scol : min(t0 + scol, d - 4) - t0;
            if (ALIGNED || t0 + 4 <= d) {
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) xt[(8 * u + srow) * kStride + to + e] = g[u][e];
            } else {  // fewer than four coordinates in the row's last piece: some of the group belong to the piece before
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (to + e >= 0) xt[(8 * u + srow) * kStride + to + e] = g[u][e];
            }
            wave_sync();
            if (t0 + kPiece < d) fetch(j, t0 + kPiece);
            else if (j + 64 < j1) fetch(j + 64, 0);
            const float* x = xt + lane * kStride;
            if (t0 + kPiece <= d) {
#pragma unroll
                for (int t = 0; t < kPiece; ++t) {
                    const float xv = x[t];
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
                        const float df = qp[i][t0 + t] - xv;
                        if (t & 4) s1[i] = fmaf(df, df, s1[i]);
                        else s0[i] = fmaf(df, df, s0[i]);
                    }
                }
            } else {
                // whole groups of eight, then one by one (a coordinate past d adds nothing)
                int t = 0;
                for (; t0 + t + 8 <= d; t += 8) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float xv = x[t + e];
#pragma unroll
                        for (int i = 0; i < NQ; ++i) {
                            const float df = qp[i][t0 + t + e] - xv;
                            if (e & 4) s1[i] = fmaf(df, df, s1[i]);
                            else s0[i] = fmaf(df, df, s0[i]);
                        }
                    }
                }
                for (; t0 + t < d; ++t) {
                    const float xv = x[t];
                    const bool odd = t & 4;  // uniform
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
                        const float df = qp[i][t0 + t] - xv;
                        if (odd) s1[i] = fmaf(df, df, s1[i]);
                        else s0[i] = fmaf(df, df, s0[i]);
                    }
                }
            }
        }
        const bool in = j + lane < j1;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const float key = s0[i] + s1[i];
            uint64_t ok = __builtin_amdgcn_ballot_w64(in && key < tau[i]);
            if (ok == 0) continue;
            if (cnt[i] + __builtin_popcountll(ok) > kWave) {
                flush(i);
                ok = __builtin_amdgcn_ballot_w64(in && key < tau[i]);
            }
            if ((ok >> lane) & 1) {
                const int at = cnt[i] + __builtin_popcountll(ok & ((1ull << lane) - 1));
                ck[i * kWave + at] = key;
                ci[i * kWave + at] = j + lane;
            }
            cnt[i] += __builtin_popcountll(ok);
        }
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i)
        if (cnt[i] > 0) flush(i);
}

}  // namespace

// A pair costs d + 16 or so (the rest is its share of the test against the threshold), 1e13 of these a
// second where rows can be loaded 16 bytes at a time and 5.7e12 where not; the filters cost a pass over
// the points and the restarts of their lists before they gain anything, the more so the fewer
// queries there are and the longer the lists.  Measured, us a call here / on the filter paths, by m, n, d, k:
//   16, 1e5, 50, 10: 97 / 590       1000, 1e4, 16, 10: 106 / 457     300, 1e5, 64, 10: 226 / 531
//   1000, 1e5, 16, 10: 356 / 702    1e4, 1e4, 16, 10: 408 / 516      1000, 2e4, 100, 100: 449 / 4845
//   1000, 1e5, 64, 10: 584 / 548    3000, 1e5, 16, 10: 831 / 539     3000, 3e4, 100, 10: 851 / 740
//   64, 1e6, 128, 10: 722 / 1003    64, 1e6, 256, 32: 1851 / 1859    16, 1e6, 1000, 10: 2709 / 6423
// and at the other end of k, where lists restart hardly at all:
//   1000, 1e4, 16, 1: 68 / 161      1000, 1e4, 128, 1: 133 / 220     1000, 1e4, 300, 1: 287 / 382
//   1000, 65536, 16, 1: 214 / 206   1000, 65536, 9, 1: 336 / 221     1000, 65536, 9, 10: 394 / 754
//   1000, 2e5, 9, 1: 877 / 286      2e4, 1e4, 9, 10: 939 / 687       4000, 1e4, 50, 10: 513 / 649
// Up to 64 queries, against a split path with a range for every compute unit, k = 1 / 10 / 100, here and there:
//   40, 1e6, 230: 1754 1747 1935 / 710 1104 5610      40, 2e6, 50: 667 686 989 / 543 884 4084
//   16, 1e6, 230: 522 566 1051 / 587 839 3354         40, 5e6, 12: 706 759 1158 / 451 928 4769
// From 65 queries on the line is a bound from below of what the filters take, up to 5e9 in all.
bool few_applies(int64_t m, int64_t n, int d, int k, bool aligned) {
    const double work = (double)m * (double)n * (double)(d + 16);
    if (k > kFewMaxK) return false;
    if (m <= 64) {
        // the split path reads the points twice, whatever m is, and restarts its lists in a range per compute unit
        const double split_us = 300.0 + 1.8e-6 * (double)n * d + 40.0 * k;
        return work <= (m <= 16 ? 2e10 : 1e10) && 40.0 + 1.2e-7 * work <= 1.25 * split_us;
    }
    const double here_us = 40.0 + work * (aligned ? 1.0e-7 : 1.75e-7);
    const double copy_us = 3e-5 * (double)n * d;
    const double filter_us = (aligned ? 150.0 + 0.75 * d : 165.0 + 1.5 * d) + (copy_us < 150.0 ? copy_us : 150.0) +
                             (k - 1) * (n >= 50000 ? 55.0 : (aligned ? 22.0 : 30.0));
    return work <= 5e9 && here_us <= filter_us;
}

int few_splits(int64_t rows, int64_t n, int d, int k, uint64_t workspace_bytes) {
    // two waves a SIMD where the points last (ranges of at least 256), lists that fit.  (Registers and LDS leave room for three, but
    // a wave's list begins anew in every range: us with two / three / four 1000 x 1e4, d = 16, k = 10 91 / 100 / 133, 16 x 1e6,
    // d = 100 261 / 308 / 441; 300 x 3e4, d = 257 334 / 277 / 430; 312 sizes in the mean 107.4 / 108.8 / 120.3.)
    const int64_t groups = (rows + kFewQueries - 1) / kFewQueries;
    int64_t S = 2 * 4 * kNumCU / groups;
    if (S > (n + 255) / 256) S = (n + 255) / 256;
    if (S > kFewMaxSplits) S = kFewMaxSplits;
    // Long lists are merged at length, at some 2 us for 64 entries: no more ranges than keep that below what they save.  us with and
    // without this line: 16 x 3e5, d = 16, k = 128 389 / 495, 1 x 1e6, k = 100 315 / 528; where a range is much work they pay: 64 x 3e5,
    // d = 300, k = 100 875 with 128 ranges, 1129 with 122 (whole 32s: the groups of queries that read a range share an L2).
    if (k > kFewLongK) {
        int64_t most = n * (d + 16) / kFewLongWork;
        if (most < kFewLongEntries / k) most = kFewLongEntries / k;
        most = (most + 31) / 32 * 32;
        if (S > most) S = most;
    }
    const uint64_t room = workspace_bytes / 2 / kAlign * kAlign;  // keys and indices, each aligned
    const int64_t fit = (int64_t)(room / ((uint64_t)rows * (uint64_t)k * 4));
    if (S > fit) S = fit;
    return S < 1 ? (fit < 1 ? 0 : 1) : (int)S;
}

hipError_t launch_few(const float* Q, int64_t ldq, const float* X, int64_t ldx, int64_t rows, int64_t n, int d,
                      int k, int S, float* lk, int* li, hipStream_t stream) {
    constexpr int NQ = kFewQueries;
    const size_t lds = kFewWaves * few_lds_per_wave(NQ, k);
    int64_t split_len = (n + S - 1) / S;
    split_len = (split_len + 63) / 64 * 64;
    const bool aligned = whole_rows(d);
    const dim3 grid((unsigned)(((rows + NQ - 1) / NQ * S + kFewWaves - 1) / kFewWaves));
    hipError_t e = aligned ? raise_lds_limit(knn_few_kernel<NQ, true>, lds)
                           : raise_lds_limit(knn_few_kernel<NQ, false>, lds);
    if (e != hipSuccess) return e;
    if (aligned)
        knn_few_kernel<NQ, true><<<grid, dim3(64 * kFewWaves), lds, stream>>>(Q, ldq, X, ldx, (int)rows, (int)n, d, k,
                                                                              S, (int)split_len, lk, li);
    else
        knn_few_kernel<NQ, false><<<grid, dim3(64 * kFewWaves), lds, stream>>>(Q, ldq, X, ldx, (int)rows, (int)n, d, k,
                                                                               S, (int)split_len, lk, li);
    return hipGetLastError();
}

}  // namespace knn
