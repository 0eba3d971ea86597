// gfx950 (CDNA4, MI355X): L1 search of many queries through byte sums (the L1 rows of the paper's
// table).  knn_l1_kernel makes the fp32 key of every pair, two vector operations per coordinate.
// Here both sides are rounded to bytes on one common scale, x = lo + s b + e, and v_sad_u8 adds
// four coordinates' absolute differences per operation:
//     sum_t |q_t - x_t|  >=  s sum_t |b_q - b_x|  -  sum_t |e_q|  -  sum_t |e_x| .
// A pair whose bound exceeds its query's threshold cannot be among the k nearest; the others get
// the fp32 key of knn_l1_kernel (ascending t, one chain of additions), so that lists and results
// are the same bits.  The scale comes from a sample of the points: a value outside it is cut to 0
// or 255 and its e is as large as it is, so the bound holds for any data, and an infinity or NaN
// makes its e infinite or NaN and passes the filter on every pair.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "knn_config.h"
#include "knn_device.h"
#include "knn_kernels.h"

namespace knn {

namespace {

constexpr int kSadPoints = 64;             // points of a tile (four threads round one of them)
constexpr int kSadCand = 16;               // buffered point indices per query (LDS)
constexpr unsigned kSadBase = 1u << 24;    // where a pair's sum starts, minus its point's allowance
constexpr float kSadMost = 8388608.f;      // allowances are cut here: beyond 255 * 256, so "passes always"
constexpr int kSadMaxK = 64;
constexpr int64_t kSadMinPoints = 4096;
constexpr int64_t kSadPointsPerK = 3000;
constexpr int kSadMaxD = 192;
constexpr int kSadPassDivisor = 60;       // more than one pair in so many passes the probe: not worth filtering
constexpr int kSadTwoWorkgroups = 200;       // fewer (of two queries per lane): one per lane

struct SadScale {
    float lo, s, inv;
    float slack;  // what the rounding errors of the residuals themselves add, in units of s
};

struct SadHeader {
    SadScale scale;
    unsigned passed;  // pairs of the probe that passed the first thresholds
};

// A residual sum or a key (in units of the data) as a whole number of units s, never too small.
// NaN, infinities and anything past kSadMost give kSadMost.
__device__ __forceinline__ unsigned sad_units(float v, const SadScale& c) {
    const float u = v * c.inv * 1.0001f + c.slack;
    return u < kSadMost ? (unsigned)u + 1u : (unsigned)kSadMost;
}

// One workgroup: the range of a sample of 32768 values, cut at eight mean deviations from their mean
// (a few far values would make every unit coarse; cut, they cost their own points a looser bound).
__global__ __launch_bounds__(1024) void knn_l1_scale_kernel(const float* __restrict__ X, int64_t ldx, int n, int d,
                                                            SadHeader* __restrict__ out) {
    __shared__ float part[3][16];
    const int tid = threadIdx.x;
    const float* p = X + (int64_t)((int64_t)tid * n / 1024) * ldx;
    float v[32];
    float lo = kInf, hi = -kInf, sum = 0.f, many = 0.f;
    // the workgroup's minimum, maximum and sum of one value per thread each, in every thread
    auto all = [&](float& a, float& b, float& c) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            a = fminf(a, __shfl_xor(a, o));
            b = fmaxf(b, __shfl_xor(b, o));
            c += __shfl_xor(c, o);
        }
        __syncthreads();
        if ((tid & 63) == 0) {
            part[0][tid >> 6] = a;
            part[1][tid >> 6] = b;
            part[2][tid >> 6] = c;
        }
        __syncthreads();
        a = part[0][0];
        b = part[1][0];
        c = part[2][0];
        for (int w = 1; w < 16; ++w) {
            a = fminf(a, part[0][w]);
            b = fmaxf(b, part[1][w]);
            c += part[2][w];
        }
    };
#pragma unroll
    for (int u = 0; u < 32; ++u) {
        v[u] = p[(tid * 7 + u) % d];
        const bool ok = fabsf(v[u]) < 1e30f;
        lo = ok ? fminf(lo, v[u]) : lo;
        hi = ok ? fmaxf(hi, v[u]) : hi;
        sum += ok ? v[u] : 0.f;
        many += ok ? 1.f : 0.f;
    }
    float x0 = 0.f, x1 = 0.f;
    all(lo, hi, sum);
    all(x0, x1, many);
    const float mean = sum / fmaxf(many, 1.f);
    float dev = 0.f;
#pragma unroll
    for (int u = 0; u < 32; ++u) dev += fabsf(v[u]) < 1e30f ? fabsf(v[u] - mean) : 0.f;
    all(x0, x1, dev);
    dev /= fmaxf(many, 1.f);
    if (tid != 0) return;
    lo = fmaxf(lo, mean - 8.f * dev);
    hi = fminf(hi, mean + 8.f * dev);
    SadScale c;
    const bool any = lo <= hi;
    c.lo = any ? lo : 0.f;
    const float s = any ? (hi - lo) * (1.f / 255.f) : 1.f;
    // (equal values: any unit will do; one far below their size would only lose in rounding)
    c.s = fmaxf(fmaxf(s, fabsf(c.lo) * 1e-6f), 1e-30f);
    c.inv = 1.f / c.s;
    // an e is off by 2^-24 of lo + s b and of itself (the factor in sad_units); d of them
    c.slack = (float)d * 1.2e-7f * (fabsf(c.lo) * c.inv + 256.f);
    out->scale = c;
    out->passed = 0;
}

// byte and residual of one value
__device__ __forceinline__ unsigned sad_byte(float x, const SadScale& c, float& resid) {
    const float v = rintf((x - c.lo) * c.inv);
    const float b = fminf(fmaxf(v, 0.f), 255.f);  // NaN: 0
    resid += fabsf(x - fmaf(c.s, b, c.lo));
    return (unsigned)b;
}

// Queries: bytes in blocks of 64 rows, word w of the block's rows side by side, zeros past the rows
// and past d; their residual sums; thresholds that start from 0, for knn_l1_seed_kernel to raise.
__global__ __launch_bounds__(256) void knn_l1_bytes_kernel(const float* __restrict__ Q, int64_t ldq, int rows, int d,
                                                           int words, const SadHeader* __restrict__ head,
                                                           unsigned* __restrict__ qb, float* __restrict__ qr,
                                                           unsigned* __restrict__ tsh) {
    const int r = blockIdx.x * 64 + (threadIdx.x >> 2), sub = threadIdx.x & 3;
    const SadScale c = head->scale;
    float resid = 0.f;
    for (int w = sub; w < words; w += 4) {
        unsigned v = 0;
        if (r < rows) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * w + e < d) v |= sad_byte(Q[(int64_t)r * ldq + 4 * w + e], c, resid) << (8 * e);
        }
        qb[((int64_t)blockIdx.x * words + w) * 64 + (threadIdx.x >> 2)] = v;
    }
    resid += lane_xor<1>(resid);
    resid += lane_xor<2>(resid);
    if (sub == 0) {
        qr[r] = resid;
        tsh[r] = 0;
    }
}

// A tile of points on its way to bytes in LDS: a workgroup of 256 threads, chunks sub, sub + 4, ... of
// point tid / 4 in each.  fetch asks for the values, store rounds them and returns the point's
// allowance (in all four of its threads).
template <int NC>
struct PointRounder {
    static constexpr int CT = (NC + 3) / 4;
    const float* __restrict__ X;
    int64_t ldx;
    int n, dims, aligned;
    SadScale cs;
    float ahead[CT][16];

    __device__ __forceinline__ PointRounder(const float* X_, int64_t ldx_, int n_, int d_, int aligned_, SadScale cs_)
        : X(X_), ldx(ldx_), n(n_), dims(d_), aligned(aligned_), cs(cs_) {}

    // (the comparisons with d are made anew for every tile: kept, they would fill the register file)
    __device__ __forceinline__ int fresh_d() const {
        int d = dims;
        asm volatile("" : "+s"(d));
        return d;
    }
    __device__ __forceinline__ void fetch(int j, int j1) {
        const int d = fresh_d();
        const float* __restrict__ p = X + (int64_t)min(j + (int)(threadIdx.x >> 2), j1 - 1) * ldx;
#pragma unroll
        for (int i = 0; i < CT; ++i) {
            const int t = ((threadIdx.x & 3) + 4 * i) * 16;
            if (aligned) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(p + (t + 4 * u < d ? t + 4 * u : 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) ahead[i][4 * u + e] = v[e];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 16; ++u) ahead[i][u] = p[t + u < d ? t + u : 0];
            }
        }
    }
    __device__ __forceinline__ unsigned store(uint4* tile) {
        const int d = fresh_d();
        float resid = 0.f;
#pragma unroll
        for (int i = 0; i < CT; ++i) {
            const int c = (threadIdx.x & 3) + 4 * i;
            unsigned w[4] = {0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                float e = 0.f;
                const unsigned b = sad_byte(ahead[i][u], cs, e);
                const bool in = c * 16 + u < d;
                w[u >> 2] |= in ? b << (8 * (u & 3)) : 0u;
                resid += in ? e : 0.f;
            }
            if (c < NC) tile[(threadIdx.x >> 2) * NC + c] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        resid += lane_xor<1>(resid);
        resid += lane_xor<2>(resid);
        return sad_units(resid, cs);
    }
};

// Sums of 64 queries x QL per wave against two points of a tile.
template <int W, int QL>
__device__ __forceinline__ void sad_two(const uint4* tile, const unsigned (&qv)[QL][W], int p,
                                        unsigned (&acc)[2][QL]) {
    constexpr int NC = (W + 3) / 4;
#pragma unroll
    for (int c = 0; c < W / 4; ++c) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint4 w = tile[(p + u) * NC + c];
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                acc[u][q] = __builtin_amdgcn_sad_u8(qv[q][4 * c + 0], w.x, acc[u][q]);
                acc[u][q] = __builtin_amdgcn_sad_u8(qv[q][4 * c + 1], w.y, acc[u][q]);
                acc[u][q] = __builtin_amdgcn_sad_u8(qv[q][4 * c + 2], w.z, acc[u][q]);
                acc[u][q] = __builtin_amdgcn_sad_u8(qv[q][4 * c + 3], w.w, acc[u][q]);
            }
        }
    }
    if constexpr (W % 4 != 0) {
        static_assert(W % 4 == 2, "rows are whole pairs of words");
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint2 w = *reinterpret_cast<const uint2*>(tile + (p + u) * NC + W / 4);
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                acc[u][q] = __builtin_amdgcn_sad_u8(qv[q][W - 2], w.x, acc[u][q]);
                acc[u][q] = __builtin_amdgcn_sad_u8(qv[q][W - 1], w.y, acc[u][q]);
            }
        }
    }
}

// First thresholds.  A sample of `tiles` tiles of 64 points, spread evenly, is dealt into k groups;
// the nearest point of every group by the upper bound s sum + e_q + e_x makes k different points,
// so the largest of those k bounds is no less than the k-th key.  Group g is made by workgroup
// row g % gridDim.y.  probe: instead, one tile per workgroup row, halfway between tiles of the
// sample, is tested with these thresholds and the pairs that pass are counted.
// A workgroup has 128 queries, all in every wave, and its waves share out a tile's points: few
// queries still make k workgroups per 128 of them.
template <int W>
__global__ __launch_bounds__(256) void knn_l1_seed_kernel(const float* __restrict__ X, int64_t ldx,
                                                          const unsigned* __restrict__ qb, const float* __restrict__ qr,
                                                          unsigned* __restrict__ tsh, SadHeader* __restrict__ head,
                                                          int rows, int n, int d, int k, int per_group, int aligned,
                                                          int probe) {
    constexpr int NC = (W + 3) / 4, QL = 2, PW = kSadPoints / 4;
    __shared__ __align__(16) uint4 tile[kSadPoints * NC];
    __shared__ __align__(16) unsigned start[kSadPoints];
    __shared__ unsigned nearest[4][QL][kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const SadScale cs = head->scale;
    const int row0 = blockIdx.x * (kWave * QL);
    const int nq = min(kWave * QL, rows - row0);
    unsigned qv[QL][W];
    float qres[QL];
#pragma unroll
    for (int q = 0; q < QL; ++q) {
        const bool block = q * kWave < nq;
#pragma unroll
        for (int w = 0; w < W; ++w) qv[q][w] = block ? qb[((size_t)(row0 / kWave + q) * W + w) * kWave + lane] : 0u;
        qres[q] = block ? qr[row0 + q * kWave + lane] : 0.f;
    }
    PointRounder<NC> round(X, ldx, n, d, aligned, cs);
    const int tiles = k * per_group;
    const int64_t step = n / tiles;  // >= 64
    if (probe) {
        const int j = (int)min((int64_t)((int64_t)blockIdx.y * tiles / gridDim.y) * step + step / 2, (int64_t)n - kSadPoints);
        round.fetch(j, n);
        const unsigned r = round.store(tile);
        if ((tid & 3) == 0) start[tid >> 2] = kSadBase - r;
        __syncthreads();
        unsigned T[QL], passed = 0;
#pragma unroll
        for (int q = 0; q < QL; ++q)
            T[q] = q * kWave + lane < nq
                       ? kSadBase + sad_units(__uint_as_float(tsh[row0 + q * kWave + lane]) + qres[q], cs)
                       : 0u;
        for (int p = wave * PW; p < (wave + 1) * PW; p += 2) {
            unsigned acc[2][QL];
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                acc[0][q] = start[p];
                acc[1][q] = start[p + 1];
            }
            sad_two<W, QL>(tile, qv, p, acc);
#pragma unroll
            for (int q = 0; q < QL; ++q) passed += (acc[0][q] <= T[q]) + (acc[1][q] <= T[q]);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) passed += __shfl_xor(passed, o);
        if (lane == 0 && passed) atomicAdd(&head->passed, passed);
        return;
    }
    for (int g = blockIdx.y; g < k; g += gridDim.y) {
        unsigned best[QL];
#pragma unroll
        for (int q = 0; q < QL; ++q) best[q] = 0xffffffffu;
        round.fetch((int)((int64_t)g * step), n);
        for (int i = 0; i < per_group; ++i) {
            const unsigned r = round.store(tile);
            if ((tid & 3) == 0) start[tid >> 2] = r;
            __syncthreads();
            if (i + 1 < per_group) round.fetch((int)(((int64_t)(i + 1) * k + g) * step), n);
            for (int p = wave * PW; p < (wave + 1) * PW; p += 2) {
                unsigned acc[2][QL];
#pragma unroll
                for (int q = 0; q < QL; ++q) {
                    acc[0][q] = start[p];
                    acc[1][q] = start[p + 1];
                }
                sad_two<W, QL>(tile, qv, p, acc);
#pragma unroll
                for (int q = 0; q < QL; ++q) best[q] = min(best[q], min(acc[0][q], acc[1][q]));
            }
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < QL; ++q) nearest[wave][q][lane] = best[q];
        __syncthreads();
        if (wave < QL) {  // (a group has a barrier of its own before `nearest` is written again)
            const int q = wave;
            const unsigned near = min(min(nearest[0][q][lane], nearest[1][q][lane]), min(nearest[2][q][lane], nearest[3][q][lane]));
            const float resid = q * kWave < nq ? qr[row0 + q * kWave + lane] : 0.f;
            // (an allowance that was cut says nothing about the point)
            const float t = near < (unsigned)kSadMost ? ((float)near + 1.f) * cs.s * 1.0002f + resid * 1.0002f : kInf;
            if (q * kWave + lane < nq) atomicMax(tsh + row0 + q * kWave + lane, __float_as_uint(t < kInf ? t : kInf));
        }
    }
}

// d / 4 sums per pair (v_sad_u8 measured at half the rate of an fp32 operation: 1e4 queries, 1e6 points, d = 100
// need 12.7 ms at 2.4 GHz and take 16.5 with the candidates left out; waits are 62 % of the wave cycles, so that the
// vector units are not all that binds) and one LDS read of 16 bytes per QL * 4 of them.  A lane keeps QL queries' bytes in registers, the workgroup
// rounds a tile of 64 points to bytes in LDS and every wave reads a point's bytes as a broadcast.
// Two queries per lane and two workgroups per compute unit: the second hides the first one's
// flushes and barriers (four queries per lane, one workgroup: 27.6 ms against 21.6).  Whole search
// at that size, k = 10: 65.6 -> 22.4 ms; 1000 queries 13.8 -> 4.8, 16 queries 12.5 -> 3.0.
template <int W, int QL>
__global__ __launch_bounds__(256, W <= 32 ? 2 : 1) void knn_l1_sad_kernel(
    const float* __restrict__ Q, int64_t ldq, const float* __restrict__ X, int64_t ldx,
    const unsigned* __restrict__ qb, const float* __restrict__ qr, unsigned* __restrict__ tsh,
    const SadHeader* __restrict__ head, int rows, int n, int d, int k, int S, int split_len, int aligned,
    unsigned most_passed, float* __restrict__ lk, int* __restrict__ li) {
    constexpr int NC = (W + 3) / 4;
    constexpr int C = kSadCand;
    extern __shared__ __align__(16) unsigned char smem[];
    uint4* const tile = reinterpret_cast<uint4*>(smem);                              // [points][NC]
    unsigned* const start = reinterpret_cast<unsigned*>(tile + kSadPoints * NC);     // [points]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned char* const mine =
        reinterpret_cast<unsigned char*>(start + kSadPoints) + (size_t)wave * (QL * C * kWave + 2 * kWave + 2 * k) * 4;
    int* const ci = reinterpret_cast<int*>(mine);  // [QL][C][64]
    MergeScratch sc;
    sc.cand_key = reinterpret_cast<float*>(ci + QL * C * kWave);
    sc.cand_idx = reinterpret_cast<int*>(sc.cand_key + kWave);
    sc.list_key = reinterpret_cast<float*>(sc.cand_idx + kWave);
    sc.list_idx = reinterpret_cast<int*>(sc.list_key + k);

    const SadScale cs = head->scale;
    const bool redo = head->passed > most_passed;
    const int s = blockIdx.y;
    const int row0 = (blockIdx.x * 4 + wave) * (kWave * QL);
    const int nq = min(kWave * QL, rows - row0);  // <= 0: an idle wave, which still rounds points
    for (int i = lane; i < nq * k; i += kWave) {
        const size_t at = ((size_t)(row0 + i / k) * S + s) * k + i % k;
        lk[at] = kInf;
        li[at] = redo ? kL1Redo : kNoIdx;
    }
    if (redo) return;  // (the same for every workgroup) the filter lets too much through
    unsigned qv[QL][W], T[QL];  // T: the largest sum that passes
    float qres[QL];
    int cnt[QL];
#pragma unroll
    for (int q = 0; q < QL; ++q) {
        const bool on = q * kWave + lane < nq;
        const bool block = q * kWave < nq;
#pragma unroll
        for (int w = 0; w < W; ++w)
            qv[q][w] = block ? qb[((size_t)(row0 / kWave + q) * W + w) * kWave + lane] : 0u;
        qres[q] = on ? qr[row0 + q * kWave + lane] : 0.f;
        T[q] = on ? kSadBase + (unsigned)kSadMost : 0u;
        cnt[q] = 0;
    }

    const int j0 = s * split_len, j1 = min(n, j0 + split_len);

    // Exact keys and merges of every query of the wave with at least `least` buffered points: four
    // queries at a time, a lane per point.
    auto flush = [&](int least) {
#pragma unroll 1
        for (int q = 0; q < QL; ++q) {
            int cq = cnt[0];
#pragma unroll
            for (int u = 1; u < QL; ++u) cq = q == u ? cnt[u] : cq;
            uint64_t mask = __builtin_amdgcn_ballot_w64(cq >= least);
#pragma unroll
            for (int u = 0; u < QL; ++u) cnt[u] = (q == u && cq >= least) ? 0 : cnt[u];
            while (mask) {
                const int L0 = __builtin_ctzll(mask);
                int own = L0, ng = 0;
                uint64_t m4 = mask;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if (m4) {
                        const int L = __builtin_ctzll(m4);
                        m4 &= m4 - 1;
                        own = (lane >> 4) == g ? L : own;
                        ng = g + 1;
                    }
                }
                wave_sync();
                const int slot = lane & 15;
                const int have = __shfl(cq, own);
                bool ok = (lane >> 4) < ng && slot < have;
                const int j = ok ? ci[(q * C + slot) * kWave + own] : j0;
                const int r = row0 + q * kWave + own;
                const float* __restrict__ qp = Q + (int64_t)r * ldq;
                const float* __restrict__ xp = X + (int64_t)j * ldx;
                float key = 0.f;
                if (aligned) {
                    int t = 0;
                    for (; t + 16 <= d; t += 16) {
                        f32x4 a[4], b[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            a[u] = *reinterpret_cast<const f32x4*>(qp + t + 4 * u);
                            b[u] = *reinterpret_cast<const f32x4*>(xp + t + 4 * u);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) key += fabsf(a[u][e] - b[u][e]);
                    }
                    for (; t < d; t += 4) {
                        const f32x4 a = *reinterpret_cast<const f32x4*>(qp + t);
                        const f32x4 b = *reinterpret_cast<const f32x4*>(xp + t);
#pragma unroll
                        for (int e = 0; e < 4; ++e) key += fabsf(a[e] - b[e]);
                    }
                } else {
                    int t = 0;
                    for (; t + 8 <= d; t += 8) {
                        float a[8], b[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            a[u] = qp[t + u];
                            b[u] = xp[t + u];
                        }
#pragma unroll
                        for (int u = 0; u < 8; ++u) key += fabsf(a[u] - b[u]);
                    }
                    for (; t < d; ++t) key += fabsf(qp[t] - xp[t]);
                }
                const float bound = __uint_as_float(__hip_atomic_load(tsh + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                ok = ok && key < kInf && key <= bound;  // (NaN and infinite keys enter no list)
                for (int g = 0; g < ng; ++g) {
                    const int L = __builtin_ctzll(mask);
                    mask &= mask - 1;
                    const uint64_t oks = __builtin_amdgcn_ballot_w64(ok) >> (16 * g) & 0xffffull;
                    if (!oks) continue;
                    const float kk = __shfl(key, 16 * g + slot);
                    const int jj = __shfl(j, 16 * g + slot);
                    const bool in = lane < 16 && (oks >> slot & 1);
                    const int rr = row0 + q * kWave + L;
                    const size_t lb = ((size_t)rr * S + s) * k;
                    const float t_new = merged_key(wave_merge_pair_inline(lk + lb, li + lb, k, in ? kk : kInf,
                                                                          in ? jj : kNoIdx, sc, lane, 16));
                    if (lane == 0) atomicMin(tsh + rr, __float_as_uint(t_new));
#pragma unroll
                    for (int u = 0; u < QL; ++u)
                        if (u == q && lane == L) T[u] = min(T[u], kSadBase + sad_units(t_new + qres[u], cs));
                }
            }
        }
    };

    PointRounder<NC> round(X, ldx, n, d, aligned, cs);
    for (int j = j0; j < j1; j += kSadPoints) {
        round.fetch(j, j1);
        const unsigned r = round.store(tile);
        if ((tid & 3) == 0) start[tid >> 2] = j + (tid >> 2) < j1 ? kSadBase - r : 0xf0000000u;
        __syncthreads();
        if (nq > 0) {
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                if (q * kWave + lane < nq) {
                    const float t = __uint_as_float(__hip_atomic_load(tsh + row0 + q * kWave + lane, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT));
                    T[q] = min(T[q], kSadBase + sad_units(t + qres[q], cs));
                }
            }
#pragma unroll 1
            for (int p = 0; p < kSadPoints; p += 2) {
                unsigned acc[2][QL];
                const uint2 st = *reinterpret_cast<const uint2*>(start + p);
#pragma unroll
                for (int q = 0; q < QL; ++q) {
                    acc[0][q] = st.x;
                    acc[1][q] = st.y;
                }
                sad_two<W, QL>(tile, qv, p, acc);
                bool hit = false;
#pragma unroll
                for (int q = 0; q < QL; ++q) hit |= (acc[0][q] <= T[q]) | (acc[1][q] <= T[q]);
                if (__builtin_amdgcn_ballot_w64(hit)) {
                    bool full = false;
#pragma unroll
                    for (int q = 0; q < QL; ++q) {
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            if (acc[u][q] <= T[q]) {
                                ci[(q * C + cnt[q]) * kWave + lane] = j + p + u;
                                ++cnt[q];
                            }
                        }
                        full |= cnt[q] > C - 2;  // the next two points might not fit
                    }
                    if (__builtin_amdgcn_ballot_w64(full)) flush(C / 2);
                }
            }
        }
        __syncthreads();
    }
    if (nq > 0) flush(1);
}

}  // namespace

// The filter pays where a first threshold from a sample lets few pairs through, n at least some
// thousand times k (1e4 queries, ms with the filter / without: 2e4 points, d = 64, k = 10 1.7 / 2.6;
// 7e4, d = 24, k = 32 5.1 / 5.8; but 4e4, d = 100, k = 16 5.3 / 4.9, and 1e4, d = 150, k = 32, where
// nearly all time went into candidates).  From five coordinates on the queries' area has room for
// the bytes (1e6 points, d = 5, k = 10: 6.9 / 21.0); up to 192 the registers hold two queries.
bool l1_sad_applies(int64_t rows, int64_t n, int d, int k) {
    return rows > 0 && d >= 5 && d <= kSadMaxD && k <= kSadMaxK && n >= kSadMinPoints && n >= kSadPointsPerK * k;
}

struct SadCall {
    const float* Q;
    int64_t ldq;
    const float* X;
    int64_t ldx;
    SadHeader* head;
    float* qr;
    unsigned* tsh;
    unsigned* qb;
    int64_t rows, n;
    int d, k, S, aligned;
    unsigned most_passed;
    float* lk;
    int* li;
    hipStream_t stream;
};

template <int W, int QL>
static hipError_t launch_sad(const SadCall& c) {
    const size_t lds = (size_t)kSadPoints * ((W + 3) / 4) * 16 + kSadPoints * 4 +
                       (size_t)4 * (QL * kSadCand * kWave + 2 * kWave + 2 * c.k) * 4;
    hipError_t e = raise_lds_limit(knn_l1_sad_kernel<W, QL>, lds);
    if (e != hipSuccess) return e;
    const int64_t split_len = ((c.n + c.S - 1) / c.S + kSadPoints - 1) / kSadPoints * kSadPoints;
    knn_l1_sad_kernel<W, QL>
        <<<dim3((unsigned)((c.rows + 256 * QL - 1) / (256 * QL)), (unsigned)c.S), dim3(256), lds, c.stream>>>(
            c.Q, c.ldq, c.X, c.ldx, c.qb, c.qr, c.tsh, c.head, (int)c.rows, (int)c.n, c.d, c.k, c.S, (int)split_len,
            c.aligned, c.most_passed, c.lk, c.li);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_sad_words(SadCall c) {
    // The sample: k groups of whole tiles, k * per_group * 64 <= n.  A larger one costs its share of
    // the sums and lets fewer pairs through; a pair let through costs some 500 cycles of a wave, the
    // sums of a pair 2 d / 64: the least total is near this share.
    double share = sqrt(40000.0 * c.k / ((double)c.n * c.d));
    if (share > 1.0 / 3) share = 1.0 / 3;
    int per_group = (int)(share * (double)c.n / kSadPoints / c.k);
    const unsigned gx = (unsigned)((c.rows + 127) / 128);
    // Where the groups are too few to fill the chip a group's tiles are a chain of 0.75 us each, and the
    // pairs that a smaller sample lets through, n / (64 per_group) a query and more for longer lists, are
    // shared by the S ranges' waves at 0.2 us each: the least total of the two.  (1 and 16 queries x 1e5 points, d = 5, k = 1:
    // 758 us and 768 with 441 tiles in one chain, 212 and 226 so, 432 and 544 without the filter.)
    if ((int64_t)gx * c.k < 512) {
        const double lanes = c.rows < 128 ? (double)c.rows : 128.0;
        double chain = sqrt(lanes * (double)c.n * 0.2 * (1.0 + 3.0 * log((double)c.k)) / (64.0 * c.S * 0.75));
        if (chain < 32.0) chain = 32.0;
        if (per_group > chain) per_group = (int)chain;
    }
    if (per_group < 1) per_group = 1;
    knn_l1_seed_kernel<W><<<dim3(gx, (unsigned)c.k), dim3(256), 0, c.stream>>>(
        c.X, c.ldx, c.qb, c.qr, c.tsh, c.head, (int)c.rows, (int)c.n, c.d, c.k, per_group, c.aligned, 0);
    // (the probe takes the first 2^19 queries at most: the pairs that it counts stay below 2^32)
    const int probes = 16;
    const unsigned px = gx < 4096u ? gx : 4096u;
    knn_l1_seed_kernel<W><<<dim3(px, probes), dim3(256), 0, c.stream>>>(
        c.X, c.ldx, c.qb, c.qr, c.tsh, c.head, (int)c.rows, (int)c.n, c.d, c.k, per_group, c.aligned, 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t probed = c.rows < 128 * (int64_t)px ? c.rows : 128 * (int64_t)px;
    c.most_passed = (unsigned)(probed * probes * kSadPoints / kSadPassDivisor);
    // Two queries per lane halve the LDS reads; one where two would leave compute units without work.
    if ((c.rows + 511) / 512 * c.S >= kSadTwoWorkgroups) return launch_sad<W, 2>(c);
    return launch_sad<W, 1>(c);
}

// `room`: the area that knn_l1_kernel keeps its transposed queries in, 16 bytes per row (rounded up
// to 64) and four coordinates.  From 5 coordinates on that holds a byte per coordinate, rounded up
// to 8, two words per row and the header.
hipError_t launch_l1_sad(const float* Q, int64_t ldq, const float* X, int64_t ldx, void* room, int64_t rows, int64_t n,
                         int d, int k, int S, float* lk, int* li, hipStream_t stream) {
    const int words = (d + 7) / 8 * 2;  // four coordinates each, whole pairs
    const int64_t blocks = (rows + kWave - 1) / kWave, rows64 = blocks * kWave;
    SadCall c;
    c.Q = Q;
    c.ldq = ldq;
    c.X = X;
    c.ldx = ldx;
    c.head = static_cast<SadHeader*>(room);
    c.qr = reinterpret_cast<float*>(static_cast<unsigned char*>(room) + kAlign);
    c.tsh = reinterpret_cast<unsigned*>(c.qr + rows64);
    c.qb = c.tsh + rows64;
    c.rows = rows;
    c.n = n;
    c.d = d;
    c.k = k;
    c.S = S;
    c.aligned = reinterpret_cast<uintptr_t>(Q) % 16 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 && ldq % 4 == 0 &&
                ldx % 4 == 0 && d % 4 == 0;
    c.lk = lk;
    c.li = li;
    c.stream = stream;
    knn_l1_scale_kernel<<<dim3(1), dim3(1024), 0, stream>>>(X, ldx, (int)n, d, c.head);
    knn_l1_bytes_kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(Q, ldq, (int)rows, d, words, c.head, c.qb, c.qr,
                                                                         c.tsh);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // (a kernel per pair of words: 1e4 queries, 1e6 points, k = 10, d = 100 22.9 ms with 26 words, d = 112 24.1
    // with 28)
    switch (words) {
        case 2: return launch_sad_words<2>(c);
        case 4: return launch_sad_words<4>(c);
        case 6: return launch_sad_words<6>(c);
        case 8: return launch_sad_words<8>(c);
        case 10: return launch_sad_words<10>(c);
        case 12: return launch_sad_words<12>(c);
        case 14: return launch_sad_words<14>(c);
        case 16: return launch_sad_words<16>(c);
        case 18: return launch_sad_words<18>(c);
        case 20: return launch_sad_words<20>(c);
        case 22: return launch_sad_words<22>(c);
        case 24: return launch_sad_words<24>(c);
        case 26: return launch_sad_words<26>(c);
        case 28: return launch_sad_words<28>(c);
        case 30: return launch_sad_words<30>(c);
        case 32: return launch_sad_words<32>(c);
        case 34: return launch_sad_words<34>(c);
        case 36: return launch_sad_words<36>(c);
        case 38: return launch_sad_words<38>(c);
        case 40: return launch_sad_words<40>(c);
        case 42: return launch_sad_words<42>(c);
        case 44: return launch_sad_words<44>(c);
        case 46: return launch_sad_words<46>(c);
        case 48: return launch_sad_words<48>(c);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace knn
