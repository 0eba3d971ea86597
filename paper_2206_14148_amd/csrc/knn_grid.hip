// gfx950 (CDNA4, MI355X) kNN search among points of up to three dimensions, k <= 32: an octree
// over the points' bounding box instead of every pair (paper section 5.2 defines the result; the
// keys are the fp32 difference-form squared distances of knn_lowd_kernel, compared in the same
// (key, index) order, so the lists are the same whatever was left out).
//
// The points are counted into 2^(D L) cells, L bits per axis, and put in the order of their cells'
// Morton codes.  A node of the tree is a code prefix: its points are one run of that order, and the
// cells' starts are all there is to the tree.  The queries of a wave, 64 that follow each other in
// the same order, descend together: a node is entered if any lane's own query could still find a
// point in it that belongs in its list.
//
// A wave's descent has a budget of steps; the rows of one that exceeds it are left to the filter.
//
// n = m = 1e6, own queries, d = 3, k = 16: 3.25 ms for the search and 0.2 ms for the order, where the
// matrix-core filter spends 42.5 ms on all pairs.  What bounds it is the chain of a wave's steps at three
// waves a SIMD (146 registers): of the wave cycles the vector units are busy in 34 %, 48 % wait for an
// instruction or a load.  A wave of 64 neighbouring queries looks through about a thousand points, an
// eighth of them for the lists.  (Lists of 32 take 256 registers: one wave a SIMD, 13.9 ms at k = 32,
// where the filter takes 52.7.)
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "knn_cells.h"
#include "knn_config.h"
#include "knn_device.h"
#include "knn_kernels.h"

namespace knn {

namespace {

constexpr int kScanCells = 4096;  // cells per workgroup of the scan
constexpr int kGridCand = 8;      // accepted pairs a lane holds before they sink into its list
// (n = m = 1e6, d = 3, k = 16, the search in ms: 24 points 5.36, 48 4.23, 64 4.21, 96 4.21)
constexpr float kGridLeast = 0x1p-100f, kGridMost = 0x1p116f;  // squared lengths that are safe with the filter
constexpr int kLeaf = 48;         // a node of this many points or fewer is looked through, not split

// Morton code of the cell of x: bit b of axis t is bit D b + t
template <int D>
__device__ __forceinline__ int morton_of(const SeedGrid<D>& g, int L, const float (&x)[D]) {
    int code = 0;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        const int c = seed_cell<D>(g, t, x[t]);
        for (int b = 0; b < L; ++b) code |= ((c >> b) & 1) << (D * b + t);
    }
    return code;
}

template <int D>
__device__ __forceinline__ void load_point(const float* __restrict__ P, int64_t ld, int64_t j, float (&x)[D]) {
#pragma unroll
    for (int t = 0; t < D; ++t) x[t] = P[j * ld + t];
}

// One more in counts[code] for every lane with `on`.  Lanes that follow each other may share a cell: while
// the first lane's cell has at least eight of them, they share one atomic; the rest go one by one.
// (With one per lane, where all go to one word each takes 12 ns: 1e5 queries beyond a corner of 1e5
// points, d = 3, k = 16, took 2.52 ms a call and take 0.29, 1e6 of 1e6 23.8 and 1.4.  Uniform ones lose
// nothing: 4.5 ms.)  Returns what the lane's own increment would have found (FETCH), else nothing useful.
template <bool FETCH>
__device__ __forceinline__ int count_up(int* __restrict__ counts, int code, bool on) {
    const int lane = (int)__lane_id();
    uint64_t todo = __builtin_amdgcn_ballot_w64(on);
    int place = 0;
    while (todo) {
        const int lead = __builtin_ctzll(todo);
        const int cell = __builtin_amdgcn_readlane(code, lead);
        const uint64_t same = __builtin_amdgcn_ballot_w64(code == cell) & todo;
        const int many = __builtin_popcountll(same);
        if (many < 8) break;
        int before = 0;
        if (lane == lead) before = atomicAdd(counts + cell, many);
        if (FETCH) {
            before = __builtin_amdgcn_readlane(before, lead);
            if ((same >> lane) & 1) place = before + __builtin_popcountll(same & ((1ull << lane) - 1));
        }
        todo &= ~same;
    }
    if ((todo >> lane) & 1) place = atomicAdd(counts + code, 1);
    return place;
}

// The kernels that count and scan serve the points first, then every chunk of queries; `only_if` is
// null for the points and the word hdr[kGridWord] for the queries, whose counts would otherwise be
// written over what the filter path has packed into the same area.
__global__ __launch_bounds__(256) void knn_grid_clear_kernel(const unsigned* __restrict__ only_if,
                                                             int* __restrict__ counts, int ncell) {
    if (only_if && !*only_if) return;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < ncell; i += gridDim.x * 256) counts[i] = 0;
}

template <int D>
__global__ __launch_bounds__(256) void knn_grid_count_kernel(const float* __restrict__ P, int64_t ld, int n,
                                                             const unsigned* __restrict__ hdr, int L,
                                                             const unsigned* __restrict__ only_if,
                                                             int* __restrict__ counts) {
    if (only_if && !*only_if) return;
    const int j = blockIdx.x * 256 + threadIdx.x;
    const SeedGrid<D> g = seed_grid<D>(hdr, 1 << L);
    float x[D];
    load_point<D>(P, ld, j < n ? j : n - 1, x);
    count_up<false>(counts, morton_of<D>(g, L, x), j < n);
}

// sums[b] = points in the b-th run of kScanCells cells; skew (if given) += sum of the counts' squares
__global__ __launch_bounds__(256) void knn_grid_sum_kernel(const unsigned* __restrict__ only_if,
                                                           const int* __restrict__ counts, int ncell,
                                                           int* __restrict__ sums,
                                                           unsigned long long* __restrict__ skew) {
    if (only_if && !*only_if) return;
    __shared__ int ps[4];
    __shared__ unsigned long long pq[4];
    int s = 0;
    unsigned long long q = 0;
    for (int i = threadIdx.x; i < kScanCells; i += 256) {
        const int c = blockIdx.x * kScanCells + i;
        const int v = c < ncell ? counts[c] : 0;
        s += v;
        q += (unsigned long long)v * (unsigned long long)v;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        s += __shfl_xor(s, o);
        q += __shfl_xor(q, o);
    }
    if ((threadIdx.x & 63) == 0) {
        ps[threadIdx.x >> 6] = s;
        pq[threadIdx.x >> 6] = q;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sums[blockIdx.x] = ps[0] + ps[1] + ps[2] + ps[3];
        if (skew) atomicAdd(skew, pq[0] + pq[1] + pq[2] + pq[3]);
    }
}

// sums -> sums before (one workgroup of 512 threads, at most 512 runs); n > 0: also decides whether
// the tree is worth descending.  A query looks through a few of the finest cells around it, so
// about sum c^2 / n times a handful points; per point that costs some six times what the
// matrix-core filter spends on it, so above n / 128 points per cell met the filter is the better one.
__global__ __launch_bounds__(512) void knn_grid_sums_kernel(const unsigned* __restrict__ only_if,
                                                            int* __restrict__ sums, int runs, int64_t n,
                                                            unsigned* __restrict__ hdr) {
    if (only_if && !*only_if) return;
    __shared__ int v[512];
    const int t = threadIdx.x;
    v[t] = t < runs ? sums[t] : 0;
    __syncthreads();
    for (int o = 1; o < 512; o <<= 1) {
        const int add = t >= o ? v[t - o] : 0;
        __syncthreads();
        v[t] += add;
        __syncthreads();
    }
    if (t < runs) sums[t] = t > 0 ? v[t - 1] : 0;
    if (n > 0 && t == 0) {
        const unsigned long long skew = *reinterpret_cast<const unsigned long long*>(hdr + kGridSkew);
        hdr[kGridWord] = (double)skew * 128.0 <= (double)n * (double)n ? 1u : 0u;
    }
}

// starts[c] (if given) and cursor[c] = points in the cells before c; cursor holds the counts on entry
__global__ __launch_bounds__(256) void knn_grid_scan_kernel(const unsigned* __restrict__ only_if,
                                                            const int* __restrict__ sums, int ncell, int n,
                                                            int* __restrict__ cursor, int* __restrict__ starts) {
    if (only_if && !*only_if) return;
    constexpr int V = kScanCells / 256;
    __shared__ int part[4];
    const int c0 = blockIdx.x * kScanCells + threadIdx.x * V;
    int v[V], own = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        v[i] = c0 + i < ncell ? cursor[c0 + i] : 0;
        own += v[i];
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int run = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(run, o);
        if (lane >= o) run += up;
    }
    if (lane == 63) part[wave] = run;
    __syncthreads();
    run -= own;
    for (int w = 0; w < wave; ++w) run += part[w];
    run += sums[blockIdx.x];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        if (c0 + i < ncell) {
            cursor[c0 + i] = run;
            if (starts) starts[c0 + i] = run;
        }
        run += v[i];
    }
    if (starts && blockIdx.x == 0 && threadIdx.x == 0) starts[ncell] = n;
}

// the points in cell order, (x0, x1, x2, index bits); the order inside a cell is whatever the
// atomics give: nothing that is kept depends on it
template <int D>
__global__ __launch_bounds__(256) void knn_grid_points_kernel(const float* __restrict__ X, int64_t ldx, int n,
                                                              const unsigned* __restrict__ hdr, int L,
                                                              int* __restrict__ cursor,
                                                              f32x4* __restrict__ sorted) {
    if (!hdr[kGridWord]) return;
    const int j = blockIdx.x * 256 + threadIdx.x;
    const SeedGrid<D> g = seed_grid<D>(hdr, 1 << L);
    float x[D];
    load_point<D>(X, ldx, j < n ? j : n - 1, x);
    f32x4 v = {0.f, 0.f, 0.f, __int_as_float(j)};
#pragma unroll
    for (int t = 0; t < D; ++t) v[t] = x[t];
    const int at = count_up<true>(cursor, morton_of<D>(g, L, x), j < n);
    if (j < n) sorted[at] = v;
}

// the queries' numbers in cell order
template <int D>
__global__ __launch_bounds__(256) void knn_grid_queries_kernel(const float* __restrict__ Q, int64_t ldq, int rows,
                                                               const unsigned* __restrict__ hdr, int L,
                                                               int* __restrict__ cursor, int* __restrict__ order) {
    if (!hdr[kGridWord]) return;
    const int r = blockIdx.x * 256 + threadIdx.x;
    const SeedGrid<D> g = seed_grid<D>(hdr, 1 << L);
    float q[D];
    load_point<D>(Q, ldq, r < rows ? r : rows - 1, q);
    const int at = count_up<true>(cursor, morton_of<D>(g, L, q), r < rows);
    if (r < rows) order[at] = r;
}

// (key, index) as the bits of a double: keys are not negative, so such doubles are in the order of
// (key, index), and one v_min_f64 / v_max_f64 moves both.  An empty place is +inf with index 0, an
// ordinary large number in that reading that no pair with an infinite key comes before.
__device__ __forceinline__ double pair_of(float key, int idx) {
    return __hiloint2double((int)__float_as_uint(key), idx);
}

// One query per lane.  The list is K ascending pairs in registers, of which the first K - k are
// below every pair (so that the last is the k-th best whatever k is).
//   1. The list starts from what lies around the query in cell order: 2 K points, whose k-th best
//      pair bounds the result's.  They are not kept (the descent meets them again): the list starts
//      as k copies of the pair just above that bound.
//   2. The descent, depth first, the child on the side of the wave's queries first.  A node's bound
//      for a lane: squared distance from its query to the node's box, the box widened by what the
//      cell numbers' roundings allow (SeedGrid::slack), the bound lowered by what the sums' roundings
//      allow; a node whose bound equals a lane's k-th key is entered (a tie can win by its index).
// A leaf's points are the same for the whole wave and come through scalar loads.
template <int D, int K>
__global__ __launch_bounds__(256) void knn_grid_kernel(const float* __restrict__ Q, int64_t ldq,
                                                       const int* __restrict__ order,
                                                       const f32x4* __restrict__ sorted,
                                                       const int* __restrict__ starts,
                                                       const unsigned* __restrict__ hdr, int L, int rows, int n,
                                                       int k, int S, int groups, int budget,
                                                       unsigned many, unsigned* __restrict__ left, float* __restrict__ lk,
                                                       int* __restrict__ li) {
    constexpr int CH = 1 << D;
    // entries of the stack: CH - 1 left over per level and the node in hand; D L <= 21
    static_assert((CH - 1) * (21 / D) + 1 <= 64, "stack of a wave");
    __shared__ int4 stack[4][64][2];
    __shared__ double cand[4][kGridCand][64];
    if (!hdr[kGridWord]) return;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    // neighbouring groups on one XCD (workgroups go round the eight), for its L2
    const int per = (groups + 7) / 8;
    const int group = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    const int base = (group * 4 + wave) * 64;
    if ((int)(blockIdx.x >> 3) >= per || group >= groups || base >= rows) return;  // (no barrier below)
    const bool active = base + lane < rows;
    const int slot = active ? base + lane : rows - 1;
    const int r = order ? order[slot] : __float_as_int(sorted[slot][3]);
    const SeedGrid<D> g = seed_grid<D>(hdr, 1 << L);
    float q[D];
    load_point<D>(Q, ldq, r, q);
    // (a query that is not finite has no finite key: its list stays empty, as on the other paths)
    bool live = active;
#pragma unroll
    for (int t = 0; t < D; ++t) live &= fabsf(q[t]) < kInf;

    auto sqdist = [&](const f32x4& x) {
        float df = q[0] - x[0];
        float acc = df * df;
#pragma unroll
        for (int t = 1; t < D; ++t) {
            df = q[t] - x[t];
            acc = fmaf(df, df, acc);
        }
        return acc;
    };
    // over the budget: the filter looks at every pair of these rows at less cost
    auto leave = [&]() {
        if (lane == 0) atomicAdd(left, 1u);
        if (active)
            for (int p = 0; p < S; ++p) li[((size_t)r * S + p) * k] = kGridRedo;
    };
    // what of a node's bound is sure in spite of the sums' roundings; nothing where they may overflow
    float sure = 1.f - 0x1p-17f;
    {
        // At more than 2^13 box diagonals from the points what the sums' roundings allow (2^-17 of a key)
        // is a good part of what sets their keys apart: hardly a node would be left out.  (Keys near
        // the largest float or the least normal one stay here: the filter's sums would overflow or lose
        // their pieces.  If even a quarter of the squared distance overflows, so do all keys, and the
        // list stays empty.)
        float b = 0.f, diagonal = 0.f;
#pragma unroll
        for (int t = 0; t < D; ++t) {
            const float range = g.w[t] * (float)g.G;
            const float gap = fmaxf(fmaxf(g.mn[t] - q[t], q[t] - (g.mn[t] + range)), 0.f);
            b = fmaf(0.25f * gap, gap, b);
            diagonal = fmaf(range, range, diagonal);
        }
        live &= !(b == kInf);
        if (!(diagonal > kGridLeast && diagonal < kGridMost) ||
            __builtin_amdgcn_ballot_w64(live && b > kGridMost) != 0) {
            budget = INT_MAX;
            if (!(diagonal < kGridMost) || __builtin_amdgcn_ballot_w64(live && b > kGridMost) != 0) sure = 0.f;
        } else if (__builtin_amdgcn_ballot_w64(live && b > 0x1p24f * diagonal) != 0) {
            leave();
            return;
        }
    }
    // (asked for here, used behind the first pass over the neighbours)
    const unsigned gone = many ? __hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const double top = pair_of(kInf, 0);
    double best[K];
    auto reset = [&](double v) {
#pragma unroll
        for (int i = 0; i < K; ++i) best[i] = (i < K - k || !live) ? -1.0 : v;
    };
    auto insert = [&](double v) {
#pragma unroll
        for (int i = 0; i < K; ++i) {  // v sinks to its place, the last falls out
            const double lo = fmin(best[i], v);
            v = fmax(best[i], v);
            best[i] = lo;
        }
    };
    auto bound_key = [&]() {  // (an idle lane's -1.0 reads as a negative key)
        return __uint_as_float((unsigned)__double2hiint(best[K - 1]));
    };
    reset(top);
    const int own = morton_of<D>(g, L, q);
    {
        // (n >= 4096 > 2 K)
        int p0 = starts[own] - K / 2;
        p0 = p0 < 0 ? 0 : (p0 > n - 2 * K ? n - 2 * K : p0);
        for (int p = 0; p < 2 * K; ++p) {
            const f32x4 x = sorted[p0 + p];
            const float dd = sqdist(x);
            insert(dd < kInf ? pair_of(dd, __float_as_int(x[3])) : top);
        }
        const double b = best[K - 1];
        // the next double up: the least that is not accepted
        const double above = b < top ? __longlong_as_double(__double_as_longlong(b) + 1) : top;
        reset(above);
    }
    if (gone > many && budget != INT_MAX) {
        leave();
        return;
    }
    float tau = bound_key();

    // Accepted pairs wait in LDS until some lane has no room for the next four: the lists then take
    // them side by side, as many rounds as the fullest lane has pairs.  (Sunk in one by one, nearly
    // every point of a leaf cost the wave a round for one or two of its lanes.)
    double* buf = &cand[wave][0][lane];
    int cnt = 0;
    int steps = 0;  // what the wave has done: two per node, one per group of four points, one or two per round
    auto drain = [&]() {
        for (int c = 0; __builtin_amdgcn_ballot_w64(c < cnt) != 0; ++c) {
            insert(c < cnt ? buf[c * 64] : top);
            steps += (K + 8) / 16;
        }
        cnt = 0;
        tau = bound_key();
    };
    // squared distance from the lane's query to a node's box: cell numbers c at the node's level
    auto reach = [&](int level, const int (&c)[3]) {
        float b = 0.f;
#pragma unroll
        for (int t = 0; t < D; ++t) {
            const float lo = (g.mn[t] + (float)(c[t] << (L - level)) * g.w[t]) - g.slack[t];
            const float hi = (g.mn[t] + (float)((c[t] + 1) << (L - level)) * g.w[t]) + g.slack[t];
            const float gap = fmaxf(fmaxf(lo - q[t], q[t] - hi), 0.f);
            b = fmaf(gap, gap, b);
        }
        return !(b * sure > tau);
    };
    int4(*st)[2] = stack[wave];
    if (lane == 0) {
        st[0][0] = int4{0, 0, 0, n};  // level, code, first point, end
        st[0][1] = int4{0, 0, 0, 0};  // cell numbers
    }
    int sp = 1;
    // the child that most of the wave's queries are near: the way to the cell of its middle lane
    const int mid = __builtin_amdgcn_readlane(own, rows - base > 32 ? 32 : 0);
    while (sp > 0 && steps <= budget) {
        --sp;
        steps += 2;
        wave_sync();
        const int4 nd = st[sp][0], nc = st[sp][1];
        const int level = __builtin_amdgcn_readfirstlane(nd.x);
        const int code = __builtin_amdgcn_readfirstlane(nd.y);
        const int s = __builtin_amdgcn_readfirstlane(nd.z);
        const int e = __builtin_amdgcn_readfirstlane(nd.w);
        const int c0[3] = {__builtin_amdgcn_readfirstlane(nc.x), __builtin_amdgcn_readfirstlane(nc.y),
                           __builtin_amdgcn_readfirstlane(nc.z)};
        if (__builtin_amdgcn_ballot_w64(live && reach(level, c0)) == 0) continue;  // (thresholds have moved)
        if (e - s <= kLeaf || level == L) {
            steps += (e - s + 3) >> 2;
            for (int p = s; p < e; p += 4) {
                f32x4 x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = sorted[p + u < e ? p + u : e - 1];
                float dd[4];
                bool any = false;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    dd[u] = p + u < e ? sqdist(x[u]) : __builtin_nanf("");
                    any |= dd[u] <= tau;
                }
                if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (dd[u] <= tau) {
                        buf[cnt * 64] = pair_of(dd[u], __float_as_int(x[u][3]));
                        ++cnt;
                    }
                }
                if (__builtin_amdgcn_ballot_w64(cnt > kGridCand - 4) != 0) drain();
            }
            continue;
        }
        // the ends of the children's runs
        const int shift = D * (L - level - 1);
        const int edge = starts[((code << D) + (lane < CH ? lane : CH)) << shift];
        const int towards = (mid >> shift) & (CH - 1);
        for (int i = CH - 1; i >= 0; --i) {
            const int c = i ^ towards;
            const int cs = __builtin_amdgcn_readlane(edge, c), ce = __builtin_amdgcn_readlane(edge, c + 1);
            if (cs == ce) continue;
            const int cc[3] = {2 * c0[0] + (c & 1), 2 * c0[1] + ((c >> 1) & 1), 2 * c0[2] + ((c >> 2) & 1)};
            if (__builtin_amdgcn_ballot_w64(live && reach(level + 1, cc)) == 0) continue;
            if (lane == 0) {
                st[sp][0] = int4{level + 1, (code << D) | c, cs, ce};
                st[sp][1] = int4{cc[0], cc[1], cc[2], 0};
            }
            ++sp;
        }
    }
    if (sp > 0) {
        leave();
        return;
    }
    drain();
    if (!active) return;
    const size_t lb = (size_t)r * S * k;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int p = i - (K - k);
        if (p >= 0) {
            const float key = live ? __uint_as_float((unsigned)__double2hiint(best[i])) : kInf;
            lk[lb + p] = key;
            li[lb + p] = key < kInf ? __double2loint(best[i]) : kNoIdx;
        }
    }
    // (the lists of further point ranges stay empty)
    for (int p = k; p < S * k; ++p) {
        lk[lb + p] = kInf;
        li[lb + p] = kNoIdx;
    }
}

// bits per axis: the most cells that are still worth their memory, at most 2.5 per point
int levels_of(int64_t n, int d) {
    int L = 1;
    while (d * (L + 1) <= 21 && ((int64_t)1 << (d * (L + 1))) <= kGridMaxCells &&
           2 * ((int64_t)1 << (d * (L + 1))) <= 5 * n)
        ++L;
    return L;
}

// the area of 32 n bytes: [cell starts][cursors][run sums]
struct Cells {
    int L, ncell, runs;
    int *starts, *cursor, *sums;
};
Cells cells_of(int64_t n, int d, void* area) {
    Cells c;
    c.L = levels_of(n, d);
    c.ncell = 1 << (d * c.L);
    c.runs = (c.ncell + kScanCells - 1) / kScanCells;
    unsigned char* p = static_cast<unsigned char*>(area);
    c.starts = reinterpret_cast<int*>(p);
    p += align_up(((uint64_t)c.ncell + 1) * 4);
    c.cursor = reinterpret_cast<int*>(p);
    p += align_up((uint64_t)c.ncell * 4);
    c.sums = reinterpret_cast<int*>(p);  // (at most 512: 20 n + 2560 bytes in all)
    return c;
}

template <int D>
hipError_t count_and_scan(const float* P, int64_t ld, int64_t count, const Cells& c, unsigned* hdr, bool points,
                          hipStream_t stream) {
    const unsigned clear = (unsigned)((c.ncell + 1023) / 1024);
    const unsigned* only_if = points ? nullptr : hdr + kGridWord;
    knn_grid_clear_kernel<<<dim3(clear), dim3(256), 0, stream>>>(only_if, c.cursor, c.ncell);
    knn_grid_count_kernel<D><<<dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream>>>(
        P, ld, (int)count, hdr, c.L, only_if, c.cursor);
    knn_grid_sum_kernel<<<dim3((unsigned)c.runs), dim3(256), 0, stream>>>(
        only_if, c.cursor, c.ncell, c.sums,
        points ? reinterpret_cast<unsigned long long*>(hdr + kGridSkew) : nullptr);
    knn_grid_sums_kernel<<<dim3(1), dim3(512), 0, stream>>>(only_if, c.sums, c.runs, points ? count : 0, hdr);
    knn_grid_scan_kernel<<<dim3((unsigned)c.runs), dim3(256), 0, stream>>>(
        only_if, c.sums, c.ncell, (int)count, c.cursor, points ? c.starts : nullptr);
    return hipGetLastError();
}

template <int D>
hipError_t build_d(const float* X, int64_t ldx, int64_t n, unsigned* hdr, void* area, void* sorted,
                   hipStream_t stream) {
    const Cells c = cells_of(n, D, area);
    hipError_t e = count_and_scan<D>(X, ldx, n, c, hdr, true, stream);
    if (e != hipSuccess) return e;
    knn_grid_points_kernel<D><<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(
        X, ldx, (int)n, hdr, c.L, c.cursor, static_cast<f32x4*>(sorted));
    return hipGetLastError();
}

template <int D>
hipError_t search_d(const float* Q, int64_t ldq, const float* X, int64_t ldx, int64_t rows, int64_t n, int k,
                    int S, unsigned* hdr, void* area, const void* sorted, int* order, float* lk, int* li,
                    hipStream_t stream) {
    const Cells c = cells_of(n, D, area);
    const bool same = Q == X && ldq == ldx && rows == n;  // the points' order serves the queries
    if (!same) {
        hipError_t e = count_and_scan<D>(Q, ldq, rows, c, hdr, false, stream);
        if (e != hipSuccess) return e;
        knn_grid_queries_kernel<D><<<dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, stream>>>(
            Q, ldq, (int)rows, hdr, c.L, c.cursor, order);
    }
    const int groups = (int)((rows + 255) / 256);
    // Where queries and points lie alike no wave took more steps than 15, 23 and 45 sqrt(n) (lists of 8, 16
    // and 32 in registers; n from 4096 to 1e6, uniform, normal, clumps, a shell; the worst waves are those
    // whose queries follow each other across a gap of the order).  A step takes 0.2 to 0.35 us.
    const int budget = (int)((6.0 + 1.5 * (k <= 8 ? 8 : (k <= 16 ? 16 : 32))) * sqrt((double)n));
    // in a launch of several rounds the later waves leave at once if many have done so
    const int64_t waves = (rows + 63) / 64;
    const unsigned many = waves > 4 * 4 * kNumCU ? (unsigned)(waves / 16) : 0u;
    const dim3 grid((unsigned)((groups + 7) / 8 * 8));
    auto go = [&](auto kernel) {
        kernel<<<grid, dim3(256), 0, stream>>>(Q, ldq, same ? nullptr : order, static_cast<const f32x4*>(sorted),
                                               c.starts, hdr, c.L, (int)rows, (int)n, k, S, groups, budget, many, hdr + kGridLeft, lk, li);
    };
    if (k <= 8) go(knn_grid_kernel<D, 8>);
    else if (k <= 16) go(knn_grid_kernel<D, 16>);
    else go(knn_grid_kernel<D, 32>);
    return hipGetLastError();
}

__global__ void knn_grid_again_kernel(unsigned* __restrict__ hdr) {
    if (!hdr[kGridWord] || hdr[kGridLeft]) {
        hdr[kGridWord] = 0u;
        hdr[kGridPacked] = 1u;
    }
    hdr[kGridLeft] = 0u;
}

}  // namespace

// The queries of a wave descend together, so they have to lie close to each other; and a wave's descent is
// one long chain, while the filter cuts its work over the whole chip whatever the sizes.  The lines are
// drawn where the octree was not slower, uniform and normal points (us, filter / octree):
//   own queries or more queries than points   d 2, n 1e4, k 16 445 / 256    d 2, n 28000, k 32 966 / 1174
//     (d 3) n 1e4, k 8 462 / 333, k 16 485 / 508, k 32 717 / 912    n 28000, k 16 755 / 877    n 40000, k 16
//     954 / 897, k 32 1182 / 1641    n 56000, k 32 2112 / 1679    m 2e4, n 1e4, k 32 791 / 908
//   others, m = n   d 2: n 32768, k 4 339 / 190, k 8 457 / 463, k 16 637 / 685    n 65536, k 32 1903 / 987
//     (d 3) n 16384, k 1 164 / 207, k 4 358 / 234, k 16 478 / 526    n 65536, k 16 1051 / 1137    131072 2358 / 916
//   m = n / 2   d 3: n 65536, k 1 337 / 265, k 16 830 / 992    131072, k 16 1512 / 1459, k 32 1982 / 2486
//   m = n / 8   d 2: n 65536, k 1 208 / 207    4e5, k 16 1785 / 1403, k 32 2508 / 2539    1e6, k 32 7562 / 5665
//     (d 3) n 131072, k 1 348 / 367, k 32 1222 / 2248    4e5, k 16 2198 / 1299    1e6, k 32 8497 / 5179
//   d 1: n 32768, m 4096, k 16 396 / 345, k 32 547 / 589    everything else is far on the octree's side
bool grid_applies(int64_t rows, int64_t n, int d, int k, bool own) {
    if (n < kGridMinPoints || k > kGridMaxK || rows < n / 8) return false;
    if (d == 1) return k <= 16 || 4 * rows >= n || n >= 65536;
    if (rows >= 2 * n) return d == 2 || k <= 16 || rows >= 8 * n || n <= 8192 || n >= 20000;
    if (own) {
        if (k <= 8) return true;
        if (d == 2) return k <= 16 || n <= 20000 || n >= 64000;
        return n <= 8192 || n >= (k <= 16 ? 32000 : 50000);
    }
    if (4 * rows >= 3 * n) {
        if (d == 3 && k <= 8) return k >= 4 || n <= 6000 || n >= 20000;
        return k <= 4 || n <= 8192 || n >= (d == 2 ? 64000 : 100000);
    }
    if (n <= 6000 && 2 * rows >= n) return true;
    const double pairs = (double)rows * (double)n;
    if (k <= 4) return pairs >= (d == 2 ? 1e9 : 3e9);
    if (k <= 16) return pairs >= 8e9;
    return pairs >= 1.5e10 && (d == 3 || 4 * rows >= n || pairs >= 1e11);
}

hipError_t launch_grid_build(const float* X, int64_t ldx, int64_t n, int d, unsigned* hdr, void* cells,
                             void* sorted, hipStream_t stream) {
    switch (d) {
        case 1: return build_d<1>(X, ldx, n, hdr, cells, sorted, stream);
        case 2: return build_d<2>(X, ldx, n, hdr, cells, sorted, stream);
        case 3: return build_d<3>(X, ldx, n, hdr, cells, sorted, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_grid_again(unsigned* hdr, hipStream_t stream) {
    knn_grid_again_kernel<<<dim3(1), dim3(1), 0, stream>>>(hdr);
    return hipGetLastError();
}

hipError_t launch_grid_search(const float* Q, int64_t ldq, const float* X, int64_t ldx, int64_t rows,
                              int64_t n, int d, int k, int S, unsigned* hdr, void* cells, const void* sorted,
                              int* order, float* lk, int* li, hipStream_t stream) {
    switch (d) {
        case 1: return search_d<1>(Q, ldq, X, ldx, rows, n, k, S, hdr, cells, sorted, order, lk, li, stream);
        case 2: return search_d<2>(Q, ldq, X, ldx, rows, n, k, S, hdr, cells, sorted, order, lk, li, stream);
        case 3: return search_d<3>(Q, ldq, X, ldx, rows, n, k, S, hdr, cells, sorted, order, lk, li, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace knn
