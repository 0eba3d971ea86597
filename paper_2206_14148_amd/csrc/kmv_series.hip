// gfx950 (CDNA4, MI355X) kernels for y = K v on a line (d = 1): the sources z_j are grouped into
// boxes a fraction of a lengthscale wide and act through one short series per box, so the work
// goes with n + m and not with n m.  The general kernels (kmv_kernels.hip) make every entry of K.
//
// With a = (x - c) / l and b = (z - c) / l for a box of centre c,
//     exp(-(x - z)^2 / (2 l^2)) = exp(-a^2 / 2) * exp(a b) * exp(-b^2 / 2)
//     sum_j v_j K(x, z_j)       = exp(-a^2 / 2) * sum_p a^p * [ sum_j v_j exp(-b_j^2 / 2) b_j^p / p! ],
// and the bracket, the box's moment p, does not depend on x.  |b| <= h, half a box's width in
// lengthscales.  Cutting the series of exp(a b) after P terms leaves at most (|a| h)^P / P! beside
// exp(-|a| h):
//     fp32 entry: h = 1/2, P = 34: relative to the entry itself below 2e-8 for |a| <= 13.2, where the
//                 entry is the smallest normal number, 3e-6 for |a| <= 14.9, and below 1e-16 for |a| <= 8
//     fp64 entry: h = 1/4, P = 56: below 1e-15 for |a| <= 38.9
// (beyond that |a| every entry of the box is zero in the entry point's own precision).
//
// Rounding: where a and b have opposite signs the series alternates, and what it loses beside the
// entry grows as 2^-53 exp(2 |a| h).  That is 3e-10 at most for the fp32 entry point, far below its own
// 1e-7.  For the fp64 one it is 55 roundings at |a| = 8 and 1e8 at 38, so a row is answered
// here only if what boxes beyond 8 may lose is nothing beside the entries of its nearer ones: in
// bounds that hold for every source of a box,
//     sum over boxes with |a| > 8 of exp(-a^2/2 + |a| h) W  <=  2.5 sum over boxes of exp(-a^2/2 - |a| h) W,
// W the box's sum of |v_j| exp(-b_j^2 / 2).  A tile of rows with one that is not (a row far outside
// the sources; weights that are zero but for some far away) goes to the general kernel, row for
// row as without the series.
//
// Boxes of half the width with P = 22 and 36 were 25 % slower: a box costs a row its P multiply-adds
// and an exponential, about as much again.
// Everything is computed in fp64, for the fp32 entry point too, whose own entries and 64-term sums
// carry 1e-7.  Every sum has a fixed order.
//
// What bounds it: a wave's chain of boxes (the table's row, then P multiply-adds that wait for each
// other), and for many sources the look of every box's workgroups at all of them.  n = m = 1e6 in fp32,
// l = 1, normal points (10 boxes): bounds 5.6 us, moments 26, table 4.7, rows 32, against 160 ms
// for the entries one by one; 2e5 x 2e5 in fp64: 4.8, 30, 5.8, 39 us against 35.4 ms.  Error against
// 64 bits 7e-16 (fp32 entry by entry: 2.6e-7; fp64: 5e-15).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "kmv_kernels.h"
#include "knn_config.h"
#include "knn_device.h"

namespace kmv {

namespace {

template <typename T>
struct Series;
template <>
struct Series<float> {
    static constexpr int P = 34;
    static constexpr double h = 0.5;
    // a^2 / 2 above which every entry of a box is zero: (sqrt(2 x 104) + h)^2 / 2, an entry being zero in fp32,
    // denormals included, below exp(-104)
    static constexpr double far = 111.5;
    // what the four kernels take, us: all, per source, per box, per box and source, per box and row
    static constexpr double base_us = 28.0, source_us = 3e-5, box_us = 1.4, box_source_us = 2.3e-6, box_row_us = 3.6e-6;
};
template <>
struct Series<double> {
    static constexpr int P = 56;
    static constexpr double h = 0.25;
    static constexpr double far = 756.0;  // (from exp(-745.2))
    static constexpr double base_us = 28.0, source_us = 4e-5, box_us = 2.6, box_source_us = 4e-6, box_row_us = 3e-6;
};

constexpr int kRow = 64;          // doubles per box: P moments, W, and in the table the centre at kRow - 1
constexpr int kWeight = kRow - 2;  // in the table: log2 W as a float
constexpr double kNear = 8.0;      // |a| up to which the series loses next to nothing
constexpr int64_t kManyRows = 1 << 15;  // from here on two rows per lane
constexpr int kBoundsGroups = 256;
constexpr int kMaxBoxes = 1024;
constexpr int kMomentGroups = 2048;  // workgroups of the moment kernel: box x slice of the sources
constexpr int kMaxSlices = 128;

// workspace: header | bounds of the workgroups [3][256] | the boxes' table | partial moments | how many tiles
// of 256 rows are left to the general kernel (-1: all), and for each (fp64) whether it is done
struct Header {
    int ok;      // the series applies
    int boxes;
    int slices;
};
constexpr int64_t kBoundsAt = 256;
constexpr int64_t kTableAt = kBoundsAt + 3 * kBoundsGroups * 8;
constexpr int64_t kPartialAt = kTableAt + (int64_t)kMaxBoxes * kRow * 8;
constexpr int64_t kDoneAt = kPartialAt + (int64_t)kMomentGroups * kRow * 8;
static_assert(kBoundsAt % 256 == 0 && kTableAt % 256 == 0 && kPartialAt % 256 == 0, "aligned pieces");

// lowest and highest source, and whether all sources and weights are finite and not too large
template <typename T>
__global__ __launch_bounds__(256) void kmv_bounds_kernel(const T* __restrict__ Z, int64_t ldz,
                                                         const T* __restrict__ v, int64_t m,
                                                         double* __restrict__ bounds) {
    __shared__ double part[3][4];
    double lo = HUGE_VAL, hi = -HUGE_VAL, bad = 0.0;
    const double most = 1e300 / (double)m;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < m; j += 256 * kBoundsGroups) {
        const double z = (double)Z[j * ldz], w = (double)v[j];
        lo = fmin(lo, z);
        hi = fmax(hi, z);
        // (weights whose sum without the entries of K could overflow are left to the general kernel)
        if (!(fabs(z) < HUGE_VAL) || !(fabs(w) < most)) bad = 1.0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o));
        hi = fmax(hi, __shfl_xor(hi, o));
        bad = fmax(bad, __shfl_xor(bad, o));
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        part[0][wave] = lo;
        part[1][wave] = hi;
        part[2][wave] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        bounds[blockIdx.x] = fmin(fmin(part[0][0], part[0][1]), fmin(part[0][2], part[0][3]));
        bounds[kBoundsGroups + blockIdx.x] = fmax(fmax(part[1][0], part[1][1]), fmax(part[1][2], part[1][3]));
        bounds[2 * kBoundsGroups + blockIdx.x] = part[2][0] + part[2][1] + part[2][2] + part[2][3];
    }
}

// Sums over the wave of N values a lane: with every step a lane hands half of its values to the lane S away and
// keeps the others, so about N exchanges make all sums (a butterfly per value would take 6 N).  Afterwards a
// lane holds, in a[0], the sum of value number wave_sums_place(lane).  A fixed tree.
template <int S, int N>
__device__ __forceinline__ void wave_sums(double (&a)[N], int lane) {
    constexpr int H = (N + 1) / 2;
    double half[H];
    const bool upper = lane & S;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double even = a[2 * i], odd = 2 * i + 1 < N ? a[2 * i + 1 < N ? 2 * i + 1 : 0] : 0.0;
        const double give = upper ? even : odd;
        const int lo = knn::lane_xor<S>(__double2loint(give)), hi = knn::lane_xor<S>(__double2hiint(give));
        half[i] = (upper ? odd : even) + __hiloint2double(hi, lo);
    }
    if constexpr (S > 1) wave_sums<S / 2, H>(half, lane);
    a[0] = half[0];
}
__device__ __forceinline__ int wave_sums_place(int lane) { return (int)(__brev((unsigned)lane) >> 26); }

// Workgroup (box, slice): the moments of the box's sources among one slice of them.  A wave puts
// the box's sources among those it looks at into a queue in LDS, in ascending order, and takes 64 at a
// time from it, so that all lanes have a source to raise to its powers (without the queue, every wave
// did so for its few lanes inside the box: 44 us at n = m = 1e6 in fp32, 26 with it; 2e5 in fp64 60 and 30).  Lanes and waves are added in
// a fixed tree.
template <typename T>
__global__ __launch_bounds__(256) void kmv_moments_kernel(const T* __restrict__ Z, int64_t ldz,
                                                          const T* __restrict__ v, int64_t m, int64_t n,
                                                          double lengthscale, double general_us,
                                                          const double* __restrict__ bounds,
                                                          Header* __restrict__ header,
                                                          double* __restrict__ table,
                                                          double* __restrict__ partial, int* __restrict__ done) {
    constexpr int P = Series<T>::P;
    constexpr int N = P + (sizeof(T) == 8 ? 1 : 0);  // sums: the moments, and in fp64 their terms' magnitude
    __shared__ double sum[4][N];
    __shared__ double part[3][4];
    __shared__ double queue_b[4][128], queue_v[4][128];  // a ring per wave
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    // every workgroup puts the bounds together for itself
    double lo = bounds[threadIdx.x], hi = bounds[kBoundsGroups + threadIdx.x],
           bad = bounds[2 * kBoundsGroups + threadIdx.x];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o));
        hi = fmax(hi, __shfl_xor(hi, o));
        bad = fmax(bad, __shfl_xor(bad, o));
    }
    if (lane == 0) {
        part[0][wave] = lo;
        part[1][wave] = hi;
        part[2][wave] = bad;
    }
    __syncthreads();
    lo = fmin(fmin(part[0][0], part[0][1]), fmin(part[0][2], part[0][3]));
    hi = fmax(fmax(part[1][0], part[1][1]), fmax(part[1][2], part[1][3]));
    bad = part[2][0] + part[2][1] + part[2][2] + part[2][3];
    const double rl = 1.0 / lengthscale;
    const double width = 2.0 * Series<T>::h * lengthscale;
    const double rw = 1.0 / width;
    const double span = (hi - lo) * rw;
    // The general kernel takes over where a source or weight is not finite (its sums then say
    // so), where the boxes would be too many or hold fewer than 16 sources each, where the coordinates'
    // own spacing is no longer small beside a box (a centre could then not lie in the middle), or
    // where it takes less time.  Measured, us, m from 300 to 1e7, n from 40 to 1e6, 1 to 1000 boxes: a box costs
    // a row's wave its chain whatever the sizes are, its own workgroups a look at all sources, and every
    // row its terms.  (In fp32: n = m = 2e4, 10 boxes 41, 60 120, 300 443, the general kernel 90;
    // n = 300, m = 1e6 82, 266, 875 against 258; n = 1e6, m = 1000 59, 241, - against 157.)
    const double series_us = Series<T>::base_us + Series<T>::source_us * (double)m +
                             (span + 1.0) * (Series<T>::box_us + Series<T>::box_source_us * (double)m +
                                             Series<T>::box_row_us * (double)n);
    const bool ok = bad == 0.0 && span < (double)kMaxBoxes - 1.0 && (span + 1.0) * 16.0 <= (double)m &&
                    fmax(fabs(lo), fabs(hi)) * 0x1p-52 <= width * 0x1p-7 && series_us <= general_us;
    const int boxes = ok ? (int)span + 1 : 0;
    int slices = 1;
    if (ok) {
        slices = kMomentGroups / boxes;
        if (slices > kMaxSlices) slices = kMaxSlices;
        const int64_t useful = (m + 1023) / 1024;
        if (slices > useful) slices = (int)useful;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *header = Header{ok ? 1 : 0, boxes, slices};
        done[0] = ok ? 0 : -1;
    }
    const int box = (int)blockIdx.x / slices;
    const int slice = (int)blockIdx.x - box * slices;
    if (box >= boxes) return;  // whole workgroup
    const double c = fma((double)box + 0.5, width, lo);
    double acc[N];
#pragma unroll
    for (int p = 0; p < N; ++p) acc[p] = 0.0;
    const int64_t len = (m + slices - 1) / slices;
    const int64_t j0 = slice * len;
    const int64_t j1 = j0 + len < m ? j0 + len : m;
    auto take = [&](double b, double v) {
        double w = v * exp(-0.5 * b * b);
        if constexpr (N > P) acc[P] += fabs(w);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            acc[p] += w;
            w *= b;
        }
    };
    constexpr int U = 8;
    int head = 0, count = 0;  // (the same in all lanes)
    for (int64_t jw = j0 + wave * 64; jw < j1; jw += 256 * U) {
        T z[U], v_[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t jj = jw + lane + 256 * u;
            const int64_t jc = jj < j1 ? jj : j1 - 1;
            z[u] = Z[jc * ldz];
            v_[u] = v[jc];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int g = (int)(((double)z[u] - lo) * rw);
            if (g > boxes - 1) g = boxes - 1;
            const bool mine = g == box && jw + lane + 256 * u < j1;
            const uint64_t in = __builtin_amdgcn_ballot_w64(mine);
            if (in == 0) continue;
            if (mine) {
                const int at = (head + count + __builtin_popcountll(in & ((1ull << lane) - 1))) & 127;
                queue_b[wave][at] = ((double)z[u] - c) * rl;
                queue_v[wave][at] = (double)v_[u];
            }
            count += __builtin_popcountll(in);
            if (count >= 64) {
                knn::wave_sync();
                const int at = (head + lane) & 127;
                take(queue_b[wave][at], queue_v[wave][at]);
                head = (head + 64) & 127;
                count -= 64;
                knn::wave_sync();  // (read before it is written again)
            }
        }
    }
    knn::wave_sync();
    if (lane < count) take(queue_b[wave][(head + lane) & 127], queue_v[wave][(head + lane) & 127]);
    static_assert(N <= 64, "a lane per sum");
    wave_sums<32, N>(acc, lane);
    if (wave_sums_place(lane) < N) sum[wave][wave_sums_place(lane)] = acc[0];
    __syncthreads();
    const int t = threadIdx.x;
    if (t < N) partial[(int64_t)blockIdx.x * kRow + t] = (sum[0][t] + sum[1][t]) + (sum[2][t] + sum[3][t]);
    if (slice == 0 && t == kRow - 1) table[(int64_t)box * kRow + kRow - 1] = c;
}

// table[box][p] = (sum over the slices, a wave every fourth, then the waves) / p!; at kWeight log2 of the magnitudes' sum
template <typename T>
__global__ __launch_bounds__(256) void kmv_table_kernel(const Header* __restrict__ header,
                                                        const double* __restrict__ partial,
                                                        double* __restrict__ table) {
    constexpr int P = Series<T>::P;
    static_assert(P < kWeight, "a lane per moment and one for their magnitude, the centre behind them");
    __shared__ double sum[4][64];
    const int box = blockIdx.x, p = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (!header->ok || box >= header->boxes) return;  // whole workgroup
    const bool have = p < P || (p == P && sizeof(T) == 8);
    const int slices = header->slices;
    double s = 0.0;
    if (have) {
#pragma unroll 8
        for (int i = wave; i < slices; i += 4) s += partial[((int64_t)box * slices + i) * kRow + p];
    }
    sum[wave][p] = s;
    __syncthreads();
    if (wave != 0 || !have) return;
    s = (sum[0][p] + sum[1][p]) + (sum[2][p] + sum[3][p]);
    if (p == P) {
        *reinterpret_cast<float*>(table + (int64_t)box * kRow + kWeight) = (float)log2(s);
        return;
    }
    double factorial = 1.0;
    for (int i = 2; i <= p; ++i) factorial *= (double)i;
    table[(int64_t)box * kRow + p] = s / factorial;
}

// R rows per lane, one of each of R tiles of 256; the boxes are the same for the whole wave, so their moments come
// through scalar loads, whose round trips bound the kernel: R rows share them and have chains of their own.
// (n = 1e6 in fp32: the call 84 us with one row, 66 with two, 67 with four; n = 2e5 in fp64 85, 79, 93; n = 5e4 69, 65.)
// Per box and row: P multiply-adds and one exponential.  In fp64 done[1 + tile] = 1 where y
// is complete, 0 where the general kernel has to make the tile's rows; done[0] counts those.
template <typename T, int R>
__global__ __launch_bounds__(256) void kmv_series_kernel(const T* __restrict__ X, int64_t ldx, int64_t n,
                                                         double lengthscale, double variance,
                                                         const Header* __restrict__ header,
                                                         const double* __restrict__ table,
                                                         int* __restrict__ done, double* __restrict__ y) {
    constexpr int P = Series<T>::P;
    if (!header->ok) return;
    const int boxes = header->boxes;
    const double rl = 1.0 / lengthscale;
    double x[R], total[R];
    float surely[R], lost[R];  // log2: the largest terms of the two sums above
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = ((int64_t)blockIdx.x * R + r) * 256 + threadIdx.x;
        x[r] = (double)X[(i < n ? i : n - 1) * ldx];
        total[r] = 0.0;
        surely[r] = lost[r] = -HUGE_VALF;
    }
    for (int box = 0; box < boxes; ++box) {
        const double* __restrict__ row = table + (int64_t)box * kRow;
        double a[R], s[R];
        bool near = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            a[r] = (x[r] - row[kRow - 1]) * rl;
            near |= 0.5 * a[r] * a[r] <= Series<T>::far;
        }
        if (__builtin_amdgcn_ballot_w64(near) == 0) continue;
        if constexpr (sizeof(T) == 8) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!(0.5 * a[r] * a[r] <= Series<T>::far)) continue;
                constexpr float kLog2e = 1.44269504f;
                const float fa = fabsf((float)a[r]);
                const float w = *reinterpret_cast<const float*>(row + kWeight) - 0.5f * kLog2e * fa * fa;
                const float spread = (float)Series<T>::h * kLog2e * fa;
                surely[r] = fmaxf(surely[r], w - spread);
                if (fa > (float)kNear) lost[r] = fmaxf(lost[r], w + spread);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) s[r] = row[P - 1];
#pragma unroll
        for (int p = P - 2; p >= 0; --p) {
#pragma unroll
            for (int r = 0; r < R; ++r) s[r] = fma(s[r], a[r], row[p]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double e = 0.5 * a[r] * a[r];
            if (e <= Series<T>::far) total[r] = fma(exp(-e), s[r], total[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t tile = (int64_t)blockIdx.x * R + r, i = tile * 256 + threadIdx.x;
        if (x[r] != x[r]) total[r] = x[r];  // as the sum over such entries of K
        if (i < n) y[i] = variance * total[r];
        if constexpr (sizeof(T) == 8) {
            if (tile * 256 >= n) break;  // (whole workgroup)
            // (at most 160 boxes are within reach of a row: 160 / 2^6 = 2.5)
            const int leave = __syncthreads_or(i < n && lost[r] > surely[r] - 6.f);
            if (threadIdx.x == 0) {
                done[1 + tile] = leave ? 0 : 1;
                if (leave) atomicAdd(done, 1);
            }
        }
    }
}

}  // namespace

int64_t series_bytes(int64_t n) { return kDoneAt + 4 + (n + 255) / 256 * 4; }

// What the general kernels take at least, us: all entries at 6.4e12 (fp64 1.3e12) per second, or one
// wave's range of the sources at 16 ns (90) each, where rows and ranges leave the chip idle.
static double general_time_us(int64_t n, int64_t m, int S, bool f64) {
    const double entries = (double)n * (double)m / (f64 ? 1.3e6 : 6.4e6);
    const double range = (double)m / S * (f64 ? 0.09 : 0.016);
    return entries > range ? entries : range;
}

bool series_applies(int64_t n, int64_t m, int S, int d, double lengthscale, bool f64) {
    // The launches here take about 30 us.  Where the device then finds that the points do not allow the
    // series, four of them and a look at the sources have been in vain: 12 us, 90 -> 102 at n = m = 2e4 in
    // fp32, and with 4e6 sources 120 us, 1655 -> 1777.  So calls that cannot gain much are left alone.
    if (d != 1 || general_time_us(n, m, S, f64) < 60.0) return false;
    // (the general kernels form 1 / (2 l^2): where that or its inverse leaves the range of the type
    // they decide what comes out)
    return f64 ? (lengthscale >= 1e-100 && lengthscale <= 1e100)
               : (lengthscale >= 1e-15 && lengthscale <= 1e15);
}

template <typename T>
hipError_t launch_series(const T* X, int64_t ldx, const T* Z, int64_t ldz, const T* v, int64_t n, int64_t m,
                         int S, double lengthscale, double variance, void* ws, double* y, hipStream_t stream,
                         const int** done) {
    unsigned char* base = static_cast<unsigned char*>(ws);
    Header* header = reinterpret_cast<Header*>(base);
    double* bounds = reinterpret_cast<double*>(base + kBoundsAt);
    double* table = reinterpret_cast<double*>(base + kTableAt);
    double* partial = reinterpret_cast<double*>(base + kPartialAt);
    static_assert(kLowdTileRows == 256, "a flag per workgroup of the general kernels");
    int* const flags = reinterpret_cast<int*>(base + kDoneAt);
    *done = flags;
    kmv_bounds_kernel<T><<<dim3(kBoundsGroups), dim3(256), 0, stream>>>(Z, ldz, v, m, bounds);
    kmv_moments_kernel<T><<<dim3(kMomentGroups), dim3(256), 0, stream>>>(
        Z, ldz, v, m, n, lengthscale, general_time_us(n, m, S, sizeof(T) == 8), bounds, header, table, partial, flags);
    kmv_table_kernel<T><<<dim3(kMaxBoxes), dim3(256), 0, stream>>>(header, partial, table);
    // (as many rows per lane as leave enough waves for every SIMD)
    auto rows = [&](auto kernel, int64_t per_lane) {
        kernel<<<dim3((unsigned)((n + 256 * per_lane - 1) / (256 * per_lane))), dim3(256), 0, stream>>>(
            X, ldx, n, lengthscale, variance, header, table, flags, y);
    };
    if (n >= kManyRows) rows(kmv_series_kernel<T, 2>, 2);
    else rows(kmv_series_kernel<T, 1>, 1);
    return hipGetLastError();
}

template hipError_t launch_series<float>(const float*, int64_t, const float*, int64_t, const float*, int64_t,
                                         int64_t, int, double, double, void*, double*, hipStream_t, const int**);
template hipError_t launch_series<double>(const double*, int64_t, const double*, int64_t, const double*,
                                          int64_t, int64_t, int, double, double, void*, double*, hipStream_t,
                                          const int**);

}  // namespace kmv
