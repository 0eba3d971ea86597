// gfx950 (CDNA4, MI355X) kernels for y = K v (paper section 5.1) with 9 to 64 coordinates where the
// workspace has room for the points as 16-bit pieces: the squared distance through its expansion (section
// 4.1) on the matrix cores, the exponentials on the vector ALU beside them.
//
// K_ij = variance exp2(a_i . b_j - |a_i|^2 / 2 - |b_j|^2 / 2), a and b the rows of X and Z times sqrt(2 c2).  In
// these units a value as two fp16 pieces, hi + lo, is off by 2^-23 of itself or 2^-25, whichever is larger;
// the norms are those of the pieces (hi + lo)^2, so the exponent is that of two slightly moved points and not
// a difference of numbers that were rounded apart.  Four products of pieces (lo lo, lo hi, hi lo, hi hi) stand for
// the six that three bf16 pieces need.  The first is left out, per tile and wave, where the low pieces of every
// point and row are below 2^-22 in the sum of their squares: then it moves an entry by less than 2^-22, and
// points as close to the origin as that (some two lengthscales) have no pair so far apart that an entry of a
// point with itself, where it is a loss and not a rounding, would be the whole of a sum.  Error against 64
// bits in parts of the six-product kernel's (2000 x 2000, d = 9 .. 64, lengthscales 0.05 to 5 sqrt(d), means 0 to 100, clusters,
// weights of one sign or both): 0.4 to 1.0 in the mean of each kind of data, at most 1.07 but for a fifth of the points a
// thousand times as far out as the others (1.33).  Left out everywhere, and out of the norms: up to 2.2 off the origin.
// The norms are summed in fp64 and added last, as three exact bf16 pieces each times one, by one more matrix
// instruction, which costs no vector instruction and adds the largest numbers once.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "kmv_kernels.h"
#include "knn_config.h"
#include "knn_device.h"

namespace kmv {

namespace {

using knn::f32x16;
using knn::f32x4;
using knn::load_row4;
using knn::load_to_lds;
using knn::mask_row4;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kFragment = 1024;       // bytes: 32 points x 16 coordinates of one piece, in operand order
constexpr float kMostHalf = 32768.f;  // coordinates beyond this are scaled down
constexpr float kMostScaled = 0x1p60f;  // and beyond this are infinite: products of scaled ones back in fp32's range
constexpr float kFar = -1e30f;        // exponent of what pads the last tile
constexpr float kSmallLow = 0x1p-22f;  // |low pieces|^2 of a point up to which their products are left out

// of a tile's points, and of a wave's rows: |low|^2 <= kSmallLow for all, all in the pieces' range, neither
enum Kind { kTileSmallLows, kTileFits, kTileOutOfRange };

// Points of a tile: two of its records in LDS leave room for four workgroups per compute unit, as the registers do up to
// 48 coordinates (beyond, for three).
template <int NCH>
constexpr int kTilePoints = NCH <= 2 ? 128 : 64;

// A tile's record: [chunk of 16 coordinates][piece][block of 32 points] fragments, then per block 32 x 16
// bytes for the norms' instruction (its last word not used there: the factor 2^shift of the point), then the points'
// weights and the tile's kind.
template <int NCH>
struct Record {
    static constexpr int blocks = kTilePoints<NCH> / 32;
    static constexpr int norms_at = NCH * 2 * blocks * kFragment;
    static constexpr int weights_at = norms_at + blocks * 512;
    static constexpr int kind_at = weights_at + kTilePoints<NCH> * 4;
    static constexpr int bytes = (kind_at + 4 + kFragment - 1) / kFragment * kFragment;
};

__device__ __forceinline__ void split3(float x, __bf16& hi, __bf16& mid, __bf16& lo) {
    hi = (__bf16)x;
    const float r = x - (float)hi;
    mid = (__bf16)r;
    lo = (__bf16)(r - (float)mid);
}

// Eight coordinates times `scale` as two pieces each, with the squares of what the pieces stand for and of the low
// ones; whether all are in the pieces' range (not so for a NaN).
__device__ __forceinline__ bool split2_row(const float (&x)[8], double scale, f16x8& hi, f16x8& lo, double& square,
                                           float& low) {
    bool fits = true;
    square = 0.0;
    low = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const double a = scale * (double)x[e];
        hi[e] = (_Float16)(float)a;
        const double high = (double)(float)hi[e];
        lo[e] = (_Float16)(float)(a - high);
        const double stands = high + (double)(float)lo[e];
        fits &= fabs(a) <= (double)kMostHalf;
        square += stands * stands;
        low = fmaf((float)lo[e], (float)lo[e], low);
    }
    return fits;
}

// Rows and points with a coordinate out of range are cut into pieces times 2^-shift, one shift for all their coordinates.
// largest: an upper bound of theirs, `scale` included; -1: too far for any (or a NaN, or infinite): pieces of 0.
__device__ __forceinline__ int shift_of(float largest) {
    if (!(largest <= kMostScaled)) return -1;
    return largest <= kMostHalf ? 0 : __builtin_amdgcn_frexp_expf(largest) - 15;  // (below 2^15 then)
}
__device__ __forceinline__ float largest_of(const float (&x)[8], double scale) {
    float most = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float a = fabsf((float)(scale * (double)x[e]));
        most = a <= HUGE_VALF ? fmaxf(most, a) : HUGE_VALF;  // (a NaN: too far)
    }
    return most;
}
// the pieces of eight of its coordinates, and their square as that of the whole numbers
__device__ __forceinline__ void split2_shifted(const float (&x)[8], double scale, int shift, f16x8& hi, f16x8& lo,
                                               double& square) {
    if (shift < 0) {
        square = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            hi[e] = lo[e] = (_Float16)0.f;
            square = fma(scale * (double)x[e], scale * (double)x[e], square);  // (a NaN, infinite, or past kMostScaled)
        }
        return;
    }
    float low;
    split2_row(x, ldexp(scale, -shift), hi, lo, square, low);
    square = ldexp(square, 2 * shift);
}

// coordinates t0 .. t0 + 7 of a row; zeros past d and for rows that are not there
__device__ __forceinline__ void load8(const float* __restrict__ row, bool there, int t0, int d, float (&x)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = there && t0 + e < d ? row[t0 + e] : 0.f;
}

// One workgroup per tile.
template <int NCH>
__global__ __launch_bounds__(256) void kmv_records_kernel(const float* __restrict__ Z, int64_t ldz,
                                                          const float* __restrict__ v, int m, int d,
                                                          double scale, unsigned char* __restrict__ records) {
    using R = Record<NCH>;
    constexpr int TP = kTilePoints<NCH>, G = 2 * NCH;  // groups of 8 coordinates
    __shared__ double squares[TP][G + 1];
    __shared__ float lows[TP][G + 1];
    __shared__ float largest[TP][G + 1];
    __shared__ int kind;
    unsigned char* __restrict__ out = records + (int64_t)blockIdx.x * R::bytes;
    if (threadIdx.x == 0) kind = kTileSmallLows;
    __syncthreads();
    for (int k = threadIdx.x; k < TP * G; k += 256) {
        const int point = k / G, g = k % G;
        const int64_t j = (int64_t)blockIdx.x * TP + point;
        float x[8];
        load8(Z + (j < m ? j : 0) * ldz, j < m, g * 8, d, x);
        f16x8 hi, lo;
        if (!split2_row(x, scale, hi, lo, squares[point][g], lows[point][g])) atomicMax(&kind, kTileOutOfRange);
        unsigned char* at = out + ((g >> 1) * 2 * R::blocks + (point >> 5)) * kFragment + (g & 1) * 512 + (point & 31) * 16;
        *reinterpret_cast<f16x8*>(at) = hi;
        *reinterpret_cast<f16x8*>(at + R::blocks * kFragment) = lo;
    }
    __syncthreads();
    const bool shifted = kind == kTileOutOfRange;  // (the same for the whole workgroup)
    auto shift_at = [&](int point) {
        float most = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) most = fmaxf(most, largest[point][g]);
        return shift_of(most);
    };
    if (shifted) {
        for (int pass = 0; pass < 2; ++pass) {
            for (int k = threadIdx.x; k < TP * G; k += 256) {
                const int point = k / G, g = k % G;
                const int64_t j = (int64_t)blockIdx.x * TP + point;
                float x[8];
                load8(Z + (j < m ? j : 0) * ldz, j < m, g * 8, d, x);
                if (pass == 0) {
                    largest[point][g] = largest_of(x, scale);
                    continue;
                }
                f16x8 hi, lo;
                split2_shifted(x, scale, shift_at(point), hi, lo, squares[point][g]);
                unsigned char* at = out + ((g >> 1) * 2 * R::blocks + (point >> 5)) * kFragment + (g & 1) * 512 + (point & 31) * 16;
                *reinterpret_cast<f16x8*>(at) = hi;
                *reinterpret_cast<f16x8*>(at + R::blocks * kFragment) = lo;
            }
            __syncthreads();
        }
    }
    if ((int)threadIdx.x < TP) {
        const int64_t j = (int64_t)blockIdx.x * TP + threadIdx.x;
        double sq = 0.0;
        float low = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            sq += squares[threadIdx.x][g];
            low += lows[threadIdx.x][g];
        }
        if (!(low <= kSmallLow)) atomicMax(&kind, kTileFits);
        bf16x8 norm;
        __bf16 hi, mid, lo;
        split3(j < m ? fmaxf((float)(-0.5 * sq), -3e38f) : kFar, hi, mid, lo);
        norm[0] = hi;
        norm[1] = mid;
        norm[2] = lo;
        norm[3] = norm[4] = norm[5] = (__bf16)1.f;
        norm[6] = (__bf16)0.f;
        norm[7] = (__bf16)(shifted ? ldexpf(1.f, max(shift_at(threadIdx.x), 0)) : 1.f);
        *reinterpret_cast<bf16x8*>(out + R::norms_at + threadIdx.x * 16) = norm;
        // (a point with a NaN: entries of 0 below, and so its weight makes every sum a NaN)
        *reinterpret_cast<float*>(out + R::weights_at + threadIdx.x * 4) = j >= m ? 0.f : sq != sq ? (float)sq : v[j];
    }
    __syncthreads();
    if (threadIdx.x == 0) *reinterpret_cast<int*>(out + R::kind_at) = kind;
}

// ---------------------------------------------------------------------------------------
// A workgroup of 4 waves owns 128 rows of X, 32 per wave, whose pieces stay in registers, and walks its
// range of tiles through LDS (two records, loaded directly).  Points are the M side, rows the N side, so
// the 16 values a lane holds of a 32 x 32 block belong to one row: it takes their exponentials, times the
// points' weights, into one fp32 sum per tile and half wave, and those into an fp64 sum.  An exponent that
// rounding left above 0 gives 1: the result of exp2 is clamped to [0, 1], a NaN (of an infinite coordinate) to 0.
//
// In a tile with a coordinate out of range, and for rows with one, the products are multiplied back by the powers of two of
// point and row before the norms are added; those of points and rows that are in range are what they are elsewhere.  (So
// far from the origin, 27000 lengthscales, the expansion has no digits left in fp32.  With six products of bf16 pieces made
// there from memory such tiles took 10 to 17 times the time of kmv_mfma_kernel.)
//
// Bound by the power of the matrix and vector units together: at n = m = 200000, d = 32 7.8 ms (14.2 with
// three bf16 pieces cut in every workgroup, kmv_mfma_kernel), at a clock of 1.4 GHz that both keep busy for
// about 70 % of its cycles (seven matrix instructions and 33 vector instructions, 16 of them exp2, per 1024 entries and
// wave).  With the lo lo products in every tile 9.0 ms; n = m = 1e5, lengthscale 0.3 sqrt(d), where every tile has them, d = 9 / 17 / 64
// 1.48 / 2.12 / 4.43 ms against 2.31 / 3.63 / 7.14 by kmv_mfma_kernel.
// ---------------------------------------------------------------------------------------
template <int NCH>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(NCH <= 3 ? 4 : 3, NCH <= 3 ? 4 : 3))) void kmv_pieces_kernel(const float* __restrict__ X, int64_t ldx,
                                                         const float* __restrict__ Z, int64_t ldz,
                                                         const unsigned char* __restrict__ records, int n, int m, int d,
                                                         int range_tiles, double scale,
                                                         double variance, double* __restrict__ out) {
    using R = Record<NCH>;
    constexpr int TP = kTilePoints<NCH>, NB = R::blocks;
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned lds = (unsigned)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i32 = lane & 31, h = lane >> 5;
    const int row = blockIdx.x * kMfmaTileRows + wave * 32 + i32;
    const float* __restrict__ xp = X + (int64_t)min(row, n - 1) * ldx;

    const int all = (m + TP - 1) / TP;
    const int first = blockIdx.y * range_tiles, count = min(range_tiles, all - first);

    auto request = [&](int tile, int buf) {
        const unsigned char* base = records + (int64_t)(first + tile) * R::bytes;
        for (int f = wave; f < R::bytes / kFragment; f += 4)
            load_to_lds(base + f * kFragment, lane * 16, lds + buf * R::bytes + f * kFragment);
    };
    if (count > 0) request(0, 0);

    // this lane's row: the pieces of its scaled coordinates, and its norm for the norms' instruction
    f16x8 bh[NCH], bl[NCH];
    bf16x8 norm;
    bool fits = true;
    double sum = 0.0;  // (from a NaN on where the row has one: its entries come out as 0)
    float low = 0.f, factor = 1.f;
    int rows_kind;
    {
        double sq = 0.0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            float x[8];
            double square;
            float part;
            load8(xp, true, c * 16 + h * 8, d, x);
            fits &= split2_row(x, scale, bh[c], bl[c], square, part);
            sq += square;
            low += part;
        }
        low += __shfl_xor(low, 32);
        rows_kind = __ballot(!fits) ? kTileOutOfRange : __ballot(!(low <= kSmallLow)) ? kTileFits : kTileSmallLows;
        if (rows_kind == kTileOutOfRange) {
            float largest = 0.f;
            for (int c = 0; c < NCH; ++c) {
                float x[8];
                load8(xp, true, c * 16 + h * 8, d, x);
                largest = fmaxf(largest, largest_of(x, scale));
            }
            const int shift = shift_of(fmaxf(largest, __shfl_xor(largest, 32)));
            factor = ldexpf(1.f, max(shift, 0));
            sq = 0.0;
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                float x[8];
                double square;
                load8(xp, true, c * 16 + h * 8, d, x);
                split2_shifted(x, scale, shift, bh[c], bl[c], square);
                sq += square;
            }
        }
        sq += __shfl_xor(sq, 32);
        if (sq != sq) sum = sq;
        __bf16 hi, mid, lo;
        split3(fmaxf((float)(-0.5 * sq), -3e38f), hi, mid, lo);
        const __bf16 one = (__bf16)(h ? 0.f : 1.f), zero = (__bf16)0.f;  // the upper half wave's coordinates 8 .. 15: none
        norm[0] = norm[1] = norm[2] = one;
        norm[3] = h ? zero : hi;
        norm[4] = h ? zero : mid;
        norm[5] = h ? zero : lo;
        norm[6] = norm[7] = zero;
    }

    for (int tile = 0; tile < count; ++tile) {
        const int buf = tile & 1;
        // this tile's record is in LDS, and every wave is through with the other one
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (tile + 1 < count) request(tile + 1, buf ^ 1);
        const unsigned char* rec = smem + buf * R::bytes;
        const unsigned char* frag = rec + lane * 16;
        const unsigned char* norms = rec + R::norms_at + i32 * 16;
        const float* weights = reinterpret_cast<const float*>(rec + R::weights_at) + h * 4;
        const int kind = max(rows_kind, __builtin_amdgcn_readfirstlane(*reinterpret_cast<const int*>(rec + R::kind_at)));
        float part = 0.f;
        auto add = [&](const f32x16& arg, int block) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 w = *reinterpret_cast<const f32x4*>(weights + block * 32 + g * 8);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    part = fmaf(__builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(arg[g * 4 + e]), 0.f, 1.f), w[e], part);
            }
        };
        auto blocks = [&](auto low_product, auto shifted) {
            auto products = [&](int block) {
                f32x16 acc;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 0.f;
                f16x8 ah[NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    ah[c] = *reinterpret_cast<const f16x8*>(frag + (c * 2 * NB + block) * kFragment);
                    const f16x8 al = *reinterpret_cast<const f16x8*>(frag + (c * 2 * NB + NB + block) * kFragment);
                    if constexpr (decltype(low_product)::value)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bl[c], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[c], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[c], bl[c], acc, 0, 0, 0);
                }
#pragma unroll
                for (int c = 0; c < NCH; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[c], bh[c], acc, 0, 0, 0);
                if constexpr (decltype(shifted)::value) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const unsigned char* of = rec + R::norms_at + (block * 32 + (e >> 2) * 8 + h * 4 + (e & 3)) * 16 + 14;
                        acc[e] *= factor * (float)*reinterpret_cast<const __bf16*>(of);
                    }
                }
                const bf16x8 an = *reinterpret_cast<const bf16x8*>(norms + block * 512);
                return __builtin_amdgcn_mfma_f32_32x32x16_bf16(an, norm, acc, 0, 0, 0);
            };
            f32x16 now = products(0);
#pragma unroll
            for (int block = 0; block < NB; ++block) {
                f32x16 next = now;
                if (block + 1 < NB) next = products(block + 1);
                add(now, block);
                now = next;
            }
        };
        if (kind == kTileSmallLows) {
            blocks(std::false_type{}, std::false_type{});
        } else if (kind == kTileFits) {
            blocks(std::true_type{}, std::false_type{});
        } else {
            blocks(std::true_type{}, std::true_type{});
        }
        sum += (double)part;
    }
    const double other = __shfl_xor(sum, 32);
    if (row < n && h == 0) out[(int64_t)blockIdx.y * n + row] = variance * (sum + other);
}

template <int NCH>
hipError_t launch(const float* X, int64_t ldx, const float* Z, int64_t ldz, const float* v, unsigned char* records,
                  int64_t n, int64_t m, int d, double scale, double variance, int S, double* out, hipStream_t stream) {
    const int64_t tiles = (m + kTilePoints<NCH> - 1) / kTilePoints<NCH>;
    const int range = (int)((tiles + S - 1) / S);
    kmv_records_kernel<NCH><<<dim3((unsigned)tiles), dim3(256), 0, stream>>>(Z, ldz, v, (int)m, d, scale, records);
    kmv_pieces_kernel<NCH><<<dim3((unsigned)((n + kMfmaTileRows - 1) / kMfmaTileRows), (unsigned)S), dim3(256),
                             2 * Record<NCH>::bytes, stream>>>(X, ldx, Z, ldz, records, (int)n, (int)m, d, range, scale,
                                                              variance, out);
    return hipGetLastError();
}

template <int NCH>
int64_t record_bytes(int64_t m) {
    return (m + kTilePoints<NCH> - 1) / kTilePoints<NCH> * Record<NCH>::bytes;
}

}  // namespace

int64_t pieces_bytes(int64_t n, int64_t m, int d) {
    if (d <= kLowdMaxD || d > kMfmaKC * kMfmaResidentChunks || m < 1 || n < 1) return 0;
    switch ((d + kMfmaKC - 1) / kMfmaKC) {
        case 1: return record_bytes<1>(m);
        case 2: return record_bytes<2>(m);
        case 3: return record_bytes<3>(m);
        default: return record_bytes<4>(m);
    }
}

hipError_t launch_pieces(const float* X, int64_t ldx, const float* Z, int64_t ldz, const float* v, void* ws, int64_t n,
                         int64_t m, int d, double lengthscale, double variance, int S, double* out, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const double scale = std::sqrt(1.4426950408889634) / lengthscale;  // sqrt(2 c2)
    unsigned char* records = static_cast<unsigned char*>(ws);
    switch ((d + kMfmaKC - 1) / kMfmaKC) {
        case 1: return launch<1>(X, ldx, Z, ldz, v, records, n, m, d, scale, variance, S, out, stream);
        case 2: return launch<2>(X, ldx, Z, ldz, v, records, n, m, d, scale, variance, S, out, stream);
        case 3: return launch<3>(X, ldx, Z, ldz, v, records, n, m, d, scale, variance, S, out, stream);
        default: return launch<4>(X, ldx, Z, ldz, v, records, n, m, d, scale, variance, S, out, stream);
    }
}

}  // namespace kmv
