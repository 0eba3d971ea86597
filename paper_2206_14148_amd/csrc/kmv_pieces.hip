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
constexpr float kMostHalf = 32768.f;  // coordinates beyond this go to the slow way
constexpr float kFar = -1e30f;        // exponent of what pads the last tile
constexpr float kSmallLow = 0x1p-22f;  // |low pieces|^2 of a point up to which their products are left out

// of a tile's points, and of a wave's rows: |low|^2 <= kSmallLow for all, all in the pieces' range, neither
enum Kind { kTileSmallLows, kTileFits, kTileOutOfRange };

// Points of a tile: two of its records in LDS leave room for four workgroups per compute unit, as the registers do up to
// 48 coordinates (beyond, for three).
template <int NCH>
constexpr int kTilePoints = NCH <= 2 ? 128 : 64;

// A tile's record: [chunk of 16 coordinates][piece][block of 32 points] fragments, then per block 32 x 16
// bytes for the norms' instruction, then the points' weights and one word that is not 0 where a
// coordinate is out of the pieces' range.
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

// A coordinate a as two pieces: whether it is in their range (not so for a NaN), and what they stand for,
// a itself where it is not.
__device__ __forceinline__ bool split2(double a, _Float16& hi, _Float16& lo, double& stands) {
    hi = (_Float16)(float)a;
    const double high = (double)(float)hi;
    lo = (_Float16)(float)(a - high);
    const bool fits = fabs(a) <= (double)kMostHalf;
    stands = fits ? high + (double)(float)lo : a;
    return fits;
}

// the same of eight coordinates times `scale`, with the squares of what the pieces stand for and of the low ones
__device__ __forceinline__ bool split2_row(const float (&x)[8], double scale, f16x8& hi, f16x8& lo, double& square,
                                           float& low) {
    bool fits = true;
    square = 0.0;
    low = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        _Float16 h, l;
        double a;
        fits &= split2(scale * (double)x[e], h, l, a);
        hi[e] = h;
        lo[e] = l;
        square += a * a;
        low = fmaf((float)l, (float)l, low);
    }
    return fits;
}

// three pieces of what the two pieces of eight coordinates times `scale` stand for
__device__ __forceinline__ void split3_row(const float (&x)[8], double scale, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        _Float16 h, l;
        double stands;
        split2(scale * (double)x[e], h, l, stands);
        __bf16 a, b, c;
        split3((float)stands, a, b, c);
        hi[e] = a;
        mid[e] = b;
        lo[e] = c;
    }
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
        norm[6] = norm[7] = (__bf16)0.f;
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
// A tile with a coordinate out of range, and rows with one, take the products of three bf16 pieces, made from
// memory on the way, of what the two pieces stand for where they are in range.  So far from the origin (2e4
// lengthscales) the expansion has no digits left in fp32.
//
// Bound by the power of the matrix and vector units together: at n = m = 200000, d = 32 7.8 ms (14.2 with
// three bf16 pieces cut in every workgroup, kmv_mfma_kernel), at a clock of 1.4 GHz that both keep busy for
// about 70 % of its cycles (seven matrix instructions and 33 vector instructions, 16 of them exp2, per 1024 entries and
// wave).  With the lo lo products in every tile 9.0 ms; n = m = 1e5, lengthscale 0.3 sqrt(d), where every tile has them, d = 9 / 17 / 64
// 1.48 / 2.12 / 4.43 ms against 2.31 / 3.63 / 7.14 by kmv_mfma_kernel.
// ---------------------------------------------------------------------------------------
template <int NCH>
__global__ __launch_bounds__(256) void kmv_pieces_kernel(const float* __restrict__ X, int64_t ldx,
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
    float low = 0.f;
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
        sq += __shfl_xor(sq, 32);
        low += __shfl_xor(low, 32);
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
    const int rows_kind = __ballot(!fits) ? kTileOutOfRange : __ballot(!(low <= kSmallLow)) ? kTileFits : kTileSmallLows;

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
        auto blocks = [&](auto low_product) {
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
            blocks(std::false_type{});
        } else if (kind == kTileFits) {
            blocks(std::true_type{});
        } else {
            for (int block = 0; block < NB; ++block) {
                f32x16 acc;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 0.f;
                const int64_t j = (int64_t)(first + tile) * TP + block * 32 + i32;
                for (int c = 0; c < NCH; ++c) {
                    float x[8];
                    bf16x8 a[3], b[3];
                    load8(Z + (j < m ? j : 0) * ldz, j < m, c * 16 + h * 8, d, x);
                    split3_row(x, scale, a[0], a[1], a[2]);
                    load8(xp, true, c * 16 + h * 8, d, x);
                    split3_row(x, scale, b[0], b[1], b[2]);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
                }
                const bf16x8 an = *reinterpret_cast<const bf16x8*>(norms + block * 512);
                add(__builtin_amdgcn_mfma_f32_32x32x16_bf16(an, norm, acc, 0, 0, 0), block);
            }
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
