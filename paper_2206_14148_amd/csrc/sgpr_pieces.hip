// gfx950 (CDNA4, MI355X) kernels for the data-sized sums of sparse GP regression where the limit has
// room for the entries of K_uf as pieces of 16 bits: A = K_uf K_fu and b = K_uf y (paper section 5.3),
// again over chunks of the data (section 4.3), but with chunks as long as the room allows, a product
// whose workgroups share every chunk evenly, and sums over all of a chunk that lose nothing to its length.
//
// Pieces.  The matrix cores multiply 16-bit numbers at sixteen times the fp32 rate, so an entry is cut
// into pieces when it is made, once, and stored in the order in which a wave's operand register reads it:
//   two fp16 pieces, x 2^15 = hi + lo, three products (hi hi, hi lo, lo hi): 23 bits of an entry, so only
//     where no entry is below 2^-16 and lo keeps its 11 bits above fp16's least number (2^-24);
//   three bf16 pieces, x = hi + mid + lo exactly, six products: everywhere else.
// Which of the two a call takes is decided on the device from the radii of U and X around a common
// centre: |u - x| <= radius(U) + radius(X) bounds the least entry.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "knn_config.h"
#include "knn_device.h"
#include "sgpr_kernels.h"

namespace sgpr {

namespace {

using knn::f32x16;
using knn::f32x4;
using knn::load_to_lds;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kFragment = 1024;      // bytes: 32 rows x 16 columns of one piece, in operand order
constexpr int kTile = 128;           // rows and columns of a workgroup's tile of A
constexpr int kXcds = 8, kPerXcd = 2 * knn::kNumCU / kXcds, kGroups = kXcds * kPerXcd;  // two workgroups per compute unit
constexpr int kStageCols = 16;       // columns of K_uf per pipeline stage
constexpr int kKufCols = 256;        // columns of K_uf per workgroup of the kernel that makes them
constexpr int kMostResident = 16;     // coordinates that a lane keeps in registers
constexpr float kHalfScale = 32768.f;

// ---------------------------------------------------------------------------------------
// Radii.  head[0], head[1]: largest squared distance of a row of U and of X from the centre, as the bits
// of a float (NaN bits are larger than any number's, so a NaN decides for the pieces that need no bound).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void sgpr_centre_kernel(const float* __restrict__ U, int64_t ldu, int m, int d,
                                                          unsigned* __restrict__ head, float* __restrict__ centre) {
    // the mean of at most 256 rows of U (any point is a valid centre; near the middle it is a good one)
    __shared__ float part[256];
    const int t = blockIdx.x;
    const int count = min(m, 256);
    const int64_t row = (int64_t)threadIdx.x * m / count;
    part[threadIdx.x] = (int)threadIdx.x < count ? U[row * ldu + t] : 0.f;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        centre[t] = part[0] / (float)count;
        if (t < 2) head[t] = 0;
        if (d == 1) head[1] = 0;
    }
}

__global__ __launch_bounds__(256) void sgpr_radius_kernel(const float* __restrict__ U, int64_t ldu, int m,
                                                          const float* __restrict__ X, int64_t ldx, int64_t n, int d,
                                                          const float* __restrict__ centre,
                                                          unsigned* __restrict__ head) {
    const int64_t total = n + m;
    unsigned most[2] = {0, 0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const bool of_u = i < m;
        const float* __restrict__ p = of_u ? U + i * ldu : X + (i - m) * ldx;
        float sq = 0.f;
        for (int t = 0; t < d; ++t) {
            const float df = p[t] - centre[t];
            sq = fmaf(df, df, sq);
        }
        const unsigned bits = __float_as_uint(sq);  // (sq >= 0 or NaN)
        most[0] = max(most[0], of_u ? bits : 0u);
        most[1] = max(most[1], of_u ? 0u : bits);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) most[s] = max(most[s], (unsigned)__shfl_xor((int)most[s], o));
        if ((threadIdx.x & 63) == 0 && most[s]) atomicMax(head + s, most[s]);
    }
}

// Whether every entry is at least 2^-16 of the variance (with a margin for the roundings of the radii).
__device__ __forceinline__ bool two_pieces(const unsigned* __restrict__ head, float c2) {
    const float r = sqrtf(__uint_as_float(head[0])) + sqrtf(__uint_as_float(head[1]));
    return r * r * c2 <= 15.9f;
}

// ---------------------------------------------------------------------------------------
// Entries of K_uf and the sums with y.  A wave makes 64 rows x 8 columns at a time: the row's coordinates
// stay in the lane's registers, the columns' coordinates are the same for the whole wave and come through
// scalar loads.  Difference form, coordinates in ascending order.  D = 0: any number of coordinates, 16 at a
// time from a transposed copy of U, whose loads are coalesced (64 coordinates, 1000 points, 1e5
// rows: 12.4 ms with U read as it lies, 1.1 this way).
// fragments: [16 columns][piece][32 rows] of 1024 bytes, a lane's 16 bytes being 8 columns of a row.
// sums[column block][row]: fp64 sums of the fp32 products with y.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void sgpr_transpose_kernel(const float* __restrict__ U, int64_t ldu, int m, int d,
                                                             int rows, float* __restrict__ turned) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= rows) return;
    for (int t = blockIdx.y; t < d; t += gridDim.y) turned[(int64_t)t * rows + i] = U[(int64_t)min(i, m - 1) * ldu + t];
}

template <int D>
__global__ __launch_bounds__(256) void sgpr_entries_kernel(const float* __restrict__ U, int64_t ldu,
                                                           const float* __restrict__ X, int64_t ldx,
                                                           const float* __restrict__ y, int m, int64_t c0, int cols,
                                                           int d_any, float c2, float variance,
                                                           const unsigned* __restrict__ head,
                                                           unsigned char* __restrict__ fragments, int row_blocks,
                                                           const float* __restrict__ turned,
                                                           double* __restrict__ sums, int first) {
    __shared__ double part[4][64];
    const int d = D ? D : d_any;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = blockIdx.y * 64 + lane;
    const bool two = two_pieces(head, c2);
    const float* __restrict__ up = U + (int64_t)min(row, m - 1) * ldu;
    float u[D ? D : 1];
    if constexpr (D > 0) {
#pragma unroll
        for (int t = 0; t < D; ++t) u[t] = up[t];
    }
    const float factor = row < m ? variance : 0.f;  // rows that pad the last block are zeros
    const int last = (cols + kStageCols - 1) / kStageCols * kStageCols;
    double sum = 0.0;
    for (int g = 0; g < kKufCols / 4 / 8; ++g) {
        const int c = blockIdx.x * kKufCols + wave * (kKufCols / 4) + g * 8;
        if (c >= last) break;
        float k[8], sq[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sq[j] = 0.f;
        const auto add = [&](const float* __restrict__ at, auto count, int t0) {
            constexpr int N = decltype(count)::value;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float* __restrict__ xp = X + (c0 + min(c + j, cols - 1)) * ldx + t0;
#pragma unroll
                for (int t = 0; t < N; ++t) {
                    const float df = xp[t] - at[t];
                    sq[j] = fmaf(df, df, sq[j]);
                }
            }
        };
        if constexpr (D > 0) {
            add(u, std::integral_constant<int, D>{}, 0);
        } else {
            const int rows = row_blocks * 32;
            int t0 = 0;
            for (; t0 + 16 <= d; t0 += 16) {
                float part_u[16];
#pragma unroll
                for (int t = 0; t < 16; ++t) part_u[t] = turned[(int64_t)(t0 + t) * rows + row];
                add(part_u, std::integral_constant<int, 16>{}, t0);
            }
            for (; t0 < d; ++t0) {
                const float one = turned[(int64_t)t0 * rows + row];
                add(&one, std::integral_constant<int, 1>{}, t0);
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int cj = min(c + j, cols - 1);
            k[j] = (c + j < cols ? factor : 0.f) * __builtin_amdgcn_exp2f(sq[j] * -c2);
            if (row >= m || c + j >= cols) k[j] = 0.f;  // (a NaN of the row or point that was read instead)
            sum += c + j < cols ? (double)(k[j] * y[c0 + cj]) : 0.0;
        }
        const int64_t step = c >> 4;
        const int half = (c >> 3) & 1;
        const int block = row >> 5;
        if (two) {
            f16x8 hi, lo;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x = k[j] * kHalfScale;
                hi[j] = (_Float16)x;
                lo[j] = (_Float16)(x - (float)hi[j]);
            }
            unsigned char* at = fragments + ((step * 2) * row_blocks + block) * kFragment + half * 512 + (row & 31) * 16;
            *reinterpret_cast<f16x8*>(at) = hi;
            *reinterpret_cast<f16x8*>(at + (int64_t)row_blocks * kFragment) = lo;
        } else {
            bf16x8 hi, mid, lo;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                hi[j] = (__bf16)k[j];
                const float r1 = k[j] - (float)hi[j];
                mid[j] = (__bf16)r1;
                lo[j] = (__bf16)(r1 - (float)mid[j]);
            }
            unsigned char* at = fragments + ((step * 3) * row_blocks + block) * kFragment + half * 512 + (row & 31) * 16;
            *reinterpret_cast<bf16x8*>(at) = hi;
            *reinterpret_cast<bf16x8*>(at + (int64_t)row_blocks * kFragment) = mid;
            *reinterpret_cast<bf16x8*>(at + (int64_t)row_blocks * 2 * kFragment) = lo;
        }
    }
    part[wave][lane] = sum;
    __syncthreads();
    if (wave == 0 && row < m) {
        const double s = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
        double* at = sums + (int64_t)blockIdx.x * m + row;
        *at = first ? s : *at + s;
    }
}

// ---------------------------------------------------------------------------------------
// Tiles of the lower triangle of A and their order: bands of 8 rows of tiles; a band's tiles left of the
// diagonal in squares of 8, row by row in each, then what touches the diagonal.
// ---------------------------------------------------------------------------------------
int tile_count(int64_t m) {
    const int64_t rows = (m + kTile - 1) / kTile;
    return (int)(rows * (rows + 1) / 2);
}
__device__ __forceinline__ void tile_at(int seq, int m, int& r, int& c) {
    const int rows_all = (m + kTile - 1) / kTile;
    for (int r0 = 0;; r0 += 8) {
        const int rows = min(8, rows_all - r0);
        if (seq < rows * r0) {
            const int square = seq / (rows * 8), in = seq - square * rows * 8;
            r = r0 + in / 8;
            c = square * 8 + in % 8;
            return;
        }
        seq -= rows * r0;
        for (int i = 0; i < rows; ++i) {
            if (seq <= i) {
                r = r0 + i;
                c = r0 + seq;
                return;
            }
            seq -= i + 1;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Who makes what.  Workgroups go round-robin to the 8 XCDs, each with its own L2 and room for kPerXcd
// workgroups.  The XCDs form `shares` sets; a set takes one share of a chunk's stages, for all the
// tiles, and its XCDs runs of neighbouring tiles.  An XCD's workgroups take kPerXcd tiles at a time and walk
// the same stages together, so what one reads of the chunk the others find in the L2.  (One line of
// all tiles' stages cut into equal lengths, which leaves no workgroup idle but has each start at another
// stage, measured 7.5 TB/s from beyond the L2: 620 us for a chunk of 8704 columns at 4000 inducing points,
// 475 this way.)  Tiles that are left over are split, each over `parts` workgroups by its stages.  The part
// of a tile that begins at the chunk's first stage goes into A, every other one into a buffer of its
// workgroup and turn, the same in every chunk.
// ---------------------------------------------------------------------------------------
struct Shares {
    int first, count, turns, left, parts;  // first, count: the XCD's tiles
    __host__ __device__ Shares(int tiles, int shares, int part_limit, int xcd) {
        const int xcds = kXcds / shares, at = xcd / shares;
        first = (int)((int64_t)at * tiles / xcds);
        count = (int)((int64_t)(at + 1) * tiles / xcds) - first;
        turns = count / kPerXcd;
        left = count - turns * kPerXcd;
        parts = left ? kPerXcd / left : 1;
        if (parts > part_limit) parts = part_limit;
    }
};

// ---------------------------------------------------------------------------------------
// Chunk product.  Stages of 16 columns go from memory into LDS directly, kStages deep.  A wave holds 64 x
// 64 entries of the tile: per stage four operands of each piece from LDS (conflict free: 64 lanes read
// 1024 bytes in order) for four blocks of products, which run while the next stage is waited for and read.
// Two workgroups per compute unit cover each other's barriers and sums (one per compute unit with tiles of
// 192 x 128 and a stage ahead in registers: 1280 us against 1178 for 25000 columns).
//
// fp32 sums: the products of the high pieces and the smaller ones have accumulators of their own (in one
// accumulator the matrix unit loses part of the small ones: error of A 3.2e-8 against 2.1e-8, 4000
// inducing points, 3e5 rows of 11 features).  The first run over kRun stages and are then added to the tile's
// total by an addition whose rounding error goes to the small ones, which are 2^8 or more below it, so
// the error does not grow with the chunk.
//
// Bound by the matrix cores: 1.10 PFLOP/s of fp16 products (m = 4000), 1.22 of bf16 (m = 10000); a large
// product of the vendor's library reaches 1.21 here.
//
// Registers: 192 accumulators and 48 of operands of the 256 a lane may have.  So the operands of a run's first stage
// are read after the additions of the run before, and where a fragment lies is kept in scalars: with both in
// vector registers 87 were spilled, to private memory outside the workspace (252 bytes a lane, 33 MB).  Whole calls with
// and without the spills, ms: 4000 inducing points, 2e6 rows of 11 101.7 / 101.6, as three pieces 182.3 / 167.5; 10000, 5e5
// of 3 293.5 / 257.1; 300, 1e5 of 11 0.257 / 0.241.
// ---------------------------------------------------------------------------------------
template <int NP>
struct Pieces;
template <>
struct Pieces<2> {
    typedef f16x8 vec;
    static __device__ __forceinline__ void products(const vec (&a)[2], const vec (&b)[2], f32x16& c, f32x16& low) {
        low = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[0], low, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[0], c, 0, 0, 0);
        low = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[1], low, 0, 0, 0);
    }
};
template <>
struct Pieces<3> {
    typedef bf16x8 vec;
    static __device__ __forceinline__ void products(const vec (&a)[3], const vec (&b)[3], f32x16& c, f32x16& low) {
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], low, 0, 0, 0);
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], low, 0, 0, 0);
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], low, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], c, 0, 0, 0);
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], low, 0, 0, 0);
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], low, 0, 0, 0);
    }
};

template <int NP>
constexpr int kStages = NP == 2 ? 4 : 3;  // in LDS: 64 or 72 KB, two workgroups per compute unit
constexpr int kRun = 24;                  // stages of one fp32 run
constexpr int kLeastStages = 16;          // of a part of a tile

struct ProductArgs {
    const unsigned char* fragments;
    int row_blocks, m, tiles, stages, shares, part_limit, slots, first;
    float c2;
    const unsigned* head;
    double scale;
    double* A;
    int64_t lda;
    double* buffers;
};

template <int NP>
__device__ __forceinline__ void multiply_tiles(const ProductArgs& g, double scale) {
    constexpr int WR = kTile / 64;                       // blocks of 32 rows of a wave, and of 32 columns
    constexpr int kSide = kTile / 32, kFrags = 2 * kSide;  // fragments of a piece of a stage
    constexpr int kStageBytes = NP * kFrags * kFragment;
    constexpr int kLoads = NP * kFrags / 4;  // per wave and stage
    static_assert(NP * kFrags % 4 == 0, "a stage's fragments are shared evenly");
    using vec = typename Pieces<NP>::vec;
    const int m = g.m, first = g.first;

    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned lds = (unsigned)reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wy = wave >> 1, wx = wave & 1;
    const unsigned lane_bytes = lane * 16;

    const int xcd = blockIdx.x % kXcds, unit = blockIdx.x / kXcds;
    const Shares mine(g.tiles, g.shares, g.part_limit, xcd);
    const int share = xcd % g.shares;
    const int share0 = (int)((int64_t)share * g.stages / g.shares), share1 = (int)((int64_t)(share + 1) * g.stages / g.shares);

    for (int turn = 0; turn <= mine.turns; ++turn) {
        int tile, s0 = share0, s1 = share1;
        if (turn < mine.turns) {
            tile = mine.first + turn * kPerXcd + unit;
        } else {  // what is left over
            if (unit >= mine.left * mine.parts) break;
            const int part = unit / mine.left;
            tile = mine.first + turn * kPerXcd + unit - part * mine.left;
            s0 = share0 + (int)((int64_t)part * (share1 - share0) / mine.parts);
            s1 = share0 + (int)((int64_t)(part + 1) * (share1 - share0) / mine.parts);
        }
        const bool into_a = share == 0 && (turn < mine.turns || unit < mine.left);
        double* buffer = g.buffers + ((int64_t)blockIdx.x * g.slots + min(turn, g.slots - 1)) * (kTile * kTile);
        const int count = s1 - s0;
        if (count <= 0) {  // a short chunk; the first one still makes every sum
            if (first) {
                int r, c;
                tile_at(tile, m, r, c);
                for (int e = wave * 64 + lane; e < kTile * kTile; e += 256) {
                    const int row = r * kTile + e / kTile, col = c * kTile + e % kTile;
                    if (!into_a)
                        buffer[e] = 0.0;
                    else if (row < m && col < m)
                        g.A[(int64_t)row * g.lda + col] = 0.0;
                }
            }
            continue;
        }
        int r, c;
        tile_at(tile, m, r, c);
        r = __builtin_amdgcn_readfirstlane(r);
        c = __builtin_amdgcn_readfirstlane(c);

        // from one (16 columns, piece) to the next
        const int64_t step_bytes = (int64_t)g.row_blocks * kFragment;
        const unsigned char* base = g.fragments + (int64_t)s0 * NP * step_bytes;
        // this wave's fragments: wave, wave + 4, ... of a stage's [piece][row blocks, column blocks]
        auto request = [&](int stage, unsigned buf) {  // stage from s0
            const unsigned char* from = base + (int64_t)stage * NP * step_bytes;
            const unsigned to = lds + buf + wave * kFragment;
#pragma unroll
            for (int l = 0; l < kLoads; ++l) {
                const int piece = 4 * l / kFrags, in = wave + 4 * l - piece * kFrags;
                const int block = in < kSide ? r * kSide + in : c * kSide + in - kSide;
                load_to_lds(from + piece * step_bytes + (int64_t)block * kFragment, lane_bytes, to + 4 * l * kFragment);
            }
        };

        vec a[WR][NP], b[2][NP];
        auto operands = [&](unsigned buf) {
            const unsigned char* p = smem + buf + lane_bytes;
#pragma unroll
            for (int q = 0; q < NP; ++q) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    b[i][q] = *reinterpret_cast<const vec*>(p + (q * kFrags + kSide + wx * 2 + i) * kFragment);
#pragma unroll
                for (int i = 0; i < WR; ++i)
                    a[i][q] = *reinterpret_cast<const vec*>(p + (q * kFrags + wy * WR + i) * kFragment);
            }
        };

        f32x16 acc[WR][2], low[WR][2], big[WR][2];
#pragma unroll
        for (int i = 0; i < WR; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = big[i][j][e] = 0.f;
        auto multiply = [&]() {
#pragma unroll
            for (int i = 0; i < WR; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) Pieces<NP>::products(a[i], b[j], acc[i][j], low[i][j]);
        };
        auto drain = [&](int block) {
            const int i = block / 2, j = block % 2;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float t = acc[i][j][e], s = big[i][j][e] + t;
                low[i][j][e] += (big[i][j][e] - s) + t;
                big[i][j][e] = s;
                acc[i][j][e] = 0.f;
            }
        };

        // all waves have read the piece before's last stage from LDS
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        unsigned buf = 0;  // of the stage in hand
#pragma unroll
        for (int ahead = 0; ahead < kStages<NP>; ++ahead)  // past the end: a harmless second load
            request(min(ahead, count - 1), ahead * kStageBytes);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((kStages<NP> - 1) * kLoads) : "memory");

        int stage = 0;
        while (stage < count) {
            const int run_end = min(stage + kRun, count);
            operands(buf);  // (none is kept over the additions below: their registers are needed there)
            for (;;) {
                const unsigned next = buf + kStageBytes == kStages<NP> * kStageBytes ? 0 : buf + kStageBytes;
                multiply();
                // the next stage is in LDS, and every wave has read the whole of this one
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kStages<NP> - 2) * kLoads) : "memory");
                request(min(stage + kStages<NP>, count - 1), buf);
                buf = next;
                if (++stage == run_end) break;
                operands(buf);
            }
#pragma unroll
            for (int block = 0; block < 2 * WR; ++block) drain(block);
        }

        // element e of block (i, j): row 32 i + 8 (e / 4) + 4 (lane / 32) + e % 4, column 32 j + lane % 32
        int lr = wy * 32 * WR + 4 * (lane >> 5), lc = wx * 64 + (lane & 31);
        asm("" : "+v"(lr), "+v"(lc));  // (or the entries' addresses are made, and spilled, before the loop)
#pragma unroll
        for (int i = 0; i < WR; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = lr + 32 * i + 8 * (e >> 2) + (e & 3), col = lc + 32 * j;
                    const double v = scale * ((double)big[i][j][e] + (double)low[i][j][e]);
                    double* to = buffer + row * kTile + col;
                    if (into_a) {
                        if (r * kTile + row >= m || c * kTile + col >= m) continue;
                        to = g.A + (int64_t)(r * kTile + row) * g.lda + c * kTile + col;
                    }
                    *to = first ? v : *to + v;
                }
    }
}

__global__ __launch_bounds__(256, 2) void sgpr_product_kernel(const ProductArgs g) {
    if (two_pieces(g.head, g.c2))
        multiply_tiles<2>(g, g.scale / ((double)kHalfScale * kHalfScale));
    else
        multiply_tiles<3>(g, g.scale);
}

// The rest, in a fixed order: the buffers of a tile's other parts are added to what A holds of it, the sum goes
// to both sides of the diagonal (32 x 32 entries per workgroup, through LDS so that loads and
// stores run along rows), and the workgroups past the tiles add up b.
__global__ __launch_bounds__(256) void sgpr_finish_kernel(const double* __restrict__ buffers, int m, int tiles, int shares,
                                                          int part_limit, int slots, double* __restrict__ A, int64_t lda,
                                                          const double* __restrict__ sums, int sum_count, double scale,
                                                          double* __restrict__ b) {
    __shared__ double mirror[32][33];
    if ((int)blockIdx.x >= tiles) {
        const int i = (((int)blockIdx.x - tiles) * 16 + blockIdx.y) * 256 + threadIdx.x;
        if (i >= m) return;
        double acc = 0.0;
        for (int s = 0; s < sum_count; ++s) acc += sums[(int64_t)s * m + i];
        b[i] = scale * acc;
        return;
    }
    const int tile = blockIdx.x;
    const int sets = kXcds / shares;
    int at = 0;
    while (at + 1 < sets && Shares(tiles, shares, part_limit, (at + 1) * shares).first <= tile) ++at;
    const Shares mine(tiles, shares, part_limit, at * shares);
    const int turn = (tile - mine.first) / kPerXcd, place = (tile - mine.first) % kPerXcd;
    const int parts = turn < mine.turns ? 1 : mine.parts;
    int r, c;
    tile_at(tile, m, r, c);
    const int br = blockIdx.y >> 2, bc = blockIdx.y & 3;
    const int j0 = r * kTile + br * 32, i0 = c * kTile + bc * 32;
    if (i0 > j0) return;
    const int x = threadIdx.x & 31;
    for (int y = threadIdx.x >> 5; y < 32; y += 8) {
        const int j = j0 + y, i = i0 + x;
        if (j >= m || i > j) continue;
        double acc = A[(int64_t)j * lda + i];
        for (int share = 0; share < shares; ++share)
            for (int part = share == 0 ? 1 : 0; part < parts; ++part) {
                const int64_t group = (int64_t)(place + part * mine.left) * kXcds + at * shares + share;
                acc += buffers[(group * slots + min(turn, slots - 1)) * (kTile * kTile) + (br * 32 + y) * kTile + bc * 32 + x];
            }
        A[(int64_t)j * lda + i] = acc;
        mirror[y][x] = acc;
    }
    __syncthreads();
    for (int y = threadIdx.x >> 5; y < 32; y += 8) {
        const int j = j0 + x, i = i0 + y;
        if (j < m && i < j) A[(int64_t)i * lda + j] = mirror[x][y];
    }
}

}  // namespace

// ---- host -------------------------------------------------------------------------------

namespace {

int64_t up(int64_t v, int64_t to) { return (v + to - 1) / to * to; }

}  // namespace

PiecesPlan plan_pieces(int64_t m, int64_t n, int d, uint64_t bytes) {
    PiecesPlan p{};
    if (n < 1) return p;
    const int64_t rows = up(m, kTile);
    p.row_blocks = (int)(rows / 32);
    p.tiles = tile_count(m);
    const int64_t n16 = up(n, kStageCols);
    auto layout = [&](int64_t cols) {
        const int64_t stages = cols / kStageCols;
        // Enough parts of tiles for every compute unit, none of fewer than kLeastStages stages.
        p.shares = 1;
        while (p.shares < kXcds && (int64_t)p.tiles * p.shares <= kGroups && stages >= 2 * p.shares * kLeastStages) p.shares *= 2;
        const int64_t per_share = stages / p.shares / kLeastStages;
        p.part_limit = (int)(per_share < 1 ? 1 : per_share < kPerXcd ? per_share : kPerXcd);
        int turns = 0;
        p.units = 0;
        for (int x = 0; x < kXcds; ++x) {
            const Shares s(p.tiles, p.shares, p.part_limit, x);
            const int units = s.turns > 0 ? kPerXcd : s.left * s.parts;
            if (s.turns > turns) turns = s.turns;
            if (units > p.units) p.units = units;
        }
        p.slots = p.shares > 1 ? turns + 1 : 1;
        int64_t at = 0;
        auto take = [&](int64_t b) {
            const int64_t here = at;
            at = up(at + b, knn::kAlign);
            return here;
        };
        p.head_at = take(64);
        p.centre_at = take(4 * (int64_t)d);
        p.turned_at = take(d > kMostResident ? 4 * rows * d : 0);
        p.sums_at = take(up(cols, kKufCols) / kKufCols * m * 8);
        p.buffers_at = take((int64_t)kXcds * p.units * p.slots * kTile * kTile * 8);
        p.fragments_at = take(cols * rows * 6);
        return at;
    };
    // As many columns as the room holds, up to kMostPieceBytes of pieces: the sums' way to memory and back, once per
    // chunk, is some 40 us at 4000 inducing points (200 MiB of pieces: 18.1 ms for 3e5 rows, 600: 15.8).
    int64_t cols = up(kMostPieceBytes / (rows * 6), kKufCols);
    if (cols < n16) {  // equal chunks
        const int64_t count = (n + cols - 1) / cols;
        cols = up((n + count - 1) / count, kKufCols);
    }
    if (cols > n16) cols = n16;
    for (;;) {
        const int64_t over = layout(cols) - (int64_t)bytes;
        if (over <= 0) break;
        cols = (cols - (over + rows * 6 - 1) / (rows * 6)) / kKufCols * kKufCols;
        if (cols <= 0) return PiecesPlan{};
    }
    // Shorter chunks than this spend more on their sums' way to memory and back than the plan without pieces
    // saves: 1e4 inducing points, 3e4 rows of 3 21.4 ms in chunks of 1536 against 20.3, 18.1 in chunks of 2560.
    if (cols < kLeastCols && cols < n16) return PiecesPlan{};
    p.cols = cols;
    p.bytes = layout(cols);
    return p;
}

namespace {

template <int D>
void entries(dim3 grid, hipStream_t stream, const float* U, int64_t ldu, const float* X, int64_t ldx, const float* y,
             int m, int64_t c0, int cols, int d, float c2, float variance, const unsigned* head,
             unsigned char* fragments, int row_blocks, const float* turned, double* sums, int first) {
    if constexpr (D > 0) {
        if (d != D) return entries<D - 1>(grid, stream, U, ldu, X, ldx, y, m, c0, cols, d, c2, variance, head, fragments, row_blocks, turned, sums, first);
    }
    sgpr_entries_kernel<D><<<grid, dim3(256), 0, stream>>>(U, ldu, X, ldx, y, m, c0, cols, d, c2, variance, head,
                                                           fragments, row_blocks, turned, sums, first);
}

}  // namespace

hipError_t launch_radii(const PiecesPlan& p, unsigned char* ws, const float* U, int64_t ldu, const float* X, int64_t ldx,
                        int64_t m, int64_t n, int d, hipStream_t stream) {
    unsigned* head = reinterpret_cast<unsigned*>(ws + p.head_at);
    float* centre = reinterpret_cast<float*>(ws + p.centre_at);
    sgpr_centre_kernel<<<dim3(d), dim3(256), 0, stream>>>(U, ldu, (int)m, d, head, centre);
    const int64_t blocks = (n + m + 255) / 256;
    sgpr_radius_kernel<<<dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(256), 0, stream>>>(U, ldu, (int)m, X, ldx, n,
                                                                                               d, centre, head);
    if (d > kMostResident) {
        const int rows = p.row_blocks * 32;
        sgpr_transpose_kernel<<<dim3((unsigned)((rows + 255) / 256), (unsigned)(d < 1024 ? d : 1024)), dim3(256), 0, stream>>>(
            U, ldu, (int)m, d, rows, reinterpret_cast<float*>(ws + p.turned_at));
    }
    return hipGetLastError();
}

hipError_t launch_entries(const PiecesPlan& p, unsigned char* ws, const float* U, int64_t ldu, const float* X, int64_t ldx,
                          const float* y, int64_t m, int64_t c0, int64_t cols, int d, float c2, float variance, int first,
                          hipStream_t stream) {
    const dim3 grid((unsigned)((cols + kKufCols - 1) / kKufCols), (unsigned)(p.row_blocks / 2));
    unsigned* head = reinterpret_cast<unsigned*>(ws + p.head_at);
    double* sums = reinterpret_cast<double*>(ws + p.sums_at);
    if (d <= kMostResident) {
        entries<kMostResident>(grid, stream, U, ldu, X, ldx, y, (int)m, c0, (int)cols, d, c2, variance, head, ws + p.fragments_at,
                    p.row_blocks, reinterpret_cast<const float*>(ws + p.turned_at), sums, first);
    } else {
        entries<0>(grid, stream, U, ldu, X, ldx, y, (int)m, c0, (int)cols, d, c2, variance, head, ws + p.fragments_at,
                   p.row_blocks, reinterpret_cast<const float*>(ws + p.turned_at), sums, first);
    }
    return hipGetLastError();
}

hipError_t launch_products(const PiecesPlan& p, unsigned char* ws, int64_t m, int64_t cols, float c2, double scale,
                           double* A, int64_t lda, int first, hipStream_t stream) {
    constexpr size_t lds_two = (size_t)kStages<2> * 2 * (2 * kTile / 32) * kFragment;
    constexpr size_t lds_three = (size_t)kStages<3> * 3 * (2 * kTile / 32) * kFragment;
    constexpr size_t lds = lds_two > lds_three ? lds_two : lds_three;
    hipError_t e = knn::raise_lds_limit(sgpr_product_kernel, lds);
    if (e != hipSuccess) return e;
    ProductArgs g;
    g.fragments = ws + p.fragments_at;
    g.row_blocks = p.row_blocks;
    g.m = (int)m;
    g.tiles = p.tiles;
    g.stages = (int)((cols + kStageCols - 1) / kStageCols);
    g.shares = p.shares;
    g.part_limit = p.part_limit;
    g.slots = p.slots;
    g.first = first;
    g.c2 = c2;
    g.head = reinterpret_cast<const unsigned*>(ws + p.head_at);
    g.scale = scale;
    g.A = A;
    g.lda = lda;
    g.buffers = reinterpret_cast<double*>(ws + p.buffers_at);
    sgpr_product_kernel<<<dim3(kXcds * p.units), dim3(256), lds, stream>>>(g);
    return hipGetLastError();
}

hipError_t launch_finish(const PiecesPlan& p, unsigned char* ws, int64_t m, double scale, double* A, int64_t lda,
                         double* b, hipStream_t stream) {
    const int count = (int)(up(p.cols, kKufCols) / kKufCols);
    sgpr_finish_kernel<<<dim3((unsigned)(p.tiles + (m + 4095) / 4096), 16), dim3(256), 0, stream>>>(
        reinterpret_cast<const double*>(ws + p.buffers_at), (int)m, p.tiles, p.shares, p.part_limit, p.slots, A, lda,
        reinterpret_cast<const double*>(ws + p.sums_at), count, scale, b);
    return hipGetLastError();
}

}  // namespace sgpr
