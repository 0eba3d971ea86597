// Internal launcher interface between the SGPR C ABI (sgpr_api.hip) and its gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace sgpr {

// A[0..m)[0..m) = 0 and (b != nullptr) b[0..m) = 0.
hipError_t launch_zero(double* A, int64_t lda, double* b, int64_t m, hipStream_t stream);

// Kc[i][c] = variance * exp2(-c2 * |U[i] - X[c0 + c]|^2) for i < m, c < cols (fp32, ld = ldk).
hipError_t launch_kuf(const float* U, int64_t ldu, const float* X, int64_t ldx, int64_t m,
                      int64_t c0, int64_t cols, int d, float c2, float variance, float* Kc,
                      int64_t ldk, hipStream_t stream);

// Lower triangle (whole diagonal tiles): A[j][i] += sum_c Kc[j][c] * Kc[i][c].  The columns are
// cut into `groups` runs (multiples of 16); run 0 adds into A, run g > 0 into the m x m copy
// copies + (g - 1) * copy_stride (leading dimension m).
hipError_t launch_syrk(const float* Kc, int64_t ldk, int64_t m, int64_t cols, int groups, double scale, double* A,
                       int64_t lda, double* copies, int64_t copy_stride, hipStream_t stream);

// Lower triangle: A[j][i] += copy_0[j][i] + copy_1[j][i] + ... in that order.
hipError_t launch_add_copies(double* A, int64_t lda, const double* copies, int64_t copy_stride,
                             int ncopies, int64_t m, hipStream_t stream);

// b[i] += sum_c Kc[i][c] * y[c0 + c].
hipError_t launch_kufy(const float* Kc, int64_t ldk, int64_t m, int64_t cols, const float* y, double scale, double* b, hipStream_t stream);

// A[i][j] = A[j][i] for j > i.
hipError_t launch_symmetrize(double* A, int64_t lda, int64_t m, hipStream_t stream);

// ---- K_uf as pieces of 16 bits (sgpr_pieces.hip) ------------------------------------------

constexpr int64_t kMostPieceBytes = 600 << 20;  // of a chunk's pieces
constexpr int64_t kLeastCols = 2048;            // of a chunk that is not the whole of the data

// Where things lie in the workspace, from its start; cols = 0: not enough room.
struct PiecesPlan {
    int64_t cols;  // per chunk
    int64_t head_at, centre_at, turned_at, sums_at, buffers_at, fragments_at, bytes;
    int row_blocks, tiles, shares, part_limit, slots, units;  // who makes what: see Shares
};
PiecesPlan plan_pieces(int64_t m, int64_t n, int d, uint64_t bytes);

// In this order: the radii once, then per chunk (c0, cols) its entries, with the sums for b, and its
// products (first: the call's first chunk, whose sums are written and not added), then once the rest.
hipError_t launch_radii(const PiecesPlan& p, unsigned char* ws, const float* U, int64_t ldu, const float* X, int64_t ldx,
                        int64_t m, int64_t n, int d, hipStream_t stream);
hipError_t launch_entries(const PiecesPlan& p, unsigned char* ws, const float* U, int64_t ldu, const float* X, int64_t ldx,
                          const float* y, int64_t m, int64_t c0, int64_t cols, int d, float c2, float variance, int first,
                          hipStream_t stream);
hipError_t launch_products(const PiecesPlan& p, unsigned char* ws, int64_t m, int64_t cols, float c2, double scale,
                           double* A, int64_t lda, int first, hipStream_t stream);
hipError_t launch_finish(const PiecesPlan& p, unsigned char* ws, int64_t m, double scale, double* A, int64_t lda,
                         double* b, hipStream_t stream);

}  // namespace sgpr
