// gfx950 (CDNA4, MI355X): squared row norms, the  sum x^2  term of the expansion in paper
// section 4.1, and their reciprocal square roots (the row scale of the cosine metric).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "knn_config.h"
#include "knn_device.h"
#include "knn_kernels.h"

namespace knn {

namespace {

// ---------------------------------------------------------------------------------------
// Row norms (section 4.1, the sum x^2 term): P lanes per row (P = 64, or the power of two that holds a
// shorter row), so 64 / P rows per wave, and kRowsAhead of these groups at a time, whose loads are in
// flight together.  Fixed summation order, the same for every P: lane t sums coordinates t, t + 64, ..,
// lanes are added by a butterfly (whose steps beyond P would add zeros).  Bound by the memory: 2.8e6 rows
// of 230 886 us with one row per wave at a time, 530 this way.
// ---------------------------------------------------------------------------------------
// inverse != 0 writes 1 / sqrt(sum) instead (0 for a zero row): the cosine metric's row scale.
// hdr != null: from the same pass hdr[0] gets the largest value written and hdr[1] max_j |x_j - bf16(x_j)|^2 (bits of
// non-negative floats, an integer maximum orders them; zeroed beforehand), the largest rounding residual
// that the bf16 filters of the d > 8 kernels have to allow for.
constexpr int kRowsAhead = 4;
template <int P>
__global__ __launch_bounds__(256) void knn_row_norms_kernel(const float* __restrict__ X,
                                                            int64_t ldx, int64_t n, int d,
                                                            int inverse, float* __restrict__ xn,
                                                            unsigned* __restrict__ hdr) {
    constexpr int G = kWave / P;  // rows of a group
    const int lane = threadIdx.x & 63, sub = lane / P, t0 = lane % P;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    float worst = 0.f, most = 0.f;
    for (int64_t j0 = wave * (G * kRowsAhead); j0 < n; j0 += nwaves * (G * kRowsAhead)) {
        float acc[kRowsAhead], res[kRowsAhead];
        const float* row[kRowsAhead];
#pragma unroll
        for (int r = 0; r < kRowsAhead; ++r) {
            acc[r] = res[r] = 0.f;
            const int64_t j = j0 + r * G + sub;
            row[r] = X + (j < n ? j : n - 1) * ldx;
        }
        for (int t = t0; t < d; t += kWave) {
            float v[kRowsAhead];
#pragma unroll
            for (int r = 0; r < kRowsAhead; ++r) v[r] = row[r][t];
#pragma unroll
            for (int r = 0; r < kRowsAhead; ++r) {
                acc[r] = fmaf(v[r], v[r], acc[r]);
                // v minus its bf16 rounding (round to nearest even), exact in fp32
                const unsigned u = __float_as_uint(v[r]);
                const float e = v[r] - __uint_as_float((u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u);
                res[r] = fmaf(e, e, res[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < kRowsAhead; ++r) {
#pragma unroll
            for (int s = P / 2; s > 0; s >>= 1) {
                acc[r] += __shfl_xor(acc[r], s);
                res[r] += __shfl_xor(res[r], s);
            }
            const int64_t j = j0 + r * G + sub;
            if (inverse) acc[r] = acc[r] > 0.f ? 1.f / sqrtf(acc[r]) : 0.f;
            if (t0 == 0 && j < n) xn[j] = acc[r];
            worst = fmaxf(worst, res[r]);  // (a row past the end repeats the last one)
            most = fmaxf(most, acc[r]);
        }
    }
    if (hdr) {  // one request per workgroup (they all go to the same words)
        __shared__ float wmax[2][4];
#pragma unroll
        for (int s = 32; s >= P; s >>= 1) {
            worst = fmaxf(worst, __shfl_xor(worst, s));
            most = fmaxf(most, __shfl_xor(most, s));
        }
        if (lane == 0) {
            wmax[0][threadIdx.x >> 6] = most;
            wmax[1][threadIdx.x >> 6] = worst;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            const float* const w = wmax[threadIdx.x];
            raise_word(hdr + threadIdx.x, __float_as_uint(fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3]))));
        }
    }
}

}  // namespace

hipError_t launch_row_norms(const float* X, int64_t ldx, int64_t n, int d, bool inverse, float* xn,
                            hipStream_t stream, void* hdr) {
    const int lanes = d > 32 ? 64 : d > 16 ? 32 : d > 8 ? 16 : d > 4 ? 8 : d > 2 ? 4 : 2;
    const int64_t per_block = 4 * (kWave / lanes) * kRowsAhead;
    int64_t blocks = (n + per_block - 1) / per_block;
    if (blocks > 4096) blocks = 4096;
    auto go = [&](auto kernel) {
        kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(X, ldx, n, d, inverse ? 1 : 0, xn,
                                                                 static_cast<unsigned*>(hdr));
    };
    switch (lanes) {
        case 64: go(knn_row_norms_kernel<64>); break;
        case 32: go(knn_row_norms_kernel<32>); break;
        case 16: go(knn_row_norms_kernel<16>); break;
        case 8: go(knn_row_norms_kernel<8>); break;
        case 4: go(knn_row_norms_kernel<4>); break;
        default: go(knn_row_norms_kernel<2>); break;
    }
    return hipGetLastError();
}
}  // namespace knn
