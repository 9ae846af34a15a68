// Row scales of RMSNorm for the MFMA path of the RMSNorm-fused Gated MLP.
//
// RMSNorm (the equation of Section 2) multiplies each row x of X by
// r = 1 / sqrt(mean(x^2) + eps).  The paper's headline reorder moves that
// multiply past the matmul, (x * r) W = r * (x W), so the two parts become
// independent: this kernel computes r for every row while X itself goes to
// the gate/up GEMM unnormalised, and the GEMM epilogue scales G and U by r.
// (The GEMV path computes r inside its gate/up kernel instead.)
#pragma once

#include "common.hpp"

namespace gmlp {

constexpr int kRowRmsThreads = 256; // one row
constexpr int kRowRmsBlocks = 1 << 20; // at most, each taking rows in turn
constexpr int kRowRmsChunks = 4;    // 16-byte chunks per thread in flight: rows of up to 8192 columns in one pass

// r[t] = 1 / sqrt(sum_d X[t, d]^2 / D + eps), X [T, D] bf16, D a multiple of
// 8.  Each thread adds its 8-element chunks in order, then a butterfly over
// the wave and the waves' sums in order (an order fixed by D alone).
//
// The rows are few and short, so this is latency, not bandwidth: a block per
// row with all of a thread's loads in flight at once.  A wave per row, whose
// loads waited for one another, took 7.8 us at T = 300, D = 5120 (75 blocks);
// this takes 4.0-5.2 (launch and one trip to memory).
__global__ __launch_bounds__(kRowRmsThreads) void row_rms_kernel(const uint16_t *X, float *r, int T, int D,
                                                                 float eps)
{
    __shared__ float part[kRowRmsThreads / 64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nchunk = D >> 3;
    for (int t = blockIdx.x; t < T; t += gridDim.x) {
        const uint16_t *x = X + (size_t)t * D;
        float s = 0.0f;
        for (int c0 = 0; c0 < nchunk; c0 += kRowRmsThreads * kRowRmsChunks) {
            u32x4 v[kRowRmsChunks];
#pragma unroll
            for (int j = 0; j < kRowRmsChunks; ++j) {
                const int c = c0 + kRowRmsThreads * j + tid;
                v[j] = *(const u32x4 *)(x + 8 * (c < nchunk ? c : nchunk - 1)); // past the row: loaded, not added
            }
#pragma unroll
            for (int j = 0; j < kRowRmsChunks; ++j)
                if (c0 + kRowRmsThreads * j + tid < nchunk)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = bf16_lo(v[j][e]), hi = bf16_hi(v[j][e]);
                        s += lo * lo;
                        s += hi * hi;
                    }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            s += __shfl_xor(s, off);
        if (lane == 0)
            part[wave] = s;
        __syncthreads();
        if (tid == 0) {
            float sum = part[0];
#pragma unroll
            for (int w = 1; w < kRowRmsThreads / 64; ++w)
                sum += part[w];
            r[t] = 1.0f / __builtin_sqrtf(sum / (float)D + eps);
        }
        __syncthreads(); // part is written again for the next row
    }
}

} // namespace gmlp
