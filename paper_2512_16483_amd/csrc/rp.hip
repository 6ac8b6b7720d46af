// Random projection of a token map (paper, Sec. "Random Projection (RP) for Low-Rank Feature"):
//
//     out[b] = Q^T X[b],   Q^T given as qt[rows][M],  X[b]:[M][d]  ->  out[b]:[rows][d]
//
// used with rows = r on the block input (Alg. "FasterVAR": F^_r = Q^T F~) and on the cached
// counterpart feature (G_c = Q^T C).  bf16 runs on the tiled MFMA kernel of the linear layers, X as its
// k-major operand (launch_gemm_bf16_kmajor); the plain kernel below is for fp32.
#include "common.h"

namespace fvar {

// fp32 storage (parity configuration): eight output rows per workgroup, one column per thread, fp64 sums
__global__ __launch_bounds__(256) void rp_project_f32_kernel(const float *__restrict__ qt, size_t q_stride,
                                                             const float *__restrict__ x, int M, int rows, int d,
                                                             float *__restrict__ out)
{
    const int b = blockIdx.z, t0 = blockIdx.y * 8;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= d) return;
    const float *Q = qt + (size_t)b * q_stride;
    const float *X = x + (size_t)b * M * d;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = 0; i < M; ++i) {
        const double xv = X[(size_t)i * d + j];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = fma((double)Q[(size_t)min(t0 + t, rows - 1) * M + i], xv, acc[t]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t0 + t < rows) out[((size_t)b * rows + t0 + t) * d + j] = (float)acc[t];
}

void launch_rp_project(DType dt, const void *qt, size_t q_stride, const void *x, int B, int M,
                       int rows, int d, void *out, hipStream_t st)
{
    if (dt == DType::BF16) launch_gemm_bf16_kmajor(qt, q_stride, x, B, M, rows, d, out, st);
    else
        launch(rp_project_f32_kernel, dim3((d + 255) / 256, (rows + 7) / 8, B), dim3(256), 0, st, (const float *)qt,
               q_stride, (const float *)x, M, rows, d, (float *)out);
}

}  // namespace fvar
