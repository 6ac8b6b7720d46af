// Random projection of a token map (paper, Sec. "Random Projection (RP) for Low-Rank Feature"):
//
//     out[b] = Q^T X[b],   Q^T given as qt[rows][M],  X[b]:[M][d]  ->  out[b]:[rows][d]
//
// used with rows = r on the block input (Alg. "FasterVAR": F^_r = Q^T F~) and on the cached
// counterpart feature (G_c = Q^T C).  bf16 runs on the tiled MFMA kernel of the linear layers, X as its
// k-major operand (launch_gemm_bf16_kmajor); the plain kernel below is the fp32 path.
#include "common.h"

namespace fvar {

// Eight output rows per workgroup, one column per thread, fp64 sums: fp32 storage (parity configuration),
// and bf16 maps of 2^25 tokens and more, whose rows the tiled kernel's 32-bit offsets do not span.
template <typename T>
__global__ __launch_bounds__(256) void rp_project_kernel(const T *__restrict__ qt, size_t q_stride,
                                                         const T *__restrict__ x, int M, int rows, int d,
                                                         T *__restrict__ out)
{
    const int b = blockIdx.z, t0 = blockIdx.y * 8;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= d) return;
    const T *Q = qt + (size_t)b * q_stride;
    const T *X = x + (size_t)b * M * d;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = 0; i < M; ++i) {
        const double xv = Elem<T>::load(X + (size_t)i * d + j);
#pragma unroll
        for (int t = 0; t < 8; ++t)
            acc[t] = fma((double)Elem<T>::load(Q + (size_t)min(t0 + t, rows - 1) * M + i), xv, acc[t]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t0 + t < rows) Elem<T>::store(out + ((size_t)b * rows + t0 + t) * d + j, (float)acc[t]);
}

void launch_rp_project(DType dt, const void *qt, size_t q_stride, const void *x, int B, int M,
                       int rows, int d, void *out, hipStream_t st)
{
    const dim3 grid((d + 255) / 256, (rows + 7) / 8, B);
    if (dt != DType::BF16)
        launch(rp_project_kernel<float>, grid, dim3(256), 0, st, (const float *)qt, q_stride, (const float *)x,
               M, rows, d, (float *)out);
    else if (!launch_gemm_bf16_kmajor(qt, q_stride, x, B, M, rows, d, out, st))
        launch(rp_project_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t *)qt, q_stride,
               (const uint16_t *)x, M, rows, d, (uint16_t *)out);
}

}  // namespace fvar
