// Row pass: (M,d) -> (k,d) gather of the kept token rows, fused with the LayerNorm that opens
// the block (paper, Sec. "Plug-and-Play Acceleration": the block sees k rows instead of M).
// One wavefront per output row; the row lives in registers between the statistics and the
// normalisation, every global access is a 16-byte chunk and a row is read exactly once.
#include "common.h"

namespace fvar {

// gamma and beta are fetched a batch of chunks at a time, the first of them while the row's statistics are under
// way.  Loaded one by one where they were used, behind a branch each, they were a chain of 2*CH trips to memory
// at the end of the kernel.  Gather and fp32 stream, us before -> now: 1848 rows of 1920 9.8 -> 7.9 and
// 11.8 -> 6.9, 300 of 4096 10.7 -> 6.4 and 16.0 -> 7.3, 6400 of 4096 39 -> 35 and 44 -> 33, 120 of 1024 4.6 -> 3.8
// and 5.5 -> 3.5.  Four 16-byte or eight 8-byte chunks a batch: with eight of 16 bytes the registers leave two
// wavefronts per SIMD at 4096 columns (39 us for 6400 rows), with two the last batches wait again (6.8 and 8.8
// for 300 rows).  At 8192 columns the eight of 8 bytes take two registers too many for two wavefronts per SIMD; four
// would not: whole blocks are 1 % slower with four up to 512 rows, 0.5 % faster at 1600, the same at 4096.
constexpr int kAffineGather = 4, kAffineStream = 8;

// CH = 16-byte chunks per lane (row length <= 64 * CH chunks); AFFINE: gamma or beta or both are there
template <typename T, int CH, bool AFFINE>
__global__ __launch_bounds__(256) void gather_ln_kernel(const T *__restrict__ x,
                                                        const int32_t *__restrict__ idx, int M, int n,
                                                        int total_rows, int d,
                                                        const T *__restrict__ gamma,
                                                        const T *__restrict__ beta, float eps,
                                                        T *__restrict__ copy_out,
                                                        T *__restrict__ ln_out)
{
    constexpr int E = Elem<T>::kPerChunk;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;          // output row in [0, B*n)
    if (row >= total_rows) return;
    const int b = row / n;
    const int src_row = idx ? idx[row] : (row - b * n);
    const uint4 *src = reinterpret_cast<const uint4 *>(x + ((size_t)b * M + src_row) * d);
    const int nchunk = d / E;

    uint4 raw[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        int ci = lane + 64 * c;
        raw[c] = ci < nchunk ? src[ci] : make_uint4(0, 0, 0, 0);
    }
    constexpr int AB = CH < kAffineGather ? CH : kAffineGather;
    uint4 gb[AFFINE ? AB : 1], bb[AFFINE ? AB : 1];
    auto load_affine = [&](int c0) {
#pragma unroll
        for (int c = 0; c < AB; ++c) {
            const int ci = min(lane + 64 * (c0 + c), nchunk - 1);
            if (gamma) gb[c] = reinterpret_cast<const uint4 *>(gamma)[ci];
            if (beta) bb[c] = reinterpret_cast<const uint4 *>(beta)[ci];
        }
    };
    if (AFFINE && ln_out) load_affine(0);
    if (copy_out) {
        uint4 *dst = reinterpret_cast<uint4 *>(copy_out + (size_t)row * d);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            int ci = lane + 64 * c;
            if (ci < nchunk) dst[ci] = raw[c];
        }
    }
    if (!ln_out) return;

    float v[CH][E];
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        Elem<T>::unpack(raw[c], v[c]);
#pragma unroll
        for (int e = 0; e < E; ++e) sum += v[c][e];        // padded chunks hold zeros
    }
    const float mu = wave_sum(sum) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const bool in = lane + 64 * c < nchunk;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float t = v[c][e] - mu;
            v[c][e] = t;
            sq += in ? t * t : 0.f;
        }
    }
    const float rstd = rsqrtf(wave_sum(sq) / (float)d + eps);

    uint4 *dst = reinterpret_cast<uint4 *>(ln_out + (size_t)row * d);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (AFFINE && c > 0 && c % AB == 0) load_affine(c);
        int ci = lane + 64 * c;
        float o[E];
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] = v[c][e] * rstd;
        if (AFFINE && gamma) {
            float g[E];
            Elem<T>::unpack(gb[c % AB], g);
#pragma unroll
            for (int e = 0; e < E; ++e) o[e] *= g[e];
        }
        if (AFFINE && beta) {
            float bt[E];
            Elem<T>::unpack(bb[c % AB], bt);
#pragma unroll
            for (int e = 0; e < E; ++e) o[e] += bt[e];
        }
        if (ci < nchunk) dst[ci] = Elem<T>::pack(o);
    }
}

// LayerNorm of the fp32 intermediate residual stream into the bf16 operand of the MLP.
// One wavefront per row; CH = 16-byte (4 float) chunks per lane.
template <int CH, bool AFFINE>
__global__ __launch_bounds__(256) void ln_f32_to_bf16_kernel(const float *__restrict__ h, int rows,
                                                             int d,
                                                             const uint16_t *__restrict__ gamma,
                                                             const uint16_t *__restrict__ beta,
                                                             float eps, uint16_t *__restrict__ out)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const uint4 *src = reinterpret_cast<const uint4 *>(h + (size_t)row * d);
    const int nchunk = d / 4;
    uint4 raw[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int ci = lane + 64 * c;
        raw[c] = ci < nchunk ? src[ci] : make_uint4(0, 0, 0, 0);
    }
    constexpr int AB = CH < kAffineStream ? CH : kAffineStream;
    uint2 gb[AFFINE ? AB : 1], bb[AFFINE ? AB : 1];
    auto load_affine = [&](int c0) {
#pragma unroll
        for (int c = 0; c < AB; ++c) {
            const int ci = min(lane + 64 * (c0 + c), nchunk - 1);
            if (gamma) gb[c] = reinterpret_cast<const uint2 *>(gamma)[ci];
            if (beta) bb[c] = reinterpret_cast<const uint2 *>(beta)[ci];
        }
    };
    if (AFFINE) load_affine(0);
    float v[CH][4];
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        Elem<float>::unpack(raw[c], v[c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += v[c][e];
    }
    const float mu = wave_sum(sum) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const bool in = lane + 64 * c < nchunk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float t = v[c][e] - mu;
            v[c][e] = t;
            sq += in ? t * t : 0.f;
        }
    }
    const float rstd = rsqrtf(wave_sum(sq) / (float)d + eps);
    uint2 *dst = reinterpret_cast<uint2 *>(out + (size_t)row * d);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (AFFINE && c > 0 && c % AB == 0) load_affine(c);
        const int ci = lane + 64 * c;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = v[c][e] * rstd;
        if (AFFINE && gamma) {
            const uint2 gv = gb[c % AB];
            o[0] *= bf16_lo(gv.x); o[1] *= bf16_hi(gv.x); o[2] *= bf16_lo(gv.y); o[3] *= bf16_hi(gv.y);
        }
        if (AFFINE && beta) {
            const uint2 bv = bb[c % AB];
            o[0] += bf16_lo(bv.x); o[1] += bf16_hi(bv.x); o[2] += bf16_lo(bv.y); o[3] += bf16_hi(bv.y);
        }
        if (ci < nchunk) dst[ci] = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
    }
}

void launch_ln_f32_to_bf16(const float *h, int rows, int d, const void *gamma, const void *beta,
                           float eps, void *ln_out, hipStream_t st)
{
    const int ch = (d / 4 + 63) / 64;
    dim3 grid((rows + 3) / 4), block(256);
#define FVAR_LN32(CH)                                                                          \
    launch(gamma || beta ? ln_f32_to_bf16_kernel<CH, true> : ln_f32_to_bf16_kernel<CH, false>,  \
           grid, block, 0, st, h, rows, d, (const uint16_t *)gamma, (const uint16_t *)beta, eps, \
           (uint16_t *)ln_out)
    if (ch <= 4) FVAR_LN32(4);
    else if (ch <= 8) FVAR_LN32(8);
    else if (ch <= 16) FVAR_LN32(16);
    else FVAR_LN32(32);
#undef FVAR_LN32
}

template <typename T>
static void launch_gather_ln_t(const void *x, const int32_t *idx, int B, int M, int n, int d,
                               const void *gamma, const void *beta, float eps, void *copy_out,
                               void *ln_out, hipStream_t st)
{
    const int total = B * n;
    const int nchunk = d / Elem<T>::kPerChunk;
    const int ch = (nchunk + 63) / 64;
    dim3 grid((total + 3) / 4), block(256);
#define FVAR_GLN(CH)                                                                             \
    launch(gamma || beta ? gather_ln_kernel<T, CH, true> : gather_ln_kernel<T, CH, false>,       \
                       grid, block, 0, st, (const T *)x, idx, M, n,                              \
                       total, d, (const T *)gamma, (const T *)beta, eps, (T *)copy_out,           \
                       (T *)ln_out)
    if (ch <= 2) FVAR_GLN(2);
    else if (ch <= 4) FVAR_GLN(4);
    else if (ch <= 8) FVAR_GLN(8);
    else FVAR_GLN(16);
#undef FVAR_GLN
}

void launch_gather_ln(DType dt, const void *x, const int32_t *idx, int B, int M, int n, int d,
                      const void *gamma, const void *beta, float eps, void *copy_out, void *ln_out,
                      hipStream_t st)
{
    if (dt == DType::BF16)
        launch_gather_ln_t<uint16_t>(x, idx, B, M, n, d, gamma, beta, eps, copy_out, ln_out, st);
    else
        launch_gather_ln_t<float>(x, idx, B, M, n, d, gamma, beta, eps, copy_out, ln_out, st);
}

}  // namespace fvar
