// Restoration matrix of the cached counterpart feature by linear least squares (paper, Eq.
// "lstsq" with the cached feature in place of the input, App. "Construction of W_r^o"):
//
//     W_c = argmin_W || W G_c - C ||_F = (C G_c^T) (G_c G_c^T)^{-1},     G_c = Q^T C  as stored.
//
// Four kernels per call (the projection G_c itself is the kernel of rp.hip):
//   T = C G_c^T   [M,r]  fp32; bf16 inputs on the tiled MFMA kernel of the linear layers, the second pass over C
//                 (bf16: with S^{-1} in the same launch)
//   gram_kernel   S = G_c G_c^T          [r,r]  fp64 (bf16: MFMA per 64-element chunk, fp64 across)
//   spd_inverse   S^{-1}                 block sweep in registers, one workgroup per sample, fp64 MFMA
//   w_kernel      W_c = T S^{-1}         [M,r]  fp64 MFMA, rounded to the storage type
#include "common.h"
#include "spd_inverse.h"

namespace fvar {

// ------------------------------------------------------------------ T = C G^T
// fp32 storage: one row of C per workgroup, fp64 accumulation
__global__ __launch_bounds__(256) void t_f32_kernel(const float *__restrict__ cache,
                                                    const float *__restrict__ g_c, int M, int r, int d,
                                                    float *__restrict__ T)
{
    const int b = blockIdx.y, i = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float *crow = cache + ((size_t)b * M + i) * d;
    const float *G = g_c + (size_t)b * r * d;
    for (int t = wave; t < r; t += 4) {
        double acc = 0.0;
        for (int j = lane; j < d; j += 64) acc = fma((double)crow[j], (double)G[(size_t)t * d + j], acc);
        acc = wave_sum(acc);
        if (lane == 0) T[((size_t)b * M + i) * r + t] = (float)acc;
    }
}

// ------------------------------------------------------------------ S = G G^T
// fp32 storage: one workgroup of 16 wavefronts per (sample, row a); the row is parked in LDS,
// each wavefront takes columns c = wave, wave+16, ... <= a, fp64 products and sums.
constexpr int kGramThreads = 1024;
__global__ __launch_bounds__(kGramThreads) void gram_f32_kernel(const float *__restrict__ g_c, int r,
                                                                int d, double *__restrict__ S)
{
    extern __shared__ float rowa[];                 // [d]
    const int b = blockIdx.y, a = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float *G = g_c + (size_t)b * r * d;
    for (int j = threadIdx.x; j < d; j += kGramThreads) rowa[j] = G[(size_t)a * d + j];
    __syncthreads();
    double *Sb = S + (size_t)b * r * r;
    for (int c = wave; c <= a; c += kGramThreads / 64) {
        double acc = 0.0;
        for (int j = lane; j < d; j += 64) acc = fma((double)G[(size_t)c * d + j], (double)rowa[j], acc);
        acc = wave_sum(acc);
        if (lane == 0) {
            Sb[(size_t)a * r + c] = acc;
            Sb[(size_t)c * r + a] = acc;
        }
    }
}

// bf16 storage, on MFMA.  A workgroup owns one 32x32 tile (ti >= tj) of S for one slice of the
// contraction axis: the 64-element chunks c = part, part + parts, ... are dealt round-robin to its
// four wavefronts.  Within a chunk the products (exact in fp32) are summed in fp32; chunk results
// are added in fp64.  The slices' partial matrices are written to Spart[b][part] (both triangles)
// and summed by the inverse, so the result does not depend on scheduling.  The inverse reads them through one
// CU, so fewer is better there (128 KB each at rank 128).  The whole call in two, four and eight slices: 94.3, 96.5 and
// 105.1 us at rank 128, 4 x 4096 rows of 4096, 235, 233 and 239 for 40 x 1024, 68.8, 67.6 and 67.0 at rank 64.
// The chunks come by DMA in whole 128-byte lines, two in flight per wavefront (a row per lane is a quarter of the
// vector L1's rate, see gemm_rows_kernel): rank 128, 4 samples of width 4096 6.5 -> 4.9 us, 40 of them 35.4 -> 28.5.
// Chunks past the end are not fetched: where a wavefront has one, as with d = 1024, those in their place tripled
// its reads (512 samples, rank 32: 17.7 -> 13.6 us; 480 x 1920: 26.3 -> 18.1).
__global__ __launch_bounds__(256) void gram_bf16_kernel(const uint16_t *__restrict__ g_c, int r, int d,
                                                        double *__restrict__ Spart)
{
    extern __shared__ uint4 gram_lds[];              // [wavefront][stage][64 rows of 128 bytes], then the partial tiles
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rl = lane & 31, g = lane >> 5;
    int ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
    const int tj = blockIdx.x - ti * (ti + 1) / 2;
    const int part = blockIdx.y, parts = gridDim.y, b = blockIdx.z;
    const uint16_t *G = g_c + (size_t)b * r * d;
    double acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0;
    const int nchunks = d / 64, step = parts * 4, c0 = part + parts * wave;
    const int n = c0 < nchunks ? (nchunks - 1 - c0) / step + 1 : 0;
    const uint32_t ring = (uint32_t)(uintptr_t)gram_lds + wave * 16384;
    const uint4 *mine = gram_lds + wave * 1024;
    // chunk i of this wavefront, 8 rows (1 KiB) per instruction: lane l fills physical chunk l%8 of row l/8 with the
    // logical chunk that the swizzle (chunk ^ row/2 % 8) maps there
    auto fetch = [&](int i) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int lrow = (u & 3) * 8 + lane / 8, row = min((u < 4 ? ti : tj) * 32 + lrow, r - 1);
            const uint16_t *src = G + (size_t)row * d + (c0 + i * step) * 64 + (((lane & 7) ^ ((lrow >> 1) & 7)) << 3);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(ring + (i & 1) * 8192 + u * 1024), "v"(src) : "memory", "m0");
        }
    };
    if (n > 0) fetch(0);
    if (n > 1) fetch(1);
    for (int i = 0; i < n; ++i) {
        if (i + 1 < n) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        uint4 av[4], bv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint4 *src = mine + (i & 1) * 512 + rl * 8 + ((2 * s + g) ^ ((rl >> 1) & 7));
            av[s] = src[0];
            bv[s] = src[256];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the stage is free
        if (i + 2 < n) fetch(i + 2);
        floatx16_t a32 = {0};
#pragma unroll
        for (int s = 0; s < 4; ++s)
            a32 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av[s]),
                                                          __builtin_bit_cast(bf16x8_t, bv[s]), a32, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] += (double)a32[e];
    }
    double *red = reinterpret_cast<double *>(gram_lds);              // every wavefront's tile in its own ring
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave * 2048 + (8 * (e >> 2) + 4 * g + (e & 3)) * 32 + rl] = acc[e];
    __syncthreads();
    double *Sb = Spart + ((size_t)b * parts + part) * r * r;
    for (int idx = tid; idx < 32 * 32; idx += 256) {
        const int i = ti * 32 + idx / 32, j = tj * 32 + idx % 32;
        const double v = (red[idx] + red[2048 + idx]) + (red[4096 + idx] + red[6144 + idx]);
        if (i < r && j < r) {
            Sb[(size_t)i * r + j] = v;
            if (ti != tj) Sb[(size_t)j * r + i] = v;
        }
    }
}

// ------------------------------------------------------------------ S^{-1}
// fp32 storage: one workgroup per sample, see spd_inverse; in bf16 the launch of T does this too
template <int NB, int NW>
__global__ __launch_bounds__(64 * NW) void spd_inverse_kernel(const double *__restrict__ S, int parts, int r,
                                                              double ridge, double *__restrict__ Sinv)
{
    extern __shared__ double inverse_lds[];
    const size_t b = blockIdx.x;
    spd_inverse<NB, NW>(S + b * parts * r * r, parts, r, ridge, Sinv + b * r * r, inverse_lds);
}

// ------------------------------------------------------------------ W = T S^{-1}
// On the fp64 MFMA (16x16x4).  Workgroup = 64 rows of T, 16 per wavefront; S^{-1} is staged in LDS, zero
// padded to 16*CT in both directions, its pitch such that the rows of the four k-slots fall on
// different banks.  A lane takes 4 consecutive entries of its row of T (the sum of its up to four
// shares) as the k-slots of four MFMAs.  4*CT*CT MFMAs of 64 clk per wavefront are 7 of the 17 us below
// (pipes busy 0.27 of the clocks; the wavefronts wait 0.41 of their time, 0.19 of the LDS cycles are conflicts).  Rank 128, 4 x 4096 rows: 76 us with fp64 FMAs fed by LDS broadcasts -> 17 us.
template <typename TT, int CT>
__global__ __launch_bounds__(256) void w_kernel(const float *__restrict__ T, int t_parts,
                                                size_t t_part_stride,
                                                const double *__restrict__ Sinv, int M, int r,
                                                TT *__restrict__ w_c)
{
    extern __shared__ double Si[];
    constexpr int RP = 16 * CT, PITCH = RP + 4;
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    const double *Sg = Sinv + (size_t)b * r * r;
    const int row0 = blockIdx.x * 64 + 16 * wave;
    const float *trow = T + ((size_t)b * M + min(row0 + c, M - 1)) * r + 4 * g;   // r is a multiple of 4
    float4 tv[CT];                                 // this lane's share of its row, in flight under the staging
#pragma unroll
    for (int i = 0; i < CT; ++i) {
        tv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (16 * i + 4 * g < r) {
            tv[i] = *reinterpret_cast<const float4 *>(trow + 16 * i);
            for (int p = 1; p < t_parts; ++p) {    // the other shares of the contraction axis
                const float4 tp = *reinterpret_cast<const float4 *>(trow + p * t_part_stride + 16 * i);
                tv[i].x += tp.x; tv[i].y += tp.y; tv[i].z += tp.z; tv[i].w += tp.w;
            }
        }
    }
    // S^{-1} to LDS, CT pairs per thread in flight (r is even)
    const double2 *Sg2 = reinterpret_cast<const double2 *>(Sg);
#pragma unroll 1
    for (int base = tid; base < RP * RP / 2; base += 256 * CT) {
        double2 v[CT];
#pragma unroll
        for (int u = 0; u < CT; ++u) {
            const int i = (base + 256 * u) / (RP / 2), j = (base + 256 * u) % (RP / 2);
            v[u] = i < r && 2 * j < r ? Sg2[((size_t)i * r >> 1) + j] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < CT; ++u) {
            const int i = (base + 256 * u) / (RP / 2), j = (base + 256 * u) % (RP / 2);
            *reinterpret_cast<double2 *>(Si + i * PITCH + 2 * j) = v[u];
        }
    }
    __syncthreads();
    doublex4_t acc[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[t] = doublex4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double td = (double)(u == 0 ? tv[i].x : u == 1 ? tv[i].y : u == 2 ? tv[i].z : tv[i].w);
            const double *sr = Si + (16 * i + 4 * g + u) * PITCH + c;
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(td, sr[16 * t], acc[t], 0, 0, 0);
        }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = row0 + 4 * e + g;
        if (row >= M) continue;
        TT *out = w_c + ((size_t)b * M + row) * r;
#pragma unroll
        for (int t = 0; t < CT; ++t)
            if (16 * t + c < r) Elem<TT>::store(out + 16 * t + c, (float)acc[t][e]);
    }
}

// shares of the contraction axis that T comes in; the kernel that consumes T sums them
int factor_t_parts(DType dt, int B, int M, int r, int d)
{
    return dt == DType::BF16 ? batched_f32_parts(B, M, r, d) : 1;
}

// rows of T, over all shares, that the workspace has room for
size_t factor_t_room(DType dt, int B, int M, int d)
{
    return dt == DType::BF16 ? batched_f32_room(B, M, d) : (size_t)B * M;
}

void launch_factor_gram(DType dt, const void *g_c, int B, int r, int d, double *S, hipStream_t st)
{
    if (dt == DType::BF16) {
        const int rt = (r + 31) / 32;
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(gram_bf16_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 65536);
        launch(gram_bf16_kernel, dim3(rt * (rt + 1) / 2, kGramParts, B), dim3(256), 65536, st,
               (const uint16_t *)g_c, r, d, S);
    } else {
        launch(gram_f32_kernel, dim3(r, B), dim3(kGramThreads), (size_t)d * sizeof(float), st,
               (const float *)g_c, r, d, S);
    }
}

// Gram matrices that the workspace has room for: eight in bf16, which is what callers have been told, of
// which kGramParts are used
int gram_room(DType dt) { return dt == DType::BF16 ? 8 : 1; }

// Sinv[b] = inverse of the sum of the `parts` matrices of S[b] (+ ridge), in a launch of its own
void launch_factor_inverse(const double *S, int parts, int B, int r, double ridge, double *Sinv,
                           hipStream_t st)
{
#define FVAR_INVERSE(NB, NW)                                                                       \
    do {                                                                                           \
        auto kern = spd_inverse_kernel<NB, NW>;                                                    \
        constexpr size_t lds = spd_inverse_lds(NB);                                                \
        if (lds > 48 * 1024)                                                                       \
            (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                        \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);       \
        launch(kern, dim3(B), dim3(64 * NW), lds, st, S, parts, r, ridge, Sinv);                   \
    } while (0)
    if (r <= 32) FVAR_INVERSE(2, 4);
    else if (r <= 64) FVAR_INVERSE(4, 8);
    else FVAR_INVERSE(8, 8);
#undef FVAR_INVERSE
}

// bf16: T, an ordinary linear layer per sample in fp32, and the inverse of S, which does not need it, in one launch
void launch_factor_t_inverse(const void *cache, const void *g_c, int B, int M, int r, int d, float *T,
                             const double *S, double ridge, double *Sinv, hipStream_t st)
{
    launch_gemm_bf16_batched_f32(cache, g_c, B, M, r, d, T, InverseJob{S, ridge, Sinv, r}, st);
}

void launch_factor_t_f32(const void *cache, const void *g_c, int B, int M, int r, int d, float *T, hipStream_t st)
{
    launch(t_f32_kernel, dim3(M, B), dim3(256), 0, st, (const float *)cache, (const float *)g_c, M, r, d, T);
}

template <typename TT>
static void launch_w_t(const float *T, int t_parts, const double *Sinv, int B, int M, int r, void *w_c,
                       hipStream_t st)
{
    const size_t t_stride = (size_t)B * M * r;
    const dim3 grid((M + 63) / 64, B);
#define FVAR_W(CT)                                                                                 \
    do {                                                                                           \
        const size_t lds = (size_t)16 * CT * (16 * CT + 4) * sizeof(double);                       \
        auto kern = w_kernel<TT, CT>;                                                              \
        if (lds > 48 * 1024)                                                                       \
            (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                        \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);       \
        launch(kern, grid, dim3(256), lds, st, T, t_parts, t_stride, Sinv, M, r, (TT *)w_c);       \
    } while (0)
    if (r <= 32) FVAR_W(2);
    else if (r <= 64) FVAR_W(4);
    else if (r <= 96) FVAR_W(6);
    else FVAR_W(8);
#undef FVAR_W
}

void launch_factor_w(DType dt, const float *T, const double *Sinv, int B, int M, int r, int d, void *w_c,
                     hipStream_t st)
{
    const int tp = factor_t_parts(dt, B, M, r, d);
    if (dt == DType::BF16) launch_w_t<uint16_t>(T, tp, Sinv, B, M, r, w_c, st);
    else launch_w_t<float>(T, tp, Sinv, B, M, r, w_c, st);
}

}  // namespace fvar
