// Restoration matrix of the cached counterpart feature by linear least squares (paper, Eq.
// "lstsq" with the cached feature in place of the input, App. "Construction of W_r^o"):
//
//     W_c = argmin_W || W G_c - C ||_F = (C G_c^T) (G_c G_c^T)^{-1},     G_c = Q^T C  as stored.
//
// Four kernels per call (the projection G_c itself is the kernel of rp.hip):
//   T = C G_c^T   [M,r]  fp32; bf16 inputs on the tiled MFMA kernel of the linear layers, the second pass over C
//   gram_kernel   S = G_c G_c^T          [r,r]  fp64 (bf16: MFMA per 64-element chunk, fp64 across)
//   spd_inverse   S^{-1}                 block sweep in registers, one workgroup per sample, fp64 MFMA
//   w_kernel      W_c = T S^{-1}         [M,r]  fp64 MFMA, rounded to the storage type
#include "common.h"

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
// and summed by the factorisation kernel, so the result does not depend on scheduling.
constexpr int kGramParts = 8;
__global__ __launch_bounds__(256) void gram_bf16_kernel(const uint16_t *__restrict__ g_c, int r, int d,
                                                        double *__restrict__ Spart)
{
    __shared__ double red[4][32 * 32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int rl = lane & 31, g = lane >> 5;
    int ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
    const int tj = blockIdx.x - ti * (ti + 1) / 2;
    const int part = blockIdx.y, parts = gridDim.y, b = blockIdx.z;
    const uint16_t *G = g_c + (size_t)b * r * d;
    const uint16_t *arow = G + (size_t)min(ti * 32 + rl, r - 1) * d;
    const uint16_t *brow = G + (size_t)min(tj * 32 + rl, r - 1) * d;
    double acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0;
    const int nchunks = d / 64;
    for (int c = part + parts * wave; c < nchunks; c += parts * 4) {
        floatx16_t a32 = {0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int t = c * 64 + 16 * s + 8 * g;
            const uint4 av = *reinterpret_cast<const uint4 *>(arow + t);
            const uint4 bv = *reinterpret_cast<const uint4 *>(brow + t);
            a32 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av),
                                                          __builtin_bit_cast(bf16x8_t, bv), a32, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] += (double)a32[e];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][(8 * (e >> 2) + 4 * g + (e & 3)) * 32 + rl] = acc[e];
    __syncthreads();
    double *Sb = Spart + ((size_t)b * parts + part) * r * r;
    for (int idx = tid; idx < 32 * 32; idx += 256) {
        const int i = ti * 32 + idx / 32, j = tj * 32 + idx % 32;
        const double v = (red[0][idx] + red[1][idx]) + (red[2][idx] + red[3][idx]);
        if (i < r && j < r) {
            Sb[(size_t)i * r + j] = v;
            if (ti != tj) Sb[(size_t)j * r + i] = v;
        }
    }
}

// ------------------------------------------------------------------ S^{-1}
typedef double doublex4_t __attribute__((ext_vector_type(4)));

// value of lane P of each 16-lane row, in every lane of the row
template <int P> __device__ __forceinline__ double row_bcast(double v)
{
    const long w = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(long, v), 0x150 + P, 0xf, 0xf, true);
    return __builtin_bit_cast(double, w);
}

// Sweep step P of the symmetric 16x16 pivot block `a` and the same row operations on NT further 16-column
// tiles `b` of its rows, all held by one wavefront in the fp64 MFMA's output layout: entry e of lane
// (c, g) = (lane % 16, lane / 16) is row 4e + g, column c.  With d the pivot and u its row of a,
//     a_ik -> a_ik - u_i u_k / d,   a_iP, a_Pi -> u_i / d,   a_PP -> -1 / d,
//     b_i -> b_i - u_i b_P / d,     b_P -> b_P / d.
// The two triangles of a stay equal to the bit (the product u_i u_k is rounded first): where they drift
// apart, T S^-1 loses four digits at condition 4e6.  b_P as it was goes to y[.][P] of its column, divided
// by d to ys[.][P] (from the four lanes that hold it alike).
template <int P, int NT>
__device__ __forceinline__ void sweep_step(doublex4_t &a, doublex4_t (&b)[NT], double (*y)[17],
                                           double (*ys)[17], int c, int g)
{
    const double row = __shfl(a[P >> 2], 16 * (P & 3) + c);          // u at this lane's column
    double brow[NT], bs[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) brow[t] = __shfl(b[t][P >> 2], 16 * (P & 3) + c);
    const double piv = row_bcast<P>(row);
    double inv = __builtin_amdgcn_rcp(piv);                          // ~1e-8, two Newton steps to full precision
    inv = fma(inv, fma(-piv, inv, 1.0), inv);
    inv = fma(inv, fma(-piv, inv, 1.0), inv);
    const double x = c == P ? -1.0 : row, xs = x * inv;
#pragma unroll
    for (int t = 0; t < NT; ++t) { bs[t] = brow[t] * inv; y[16 * t + c][P] = brow[t]; ys[16 * t + c][P] = bs[t]; }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double col = row_bcast<P>(a[e]);                       // u at this entry's row
        const double v = fma(-(col * x), inv, c == P ? 0.0 : a[e]);
        const bool pivot = e == (P >> 2) && g == (P & 3);
        a[e] = pivot ? xs : v;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const double w = fma(-col, bs[t], b[t][e]);
            b[t][e] = pivot ? bs[t] : w;
            // computed here: put off to the branch that stores them, they keep col and bs of all steps in
            // registers
            asm volatile("" : "+v"(b[t][e]));
        }
    }
}

// One workgroup per sample inverts the symmetric positive definite Gram matrix (the sum of the
// `parts` partial matrices, plus ridge * trace / r on the diagonal) in fp64, without pivoting, by the
// symmetric sweep (see sweep_step), which leaves -S^-1 after all pivots.  They are taken 16 at a time
// (block j): sixteen steps are applied one by one to the pivot block and to its tile row
// A_jk = U_k^T, and the rank-16 update of all the other tiles, A_ik -= sum_p (u_ip / d_p) u_kp, is made
// from the u and d that the steps met.  Those are the scalar sweep's own operations in another order.
// U P^-1 U^T from an explicit inverse of the pivot block is not the same: it loses the square of the
// condition number where the sweep loses it once (condition 4e6: the inverse off by 4e-6 instead of
// 5e-11, T S^-1 of a rank-8 cache with ridge 1e-6 wrong altogether).
// The matrix is padded to 16*NB with an identity block and stays in registers as 16x16 tiles in the fp64
// MFMA's output layout, NB/2 tiles of one tile row per wavefront.  The first wavefronts apply the steps,
// each to one or two tiles of the row and all to a copy of the pivot block; only the tile column, u and
// u / d go through LDS, three barriers per block.  Steps of the padding are left out.
// Bound by the chain of steps, 0.5 us each.  Rank 128, 4 samples, by itself: 63 us (eight wavefronts with one
// tile each 68, with exchanges by permlane swaps instead of shuffles 73); one thread per half row, a barrier
// per pivot and 64 unrolled steps of code that do not fit the instruction cache took 758.  Ranks 8, 16, 24 and
// 32: 5.4, 6.3, 8.4 and 9.3 us, before 6.7, 8.3, 11.3 and 13.7.
// A singular matrix yields non-finite output.
template <int NB>
__global__ __launch_bounds__(128 * NB) void spd_inverse_kernel(const double *__restrict__ S, int parts,
                                                               int r, double ridge,
                                                               double *__restrict__ Sinv)
{
    constexpr int TPW = NB / 2, NW = 2 * NB;
    // U: the tile column (then, tile by tile, the swept one); Y, Ys: u and u / d
    __shared__ double U[16 * NB][17], Y[16 * NB][17], Ys[16 * NB][17];
    __shared__ double Pi[16][17], red[NW];
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4, b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ti = wave >> 1, tk0 = (wave & 1) * TPW;                // tile row, first tile column
    const double *Sb = S + (size_t)b * parts * r * r;
    doublex4_t a[TPW];
    double tr = 0.0;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * ti + 4 * e + g, col = 16 * (tk0 + t) + c;
            // the parts' loads travel together (inside a call, where another kernel has just written them, rank 16
            // 12.2 -> 6.8 us, rank 128 84 -> 71); rows and columns are clamped, the padding is an identity block
            const double *src = Sb + (size_t)min(row, r - 1) * r + min(col, r - 1);
            double v = 0.0;
            for (int p = 0; p < parts; p += 8) {
                double part[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) part[q] = src[(size_t)min(p + q, parts - 1) * r * r];
#pragma unroll
                for (int q = 0; q < 8; ++q) v += p + q < parts ? part[q] : 0.0;
            }
            if (row >= r || col >= r) v = row == col ? 1.0 : 0.0;
            else if (row == col) tr += v;
            a[t][e] = v;
        }
    if (ridge != 0.0) {
        tr = wave_sum(tr);
        if (lane == 0) red[wave] = tr;
        __syncthreads();
        double sum = 0.0;
        for (int w = 0; w < NW; ++w) sum += red[w];
        const double add = ridge * sum / (double)r;
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * ti + 4 * e + g;
                if (row == 16 * (tk0 + t) + c && row < r) a[t][e] += add;
            }
    }
    for (int j = 0; 16 * j < r; ++j) {
#pragma unroll
        for (int t = 0; t < TPW; ++t)
            if (tk0 + t == j) {                                      // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) U[16 * ti + 4 * e + g][c] = a[t][e];
            }
        __syncthreads();
        constexpr int NT = NB == 8 ? 2 : 1;                          // tiles of the row per stepping wavefront
        if (wave < NB / NT) {
            doublex4_t p, u[NT];                                     // u: the transposed tiles, A_jk
            double (*y)[17] = Y + 16 * NT * wave, (*ys)[17] = Ys + 16 * NT * wave;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // the lower triangle for both
                p[e] = U[16 * j + max(4 * e + g, c)][min(4 * e + g, c)];
#pragma unroll
                for (int t = 0; t < NT; ++t) u[t][e] = U[16 * (NT * wave + t) + c][4 * e + g];
            }
#define FVAR_SWEEP(P)                                                                              \
    if (16 * j + P < r)                                                                            \
        sweep_step<P, NT>(p, u, y, ys, c, g);                                                      \
    else                                                                                           \
        for (int t = 0; t < NT; ++t) y[16 * t + c][P] = ys[16 * t + c][P] = 0.0
            FVAR_SWEEP(0); FVAR_SWEEP(1); FVAR_SWEEP(2); FVAR_SWEEP(3);
            FVAR_SWEEP(4); FVAR_SWEEP(5); FVAR_SWEEP(6); FVAR_SWEEP(7);
            FVAR_SWEEP(8); FVAR_SWEEP(9); FVAR_SWEEP(10); FVAR_SWEEP(11);
            FVAR_SWEEP(12); FVAR_SWEEP(13); FVAR_SWEEP(14); FVAR_SWEEP(15);
#undef FVAR_SWEEP
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (NT * wave + t == j) {                            // rows 16j .. of U stay as the others read them
#pragma unroll
                    for (int e = 0; e < 4; ++e) Pi[4 * e + g][c] = p[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) U[16 * (NT * wave + t) + c][4 * e + g] = u[t][e];
                }
        }
        __syncthreads();
        double ui[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) ui[s] = ti == j ? 0.0 : -Ys[16 * ti + c][4 * s + g];
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const int tk = tk0 + t;
            if (ti == j && tk == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] = Pi[4 * e + g][c];
            } else if (ti == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] = U[16 * tk + c][4 * e + g];
            } else if (tk == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] = U[16 * ti + 4 * e + g][c];
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    a[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ui[s], Y[16 * tk + c][4 * s + g], a[t], 0, 0, 0);
            }
        }
        __syncthreads();                                             // U is rewritten by the next block
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * ti + 4 * e + g, col = 16 * (tk0 + t) + c;
            if (row < r && col < r) Sinv[((size_t)b * r + row) * r + col] = -a[t][e];
        }
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

void launch_factor_t(DType dt, const void *cache, const void *g_c, int B, int M, int r, int d, float *T,
                     hipStream_t st)
{
    // bf16: an ordinary linear layer per sample, in fp32
    if (dt == DType::BF16)
        launch_gemm_bf16_batched_f32(cache, g_c, B, M, r, d, T, st);
    else
        launch(t_f32_kernel, dim3(M, B), dim3(256), 0, st, (const float *)cache, (const float *)g_c, M, r,
               d, T);
}

void launch_factor_gram(DType dt, const void *g_c, int B, int r, int d, double *S, hipStream_t st)
{
    if (dt == DType::BF16) {
        const int rt = (r + 31) / 32;
        launch(gram_bf16_kernel, dim3(rt * (rt + 1) / 2, kGramParts, B), dim3(256), 0, st,
               (const uint16_t *)g_c, r, d, S);
    } else {
        launch(gram_f32_kernel, dim3(r, B), dim3(kGramThreads), (size_t)d * sizeof(float), st,
               (const float *)g_c, r, d, S);
    }
}

int gram_parts(DType dt) { return dt == DType::BF16 ? kGramParts : 1; }

void launch_factor_inverse(const double *S, int parts, int B, int r, double ridge, double *Sinv,
                           hipStream_t st)
{
    if (r <= 32)
        launch(spd_inverse_kernel<2>, dim3(B), dim3(256), 0, st, S, parts, r, ridge, Sinv);
    else if (r <= 64)
        launch(spd_inverse_kernel<4>, dim3(B), dim3(512), 0, st, S, parts, r, ridge, Sinv);
    else
        launch(spd_inverse_kernel<8>, dim3(B), dim3(1024), 0, st, S, parts, r, ridge, Sinv);
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
