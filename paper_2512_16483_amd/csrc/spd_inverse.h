// Inverse of a small symmetric positive definite matrix by one workgroup, in fp64.
#pragma once
#include "common.h"

namespace fvar {

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
// row, brow: rows 4 * (P / 4) .. +3 of a and b at this lane's column, in every lane; the later ones take part in the
// step, by the same operations, so that the next pivot does not wait for a trip through LDS.
template <int P, int NT>
__device__ __forceinline__ void sweep_step(doublex4_t &a, doublex4_t (&b)[NT], double (&row)[4], double (&brow)[4][NT],
                                           double (*y)[17], double (*ys)[17], int c, int g)
{
    constexpr int I = P & 3;
    const double piv = row_bcast<P>(row[I]);
    double inv = __builtin_amdgcn_rcp(piv);                          // ~1e-8, two Newton steps to full precision
    inv = fma(inv, fma(-piv, inv, 1.0), inv);
    inv = fma(inv, fma(-piv, inv, 1.0), inv);
    const double x = c == P ? -1.0 : row[I], xs = x * inv;
    double bs[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) bs[t] = brow[I][t] * inv;
#pragma unroll
    for (int i = I + 1; i < 4; ++i) {
        const double col = row_bcast<P>(row[i]);
        row[i] = fma(-(col * x), inv, c == P ? 0.0 : row[i]);
#pragma unroll
        for (int t = 0; t < NT; ++t) brow[i][t] = fma(-col, bs[t], brow[i][t]);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) { y[16 * t + c][P] = brow[I][t]; ys[16 * t + c][P] = bs[t]; }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double col = row_bcast<P>(a[e]);                       // u at this entry's row
        const double v = fma(-(col * x), inv, c == P ? 0.0 : a[e]);
        const bool pivot = e == (P >> 2) && g == I;
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

// Sweep steps 4E .. 4E + 3: their rows come through LDS together
template <int E, int NT>
__device__ __forceinline__ void sweep_steps(doublex4_t &a, doublex4_t (&b)[NT], double (*y)[17], double (*ys)[17],
                                            int c, int g)
{
    double row[4], brow[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        row[i] = __shfl(a[E], 16 * i + c);
#pragma unroll
        for (int t = 0; t < NT; ++t) brow[i][t] = __shfl(b[t][E], 16 * i + c);
    }
    sweep_step<4 * E + 0, NT>(a, b, row, brow, y, ys, c, g);
    sweep_step<4 * E + 1, NT>(a, b, row, brow, y, ys, c, g);
    sweep_step<4 * E + 2, NT>(a, b, row, brow, y, ys, c, g);
    sweep_step<4 * E + 3, NT>(a, b, row, brow, y, ys, c, g);
}

// LDS of spd_inverse, bytes
constexpr size_t spd_inverse_lds(int NB) { return ((size_t)3 * 16 * NB * 17 + 16 * 17 + 16) * sizeof(double); }

// The NW wavefronts of a workgroup invert an r x r Gram matrix (the sum of `parts` matrices, plus ridge * trace / r
// on the diagonal), without pivoting, by the symmetric sweep, which leaves -S^-1 after
// all pivots.  They are taken 16 at a time (block j): sixteen steps are applied one by one to the pivot block
// and to its tile row A_jk = U_k^T, and the rank-16 update of all the other tiles,
// A_ik -= sum_p (u_ip / d_p) u_kp, is made from the u and d that the steps met.  Those are the scalar sweep's own
// operations in another order.  U P^-1 U^T from an explicit inverse of the pivot block is not the same: it loses
// the square of the condition number where the sweep loses it once (condition 4e6: the inverse off by 4e-6
// instead of 5e-11, T S^-1 of a rank-8 cache with ridge 1e-6 wrong altogether).
// The matrix is padded to 16*NB with an identity block and stays in registers, its lower triangle only, as 16x16
// tiles in the fp64 MFMA's output layout, dealt to the wavefronts in turn.  The first wavefronts apply the steps,
// each to one or two tiles of the row and all to a copy of the pivot block; only the tile column (rows above the
// pivot block from the transposed tiles of its row), u and u / d go through LDS, three barriers per block.
// Steps of the padding are left out.
// At rank 128 its 112 000 clk are: steps 61 000 (480 each with two tiles, 350 with one: a lone wavefront issues one
// fp64 operation in eight clk or more), updates 22 000 (fp64 MFMAs of 64 clk), parking the column 11 000, reading S 9 000.
// By itself, with both triangles, a trip through LDS in front of every step and the stores of the upper triangle
// element by element -> here: rank 128 57.3 -> 48.3 us, 72 38.1 -> 32.1, 64 19.1 -> 16.7, 36 with four wavefronts
// 17.5 -> 13.2, 8 4.6 -> 4.3.  The rows of a step fetched by permlane swaps instead of shuffles: 600 clk a step.
// One tile per stepping wavefront at rank 128: 560, two wavefronts share a SIMD's issue.
// A singular matrix yields non-finite output.
template <int NB, int NW>
__device__ __forceinline__ void spd_inverse(const double *__restrict__ Sb, int parts, int r, double ridge,
                                            double *__restrict__ Sinv, double *lds)
{
    constexpr int TILES = NB * (NB + 1) / 2, TPW = (TILES + NW - 1) / NW;
    constexpr int NT = NB == 8 ? 2 : 1, STEPPING = NB / NT;          // tiles of the row per stepping wavefront
    static_assert((NW < TILES ? NW : TILES) <= 3 * NB, "a tile of LDS per wavefront that has any");
    static_assert(STEPPING <= NW, "a wavefront per one or two tiles of the row");
    double (*U)[17] = reinterpret_cast<double (*)[17]>(lds);         // the tile column, then the swept one
    double (*Y)[17] = U + 16 * NB, (*Ys)[17] = Y + 16 * NB;          // u and u / d
    double (*Pi)[17] = Ys + 16 * NB;
    double *red = &Pi[16][0];
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int ti[TPW], tk[TPW];                                            // tile row and column, ti >= tk; ti = NB: none
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int q = wave + NW * t;
        int i = 0;
        while (i < NB && (i + 1) * (i + 2) / 2 <= q) ++i;
        ti[t] = i;
        tk[t] = q - i * (i + 1) / 2;
    }
    doublex4_t a[TPW];
    double tr = 0.0;
    // the loads of four parts travel together; rows and columns are clamped, the padding is an identity block
#pragma unroll
    for (int t = 0; t < TPW; ++t) a[t] = doublex4_t{0.0, 0.0, 0.0, 0.0};
    for (int p = 0; p < parts; p += 4) {
        double v[4][TPW][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[u][t][e] = Sb[((size_t)min(p + u, parts - 1) * r + min(16 * ti[t] + 4 * e + g, r - 1)) * r +
                                    min(16 * tk[t] + c, r - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (p + u < parts) a[t][e] += v[u][t][e];        // uniform
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * ti[t] + 4 * e + g, col = 16 * tk[t] + c;
            if (row >= r || col >= r) a[t][e] = row == col ? 1.0 : 0.0;
            else if (row == col) tr += a[t][e];
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
                const int row = 16 * ti[t] + 4 * e + g;
                if (row == 16 * tk[t] + c && row < r) a[t][e] += add;
            }
    }
    for (int j = 0; 16 * j < r; ++j) {
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            if (ti[t] == NB) continue;                               // uniform
            if (tk[t] == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) U[16 * ti[t] + 4 * e + g][c] = a[t][e];
            } else if (ti[t] == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) U[16 * tk[t] + c][4 * e + g] = a[t][e];
            }
        }
        __syncthreads();
        if (wave < STEPPING) {
            doublex4_t p, u[NT];                                     // u: the transposed tiles, A_jk
            double (*y)[17] = Y + 16 * NT * wave, (*ys)[17] = Ys + 16 * NT * wave;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // the lower triangle for both
                p[e] = U[16 * j + max(4 * e + g, c)][min(4 * e + g, c)];
#pragma unroll
                for (int t = 0; t < NT; ++t) u[t][e] = U[16 * (NT * wave + t) + c][4 * e + g];
            }
#define FVAR_SWEEP(E)                                                                              \
    if (16 * j + 4 * E < r)                     /* r is a multiple of 4 */                         \
        sweep_steps<E, NT>(p, u, y, ys, c, g);                                                     \
    else                                                                                           \
        for (int q = 4 * E; q < 4 * E + 4; ++q)                                                    \
            for (int t = 0; t < NT; ++t) y[16 * t + c][q] = ys[16 * t + c][q] = 0.0
            FVAR_SWEEP(0); FVAR_SWEEP(1); FVAR_SWEEP(2); FVAR_SWEEP(3);
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
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            if (ti[t] == NB) continue;
            if (ti[t] == j && tk[t] == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] = Pi[4 * e + g][c];
            } else if (ti[t] == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] = U[16 * tk[t] + c][4 * e + g];
            } else if (tk[t] == j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] = U[16 * ti[t] + 4 * e + g][c];
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    a[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-Ys[16 * ti[t] + c][4 * s + g],
                                                                Y[16 * tk[t] + c][4 * s + g], a[t], 0, 0, 0);
            }
        }
        __syncthreads();                                             // U is rewritten by the next block
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * ti[t] + 4 * e + g, col = 16 * tk[t] + c;
            if (row < r && col < r) Sinv[(size_t)row * r + col] = -a[t][e];
        }
    // the upper triangle: turned around in LDS, so that it is stored in rows as well (the last block's barrier has
    // freed the tables)
    double (*X)[17] = U + 16 * wave;
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        if (ti[t] == NB || ti[t] == tk[t]) continue;                 // uniform
#pragma unroll
        for (int e = 0; e < 4; ++e) X[4 * e + g][c] = -a[t][e];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * tk[t] + 4 * e + g, col = 16 * ti[t] + c;
            const double v = X[c][4 * e + g];
            if (row < r && col < r) Sinv[(size_t)row * r + col] = v;
        }
        asm volatile("" ::: "memory");
    }
}

}  // namespace fvar
