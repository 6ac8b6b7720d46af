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
// The matrix is padded to 16*NB with an identity block and stays in registers as 16x16 tiles in the fp64
// MFMA's output layout, TPW tiles of one tile row per wavefront.  The first wavefronts apply the steps,
// each to one or two tiles of the row and all to a copy of the pivot block; only the tile column, u and
// u / d go through LDS, three barriers per block.  Steps of the padding are left out.
// Bound by the chain of steps, 500 clk each, and at rank 128 by the rank-16 updates, 5000 clk per block.  (Columns
// held one per lane, with the pivot column as scalar operands by readlane, take 500 to 560 clk per step too:
// 32 readlanes and 32 fp64 operations, with nothing else to issue from.)  Inside a call, 4 samples at
// rank 128: 65 us in a launch of its own -> 58 in T's launch (which took 28), reading half the matrices with their
// loads in flight together, where one element waited for the last.
// A singular matrix yields non-finite output.
template <int NB, int NW>
__device__ __forceinline__ void spd_inverse(const double *__restrict__ Sb, int parts, int r, double ridge,
                                            double *__restrict__ Sinv, double *lds)
{
    constexpr int TPW = NB * NB > NW ? NB * NB / NW : 1, ACTIVE = NB * NB / TPW;
    constexpr int NT = NB == 8 ? 2 : 1, STEPPING = NB / NT;          // tiles of the row per stepping wavefront
    static_assert(NB % TPW == 0 && ACTIVE <= NW && STEPPING <= NW, "whole tile rows");
    double (*U)[17] = reinterpret_cast<double (*)[17]>(lds);         // the tile column, then the swept one
    double (*Y)[17] = U + 16 * NB, (*Ys)[17] = Y + 16 * NB;          // u and u / d
    double (*Pi)[17] = Ys + 16 * NB;
    double *red = &Pi[16][0];
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ti = wave * TPW / NB, tk0 = wave * TPW % NB;           // tile row, first tile column
    const bool active = wave < ACTIVE;                               // others only keep the barriers
    doublex4_t a[TPW];
    double tr = 0.0;
    if (active) {
        // the loads of a part travel together; rows and columns are clamped, the padding is an identity block
#pragma unroll
        for (int t = 0; t < TPW; ++t) a[t] = doublex4_t{0.0, 0.0, 0.0, 0.0};
        for (int p = 0; p < parts; ++p) {
            double v[TPW][4];
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[t][e] = Sb[((size_t)p * r + min(16 * ti + 4 * e + g, r - 1)) * r + min(16 * (tk0 + t) + c, r - 1)];
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][e] += v[t][e];
        }
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * ti + 4 * e + g, col = 16 * (tk0 + t) + c;
                if (row >= r || col >= r) a[t][e] = row == col ? 1.0 : 0.0;
                else if (row == col) tr += a[t][e];
            }
    }
    if (ridge != 0.0) {
        tr = wave_sum(tr);
        if (lane == 0) red[wave] = tr;
        __syncthreads();
        double sum = 0.0;
        for (int w = 0; w < ACTIVE; ++w) sum += red[w];
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
        if (active)
#pragma unroll
            for (int t = 0; t < TPW; ++t)
                if (tk0 + t == j) {                                  // uniform
#pragma unroll
                    for (int e = 0; e < 4; ++e) U[16 * ti + 4 * e + g][c] = a[t][e];
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
        if (active) {
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
        }
        __syncthreads();                                             // U is rewritten by the next block
    }
    if (active)
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * ti + 4 * e + g, col = 16 * (tk0 + t) + c;
                if (row < r && col < r) Sinv[(size_t)row * r + col] = -a[t][e];
            }
}

}  // namespace fvar
