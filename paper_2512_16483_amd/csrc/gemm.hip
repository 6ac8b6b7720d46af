// Linear layers of the block phi on the rows that pass through it (QKV, output projection,
// MLP): C = epilogue(A[rows,K] * W[N,K]^T).  Both operands are K-contiguous ("out,in" weights),
// which is the layout the MFMA operands want: a lane holds 8 consecutive k of one row.
//
// bf16: workgroup tile BM x BN x 64 computed by WM x WN wavefronts with v_mfma_f32_16x16x32_bf16
// (fp32 accumulation; on operands with realistic bit activity the chip sustains a higher clock
// on this shape than on 32x32x16: half the accumulator register traffic per flop).  Tiles are
// DMA-ed global -> LDS (no register staging) into a ring of stages ahead of the MFMAs; operand
// fragments are read from LDS a few MFMA groups ahead of their use.  LDS rows are 128 B; the
// 16-byte chunk index is XOR-swizzled with (row/2)%8 so that the ds_read_b128 operand fetches of
// 16 consecutive rows cover all 64 banks exactly once.
// Workgroup ids are remapped so that each XCD (own L2) works on a compact patch of the tile
// grid.  Bigger tiles cut the L1/LDS traffic per flop (a 128x128 tile needs the full 64 B/clk of
// the CU's vector L1 at peak MFMA rate, a 256x256 tile half of it) but quantise badly on the few
// thousand rows of a pruned scale, and a few rows leave most CUs without a tile: eleven tiles from
// 320x256 down to 64x64, a kernel whose wavefronts have rings of their own for a few rows, and divisions of
// the contraction axis between workgroups, picked per problem by predicted time (linear_plan, at the end).
//
// fp32: the same kernel on the fp32 MFMA at every size (gemm_rows_kernel).
#include <cmath>
#include <type_traits>

#include "common.h"
#include "spd_inverse.h"

namespace fvar {

struct NoJob {};
struct EpiParams {
    const void *bias;
    const void *residual;
    int gelu;
    void *out0;
    int ld0;
    int split;
    void *kcache, *vcache;
    int hd, cap, len, rows_per_sample;
    int N;
    int out_f32;   // bf16 kernel: write fp32 instead of bf16 (the intermediate residual stream)
    int res_f32;   // bf16 kernel: the residual operand is fp32
};

__device__ __forceinline__ float gelu_tanh(float v)
{
    // 0.5 v (1 + tanh(u)) = v / (1 + exp(-2u)),  u = sqrt(2/pi) (v + 0.044715 v^3)
    // exp(-2u) = exp2(v * (a + b v^2)) with a = -2 sqrt(2/pi) log2(e), b = 0.044715 a
    const float t = v * fmaf(-0.10294324f, v * v, -2.3022082f);
    return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// value of the other lane of each pair of lanes, in registers (a shuffle is an LDS operation, one per pair of
// outputs: 2048 rows of 2048, FC1 62.9 -> 61.2 us, QKV 53.4 -> 51.9)
__device__ __forceinline__ float neighbour(float v)
{
    return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0xb1, 0xf, 0xf, true));   // quad_perm 1,0,3,2
}

// destination of element (row, col) in elements from the base pointer it returns
template <typename T>
__device__ __forceinline__ T *epi_dst(const EpiParams &ep, int row, int col)
{
    if (col < ep.split) return (T *)ep.out0 + (size_t)row * ep.ld0 + col;
    const int b = row / ep.rows_per_sample, j = row - b * ep.rows_per_sample;
    const size_t crow = (size_t)b * ep.cap + ep.len + j;
    int c = col - ep.split;
    if (c < ep.hd) return (T *)ep.kcache + crow * ep.hd + c;
    return (T *)ep.vcache + crow * ep.hd + (c - ep.hd);
}

// Epilogue of 4 consecutive output columns of one row held in fp32: bias, GELU, residual, bf16 or fp32
// output, K / V columns to the cache.  For kernels that own their outputs as float4.
__device__ __forceinline__ void finish_quad(const EpiParams &ep, int row, int col, float4 v)
{
    if (ep.bias) {
        const uint2 b = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(ep.bias) + col);
        v.x += bf16_lo(b.x); v.y += bf16_hi(b.x); v.z += bf16_lo(b.y); v.w += bf16_hi(b.y);
    }
    if (ep.gelu) { v.x = gelu_tanh(v.x); v.y = gelu_tanh(v.y); v.z = gelu_tanh(v.z); v.w = gelu_tanh(v.w); }
    if (ep.residual) {
        const size_t off = (size_t)row * ep.N + col;
        if (ep.res_f32) {
            const float4 r = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(ep.residual) + off);
            v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
        } else {
            const uint2 r = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(ep.residual) + off);
            v.x += bf16_lo(r.x); v.y += bf16_hi(r.x); v.z += bf16_lo(r.y); v.w += bf16_hi(r.y);
        }
    }
    if (ep.out_f32)
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(ep.out0) + (size_t)row * ep.ld0 + col) = v;
    else
        *reinterpret_cast<uint2 *>(epi_dst<uint16_t>(ep, row, col)) =
            make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
}

// ------------------------------------------------------------------------------ bf16 MFMA
constexpr int BK = 64;

// Second launch (us), and write and read of the partials (bytes / us), of a division of every tile and of a
// divided last round.  Chosen on the linear layers of 600 blocks (hidden 1024 .. 4096, rows drawn from 17 ..
// 16000, weights from HBM), each layer timed inside its block undivided, divided and with a divided last
// round: the constants by which picking the lower prediction costs least in sum.  On 360 other blocks the picks
// come to 50297 us where a division was possible and 86490 where a last round was (never 55913 and 87783, best
// 50108 and 86171).  A last round is divided only where that promises 3 %, less than the prediction is
// off by there (5 % rms): a third fewer of them, hence second launches and scratch, for 0.02 to 0.06 % of the
// time (86442 without).  A division of every tile needs no such margin (50352 with it).
constexpr double kMergeUs = 3.0, kMergeRate = 7.7e6;
constexpr double kTailMergeUs = 7.0, kTailMergeRate = 10.0e6, kTailMargin = 1.03;
constexpr double kHbmRate = 6.7e6;     // bytes / us, operands in and output out (fitted)

__device__ __forceinline__ int lds_off(int row, int chunk)      // in bf16 elements
{
    return row * BK + ((chunk ^ ((row >> 1) & 7)) << 3);
}

// Chunk swizzle of a k-major operand tile (rows = k, 256 or 512 bytes each, all starting at the
// same bank).  The transposing load reads, per 32 lanes, the rows {0..3, 8..11} (or {4..7,
// 12..15}) + 16n, 32 contiguous bytes of each: the 8 rows go to 8 different 32-byte eighths of the
// 256-byte bank span.
__device__ __forceinline__ int bkm_swz(int row)
{
    return ((row & 3) | (((row >> 3) & 1) << 2)) << 1;
}

// Epilogue of the bf16 kernel.  The accumulators of a wavefront are kept per 32x32 region
// [i][j] as 2x2 blocks [bi][bj] of the 16x16 MFMA: entry e of a block holds row
// 16*bi + 4*(lane/16) + e, column 16*bj + lane%16 of the region.  Each wavefront applies bias
// and GELU, packs to bf16 (adjacent lanes swap one value per row pair so that a lane owns two
// neighbouring columns)
// and parks its sub-tile row-major in a private LDS region; it then reads the sub-tile back as
// 16-byte row chunks and stores 16 bytes per lane, so a store instruction covers whole 128-byte row
// segments (with a residual, or fp32 output, the sub-tile is parked in fp32).  The destination row
// pointers (plain output, or the K / V cache rows of the sample the row belongs to) are computed once
// per chunk.
template <int FM, int FN, bool F32_STAGED, bool AHEAD>
__device__ __forceinline__ void store_tile_epilogue(const floatx4_t (*acc)[FN][2][2], const EpiParams &ep,
                                                    int rows, int N, int wrow0, int wcol0, int lane,
                                                    uint16_t *wlds)
{
    constexpr int TM = FM * 32, TN = FN * 32, PITCH = TN + 8;
    const int c16 = lane & 15, q16 = lane >> 4;
    const uint16_t *bias = reinterpret_cast<const uint16_t *>(ep.bias);
    if constexpr (F32_STAGED) {
        // fp32 output or a residual (never routed, never GELU-ed): same two-phase scheme with an fp32
        // staging tile, 4 columns per lane out, so that product and residual meet in fp32 and are rounded
        // once, as in finish_quad.  (The kinds are told apart per chunk: with a copy of this code for
        // each, the 320x256 tile spills, -8 %.)
        // The residual is fetched four chunks at a time; AHEAD: the first of them before the staging, the next before
        // the stores of the last.  Loaded one by one where each is used, behind the stores of the one before, they
        // were a chain of trips to memory: O of 2048 rows of 2048 31.0 -> 27.4 us, of 15360 rows 178.9 -> 147.6.
        // The 320x256 tile has registers for four at once but not ahead (24 bytes of spill cost it 20 %): FC2 of 6400 rows
        // of 4096 664 -> 654 us.
        constexpr int P32 = TN + 4, CPR = TN / 4;           // chunks per row
        float *w32 = reinterpret_cast<float *>(wlds);
        uint4 res[2][4];
        auto load_residual = [&](int batch, uint4 *dst) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ci = (batch * 4 + u) * 64 + lane;
                const size_t off = (size_t)min(wrow0 + ci / CPR, rows - 1) * N + min(wcol0 + ci % CPR * 4, N - 4);
                if (ep.res_f32) {
                    dst[u] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(ep.residual) + off);
                } else {
                    const uint2 r = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(ep.residual) + off);
                    dst[u].x = r.x;
                    dst[u].y = r.y;
                }
            }
        };
        if (AHEAD && ep.residual) load_residual(0, res[0]);
#pragma unroll
        for (int jj = 0; jj < 2 * FN; ++jj) {
            const int j = jj >> 1, bj = jj & 1;
            const int col = wcol0 + jj * 16 + c16;
            const float bv = (bias && col < N) ? bf16_to_f32(bias[col]) : 0.f;
#pragma unroll
            for (int ii = 0; ii < 2 * FM; ++ii)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w32[(ii * 16 + 4 * q16 + e) * P32 + jj * 16 + c16] = acc[ii >> 1][j][ii & 1][bj][e] + bv;
        }
        asm volatile("" ::: "memory");       // staging stores and loads use different vector types
        if constexpr (AHEAD) {
            constexpr int BATCHES = TM * CPR / 256;
#pragma unroll
            for (int batch = 0; batch < BATCHES; ++batch) {
                if (batch + 1 < BATCHES && ep.residual) load_residual(batch + 1, res[(batch + 1) & 1]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int ci = (batch * 4 + u) * 64 + lane;
                    const int lrow = ci / CPR, row = wrow0 + lrow, lc = ci % CPR * 4, col = wcol0 + lc;
                    float4 v = *reinterpret_cast<const float4 *>(w32 + lrow * P32 + lc);
                    if (row >= rows || col >= N) continue;
                    if (ep.residual) {
                        const uint4 r = res[batch & 1][u];
                        if (ep.res_f32) {
                            v.x += __uint_as_float(r.x); v.y += __uint_as_float(r.y);
                            v.z += __uint_as_float(r.z); v.w += __uint_as_float(r.w);
                        } else {
                            v.x += bf16_lo(r.x); v.y += bf16_hi(r.x); v.z += bf16_lo(r.y); v.w += bf16_hi(r.y);
                        }
                    }
                    const size_t off = (size_t)row * ep.ld0 + col;
                    if (ep.out_f32)
                        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(ep.out0) + off) = v;
                    else
                        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(ep.out0) + off) =
                            make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
                }
            }
        } else {
#pragma unroll
            for (int it = 0; it < TM * CPR / 64; it += 4) {
                uint4 r[4];
                auto chunk = [&](int u, int &row, int &lc) { const int ci = (it + u) * 64 + lane; row = ci / CPR; lc = ci % CPR * 4; };
                if (ep.residual) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        int lrow, lc;
                        chunk(u, lrow, lc);
                        const size_t off = (size_t)min(wrow0 + lrow, rows - 1) * N + min(wcol0 + lc, N - 4);
                        if (ep.res_f32) {
                            r[u] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(ep.residual) + off);
                        } else {
                            const uint2 h = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(ep.residual) + off);
                            r[u].x = h.x;
                            r[u].y = h.y;
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    int lrow, lc;
                    chunk(u, lrow, lc);
                    const int row = wrow0 + lrow, col = wcol0 + lc;
                    float4 v = *reinterpret_cast<const float4 *>(w32 + lrow * P32 + lc);
                    if (row >= rows || col >= N) continue;
                    if (ep.residual && ep.res_f32) {
                        v.x += __uint_as_float(r[u].x); v.y += __uint_as_float(r[u].y);
                        v.z += __uint_as_float(r[u].z); v.w += __uint_as_float(r[u].w);
                    } else if (ep.residual) {
                        v.x += bf16_lo(r[u].x); v.y += bf16_hi(r[u].x); v.z += bf16_lo(r[u].y); v.w += bf16_hi(r[u].y);
                    }
                    const size_t off = (size_t)row * ep.ld0 + col;
                    if (ep.out_f32)
                        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(ep.out0) + off) = v;
                    else
                        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(ep.out0) + off) =
                            make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
                }
            }
        }
        asm volatile("" ::: "memory");
        return;
    }
    const int odd = lane & 1;
#pragma unroll
    for (int jj = 0; jj < 2 * FN; ++jj) {
        const int j = jj >> 1, bj = jj & 1;
        const int col = wcol0 + jj * 16 + c16;
        const float bv = (bias && col < N) ? bf16_to_f32(bias[col]) : 0.f;
        const int lcol = jj * 16 + c16 - odd;                // even column of the stored pair
#pragma unroll
        for (int ii = 0; ii < 2 * FM; ++ii) {
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                float v0 = acc[ii >> 1][j][ii & 1][bj][e] + bv, v1 = acc[ii >> 1][j][ii & 1][bj][e + 1] + bv;
                if (ep.gelu) { v0 = gelu_tanh(v0); v1 = gelu_tanh(v1); }
                const float send = odd ? v0 : v1;
                const float recv = neighbour(send);
                const int lrow = ii * 16 + 4 * q16 + e + odd;
                *reinterpret_cast<uint32_t *>(wlds + lrow * PITCH + lcol) =
                    odd ? pack_bf16x2(recv, v1) : pack_bf16x2(v0, recv);
            }
        }
    }
    // the region is private to this wavefront and LDS operations of one wavefront complete in
    // order, so no barrier is needed between the two phases (the compiler is kept from moving the
    // accesses across this point: the stores and loads use different vector types)
    asm volatile("" ::: "memory");
    constexpr int CPR = TN / 8;                             // chunks per row
    const bool routed = ep.split < N;                       // K/V columns go to the cache
    const float inv_rps = 1.0f / (float)ep.rows_per_sample;
#pragma unroll
    for (int it = 0; it < TM * CPR / 64; ++it) {
        const int lrow = (it * 64 + lane) / CPR, row = wrow0 + lrow;
        const int lc = (it * 64 + lane) % CPR * 8, col = wcol0 + lc;
        uint4 v = *reinterpret_cast<const uint4 *>(wlds + lrow * PITCH + lc);
        if (row >= rows || col >= N) continue;
        uint16_t *dst;
        const int c = col - ep.split;
        if (!routed || c < 0) {
            dst = (uint16_t *)ep.out0 + (size_t)row * ep.ld0 + col;
        } else {
            // sample index: float estimate, then one exact correction step
            int b = (int)(((float)row + 0.5f) * inv_rps);
            int j0 = row - b * ep.rows_per_sample;
            if (j0 < 0) { --b; j0 += ep.rows_per_sample; }
            else if (j0 >= ep.rows_per_sample) { ++b; j0 -= ep.rows_per_sample; }
            const size_t crow = (size_t)b * ep.cap + ep.len + j0;
            dst = (c < ep.hd) ? (uint16_t *)ep.kcache + crow * ep.hd + c
                              : (uint16_t *)ep.vcache + crow * ep.hd + (c - ep.hd);
        }
        *reinterpret_cast<uint4 *>(dst) = v;
    }
    asm volatile("" ::: "memory");
}

// The operand tiles travel global -> LDS directly (global_load_lds_dwordx4: 16 bytes per lane, a
// wavefront fills 1 KiB = 8 swizzled rows per instruction) into a ring of STAGES buffers,
// STAGES-1 k-tiles ahead of the MFMAs.  No staging registers, no LDS store instructions; the
// loads are counted by hand (vmcnt) because the compiler does not see them.
// M0 carries the LDS base of the instruction; nothing else in these kernels uses M0 (gfx9+ LDS
// instructions do not), and it is rewritten before every use.
__device__ __forceinline__ void dma_b128(const void *base, uint32_t byte_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}
// the same from an address of its own per lane
__device__ __forceinline__ void dma_b128(const void *addr, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds_addr), "v"(addr) : "memory", "m0");
}
// what the chunks past the end of the contraction axis are fetched from
__device__ const uint4 kZeroChunk = {0, 0, 0, 0};

// LDS needed after the main loop: one staging tile per wavefront.
// A wavefront sends its sub-tile through the epilogue in passes of a few 32-row fragments:
// epi_frags() for bf16 output (a staging tile of at most 128 rows), epi_frags_f32() for fp32
// output (as many fragments as fit the LDS with 4-byte elements, at least one).
constexpr size_t kLdsLimit = 160 * 1024;
constexpr int epi_frags(int FM) { return FM > 4 ? (FM + 1) / 2 : FM; }
constexpr size_t epi_bytes_bf16(int BM, int BN, int WM, int WN)
{
    return (size_t)32 * epi_frags(BM / WM / 32) * (BN / WN + 8) * 2 * WM * WN;
}
constexpr size_t epi_bytes_f32(int BN, int WM, int WN, int fe)
{
    return (size_t)32 * fe * (BN / WN + 4) * 4 * WM * WN;
}
constexpr int epi_frags_f32(int BM, int BN, int WM, int WN)
{
    int fe = epi_frags(BM / WM / 32);
    while (fe > 1 && epi_bytes_f32(BN, WM, WN, fe) > kLdsLimit) --fe;
    return fe;
}
// LDS of a launch: the groups' rings, then their exchange, then the staging (in pieces, see the kernel)
constexpr size_t gemm_lds_bytes(int BM, int BN, int WM, int WN, int STAGES, int KG)
{
    const int FM = BM / WM / 32, KGM = FM % KG == 0 ? KG : FM % 2 == 0 && KG % 2 == 0 ? 2 : 1;
    const int EWM = WM * KGM, EWN = WN * (KG / KGM);
    const size_t need[4] = {(size_t)STAGES * KG * (BM + BN) * 64 * 2, (size_t)(KG - 1) * BM * BN * 4,
                            epi_bytes_bf16(BM, BN, EWM, EWN),
                            epi_bytes_f32(BN, EWM, EWN, epi_frags_f32(BM, BN, EWM, EWN))};
    size_t most = 0;
    for (size_t n : need) most = n > most ? n : most;
    return most;
}

// BKM ("B k-major"): the second operand is given as X[K][N] (row = contraction index, as a token
// map is when the contraction runs over tokens: paper, Sec. "Random Projection (RP) for Low-Rank
// Feature", Q^T X) instead of W[N][K].  Its tiles travel to LDS in their own row-major layout and
// the B fragments come from the transposing LDS load.  This mode runs `nbatch` independent
// problems of one shape in one launch (operands and output `*_bstride` elements apart), whole
// tiles only (no division of the contraction), N a multiple of 8, K of 64 or (RAGGED) of 8: the lanes whose
// chunk of the last k-tile lies past its end then fetch zeros for both operands (a copy of the kernel,
// because the test for it in every k-tile costs the whole ones 4 %: 17.4 -> 18.1 us at 692 x 2304 x 2048).
// nbatch > 1 is also available with the ordinary operand layout (no divided tail).
//
// KG > 1: that many groups of WM x WN wavefronts, each with a whole output tile in its accumulators, a ring of
// its own and every KG-th k-tile; the groups' results meet in LDS at the end.  For the small tiles, whose loop
// is bound neither by the DMA (2/3 of its time by itself), nor the LDS reads (1/2 to 2/3) nor the MFMAs (1/3 to
// 1/2), but by how badly these overlap between two barriers: KG k-tiles per barrier, and fewer fragment reads,
// since a group of half the wavefronts has sub-tiles of twice the area.  Us per k-tile with all CUs at work,
// one group -> KG: 64x64 0.32 -> 0.25, 64x128 0.34 -> 0.30, 128x64 0.34 -> 0.28.  128x128 and 192x128 keep
// one group: in two, whose rings then have two stages instead of four and three, they take 1.10 and 1.07 of the time
// over 3000 timings, 1.09 and 1.05 at 16 k-tiles per workgroup, 1.12 and 1.05 at 128.
//
// CHAINS: no fp32 accumulation runs over more than a few k-tiles; the results of these chains are added
// up, with compensation, in a second set of registers.  For a result that meets the inverse of a Gram
// matrix, which magnifies its rounding when it is badly conditioned.  The first workgroups of such a launch, one
// per problem in whole rounds of the XCDs, invert that matrix, which takes as long as the product or longer and
// a CU each.
template <int BM, int BN, int WM, int WN, int STAGES, int KG = 1, bool BKM = false, bool CHAINS = false,
          bool RAGGED = false>
__global__ __launch_bounds__(64 * WM * WN * KG) void gemm_bf16_kernel(
    const uint16_t *__restrict__ A_in, const uint16_t *__restrict__ W_in, int rows, int N, int K,
    int tiles_m, int tiles_n, int group_m, EpiParams ep, int nsplit, float *__restrict__ part,
    int full_tiles, int tail_split, int nbatch, size_t a_bstride, size_t w_bstride,
    size_t o_bstride, std::conditional_t<CHAINS, InverseJob, NoJob> inv)
{
    const uint16_t *A = A_in, *W = W_in;
    constexpr int NW = WM * WN;                        // wavefronts per group
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 32, FN = TN / 32;
    constexpr int NGA = BM / 8 / NW, NGB = BN / 8 / NW; // 1 KiB groups (8 rows) per wavefront
    constexpr int NG = NGA + NGB;                      // DMA instructions per lane per k-tile
    constexpr int STAGE_BYTES = (BM + BN) * BK * 2;
    extern __shared__ uint4 lds_raw[];
    int wg = blockIdx.x, nwg = gridDim.x;
    if constexpr (CHAINS) {
        const int ahead = (nbatch + 7) & ~7;
        if (wg < ahead) {
            constexpr int NW_ALL = WM * WN * KG;
            double *mat = reinterpret_cast<double *>(lds_raw);
            if (wg >= nbatch) return;
            const int r = inv.r;
            const double *S = inv.S + (size_t)wg * kGramParts * r * r;
            double *Sinv = inv.Sinv + (size_t)wg * r * r;
            if (r <= 32) spd_inverse<2, NW_ALL>(S, kGramParts, r, inv.ridge, Sinv, mat);
            else if (BN == 64 || r <= 64) spd_inverse<4, NW_ALL>(S, kGramParts, r, inv.ridge, Sinv, mat);
            else if constexpr (BN > 64) spd_inverse<8, NW_ALL>(S, kGramParts, r, inv.ridge, Sinv, mat);
            return;
        }
        wg -= ahead;
        nwg -= ahead;
    }
    uint32_t lds_base = (uint32_t)(uintptr_t)lds_raw;

    // Work decomposition.  Workgroups are dealt to the 8 XCDs round-robin; XCD x takes the x-th
    // eighth of the work in ascending order.  Three modes:
    //  * plain: one workgroup per tile;
    //  * nsplit > 1 (too few tiles to fill the chip): the contraction axis of every tile is divided
    //    between nsplit workgroups, partial tiles go to `part` in the output's [rows][N] layout;
    //  * tail_split > 1 (the tiles beyond the last full round of 256 would leave most CUs idle):
    //    the first full_tiles tiles run whole, each later tile is divided between tail_split
    //    workgroups whose partial tiles go to `part` tile by tile; every XCD gets an eighth of
    //    the whole tiles first and an eighth of the divided ones after them.
    // Partial tiles are summed and finished by a second kernel.
    const int ntiles = tiles_m * tiles_n * nbatch;
    const int xcd = wg % 8, slot = wg / 8;
    int pid, split = 0, ranges = 1;
    if (tail_split > 1) {
        const int nf = full_tiles / 8, tail_units = (ntiles - full_tiles) * tail_split;
        const int nt = (tail_units + 7) / 8;
        if (slot < nf) {
            pid = xcd * nf + slot;
        } else {
            const int t = xcd * nt + (slot - nf);
            if (slot - nf >= nt || t >= tail_units) return;
            pid = full_tiles + t / tail_split;
            split = t % tail_split;
            ranges = tail_split;
        }
    } else {
        const int per_xcd = (nwg + 7) / 8;
        pid = xcd * per_xcd + slot;
        if (pid >= ntiles * nsplit) return;
        split = pid % nsplit;
        pid /= nsplit;
        ranges = nsplit;
    }
    const int tile_id = pid;
    int bidx = 0;
    if (BKM || nbatch > 1) {
        const int per = tiles_m * tiles_n;
        bidx = pid / per;
        pid -= bidx * per;
        A += (size_t)bidx * a_bstride;
        W += (size_t)bidx * w_bstride;
        ep.out0 = reinterpret_cast<char *>(ep.out0) + (size_t)bidx * o_bstride * (ep.out_f32 ? 4 : 2);
    }
    // consecutive tile ids run down group_m row tiles, then across the columns: the contiguous
    // id range of one XCD is a patch of about group_m x (tiles/8/group_m) tiles
    const int group = pid / (group_m * tiles_n);
    const int first_m = group * group_m;
    const int gsize = min(tiles_m - first_m, group_m);
    const int tm = first_m + (pid % (group_m * tiles_n)) % gsize;
    const int tn = (pid % (group_m * tiles_n)) / gsize;
    const int row0 = tm * BM, col0 = tn * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int all_wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KG > 1 ? all_wave / NW : 0, wave = KG > 1 ? all_wave % NW : all_wave;   // group, wavefront in it
    lds_base += kg * (STAGES * STAGE_BYTES);           // every group has a ring of its own
    const int c16 = lane & 15, q16 = lane >> 4;
    const int wm = wave % NW / WN, wn = wave % NW % WN;     // the modulus saves the 320x256 tile a spill

    // ---- DMA assignment: wavefront w owns the 8-row groups w, w+NW, ... of each tile; lane l of a
    // group fills physical chunk l%8 of row 8*group + l/8, i.e. it fetches the logical chunk that
    // the swizzle maps there
    uint32_t a_off[NGA], b_off[NGB];                   // byte offsets of this lane's 16 B at k = 0
#pragma unroll
    for (int i = 0; i < NGA; ++i) {
        const int r = (wave + NW * i) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        a_off[i] = (uint32_t)(((size_t)(min(row0 + r, rows - 1) - row0) * K + c * 8) * sizeof(uint16_t));
    }
    A += (size_t)row0 * K;
#pragma unroll
    for (int i = 0; i < NGB; ++i) {
        if (BKM) {
            // k-major tile [BK][BN]: a 1 KiB instruction fills 1024 / (2 BN) whole k-rows; lane l
            // fills physical chunk l % (BN/8) of its row with the logical chunk the swizzle maps there
            constexpr int CPR = BN / 8, RPI = 64 / CPR;
            const int r = (wave + NW * i) * RPI + lane / CPR;
            const int c = (lane % CPR) ^ bkm_swz(r);
            b_off[i] = (uint32_t)(((size_t)r * N + min(col0 + c * 8, N - 8)) * sizeof(uint16_t));
        } else {
            const int r = (wave + NW * i) * 8 + (lane >> 3);
            const int c = (lane & 7) ^ ((r >> 1) & 7);
            b_off[i] = (uint32_t)(((size_t)min(col0 + r, N - 1) * K + c * 8) * sizeof(uint16_t));
        }
    }
    const int ktiles_all = RAGGED ? (K + BK - 1) / BK : K / BK, kper = (ktiles_all + ranges - 1) / ranges;
    const int kt0 = split * kper;
    const int ktiles = min(ktiles_all, kt0 + kper) - kt0;   // k-tiles of this workgroup (>= 1)
    const int steps = (ktiles + KG - 1) / KG;               // trips of its loop
    const int nk = (ktiles - kg + KG - 1) / KG;             // k-tiles of this group: kg, kg + KG, ... (steps or one less)
    const int rlane = lane, rK = K;      // for the ragged copy alone: lane and K themselves captured below cost
                                         // the 320x256 tile two spilled registers
    // DMA instructions i0 .. i1-1 (of the NG that make up a k-tile) of k-tile kt into `stage`
    auto issue_part = [&](int kt, int stage, int i0, int i1) {
        const int koff = (kt0 + kg + KG * kt) * BK;
        const uint32_t sbase = lds_base + stage * STAGE_BYTES + wave * 1024;
        if (RAGGED && koff + BK > rK) {                   // the last k-tile; uniform
#pragma unroll
            for (int i = 0; i < NGA; ++i) {
                const int r = (wave + NW * i) * 8 + (rlane >> 3), c = (rlane & 7) ^ ((r >> 1) & 7);
                if (i >= i0 && i < i1)
                    dma_b128(koff + c * 8 < rK ? reinterpret_cast<const char *>(A + koff) + a_off[i]
                                              : reinterpret_cast<const char *>(&kZeroChunk),
                             sbase + i * (NW * 1024));
            }
#pragma unroll
            for (int i = 0; i < NGB; ++i) {
                constexpr int CPR = BN / 8, RPI = 64 / CPR;
                const int r = (wave + NW * i) * RPI + rlane / CPR;
                if (NGA + i >= i0 && NGA + i < i1)
                    dma_b128(koff + r < rK ? reinterpret_cast<const char *>(W + (size_t)koff * N) + b_off[i]
                                          : reinterpret_cast<const char *>(&kZeroChunk),
                             sbase + BM * BK * 2 + i * (NW * 1024));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NGA; ++i)
            if (i >= i0 && i < i1) dma_b128(A + koff, a_off[i], sbase + i * (NW * 1024));
#pragma unroll
        for (int i = 0; i < NGB; ++i)
            if (NGA + i >= i0 && NGA + i < i1)
                dma_b128(BKM ? W + (size_t)koff * N : W + koff, b_off[i],
                         sbase + BM * BK * 2 + i * (NW * 1024));
    };
    // DMA of this workgroup's whole k-tile kt into `stage`
    auto issue = [&](int kt, int stage) { issue_part(kt, stage, 0, NG); };

    floatx4_t acc[FM][FN][2][2];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[i][j][b >> 1][b & 1] = floatx4_t{0};

    floatx4_t sum[CHAINS ? FM : 1][CHAINS ? FN : 1][2][2] = {};
    const int chain = nk > 16 ? 4 : 2;               // longer ones where there are many: their errors average out
    auto fold = [&] {                   // the accumulators into the sums; the next chain starts from what that rounded off
        if constexpr (CHAINS)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        floatx4_t &s = sum[i][j][b >> 1][b & 1], &a = acc[i][j][b >> 1][b & 1];
                        const floatx4_t t = s + a;
                        a -= t - s;
                        s = t;
                    }
    };

    const uint16_t *lds = reinterpret_cast<const uint16_t *>(lds_raw) + kg * (STAGES * STAGE_BYTES / 2);
    // Operand fragments (16x16x32 MFMA: lane l holds row l%16, k-values 8*(l/16) .. +7 of a 32-wide
    // k-step).  The MFMAs of a k-tile are walked as ROWS = steps x (TM/16) "rows": one A fragment
    // (16 tile rows) against the FN16 B fragments of its k-step.  A fragments go through a ring of
    // four slots filled three rows ahead of their use; the B fragments of a k-step are double
    // buffered.  The ring runs across k-tiles: the hand-over point of the loop (DMA of k-tile kt+1
    // landed, barrier) sits three rows before the end of k-tile kt, by which time every wavefront
    // holds all fragments of k-tile kt in registers, so the same barrier frees that tile's stage
    // for the DMA of k-tile kt+STAGES.
    constexpr int FM16 = TM / 16, FN16 = TN / 16;
    // a zero the compiler cannot see through: with constant fragment offsets it hoists every LDS
    // address out of the loop, and the 320x256 tile, which has no register to spare, spills (-8 %)
    int zero = 0;
    asm volatile("" : "+s"(zero));
    constexpr int SPW = BK / 32;                         // k-steps per k-tile
    constexpr int ROWS = SPW * FM16;
    static_assert(ROWS % 4 == 0 && ROWS >= 4, "ring of four A fragments");
    constexpr int SPREAD = ROWS >= 12 ? 6 : KG > 1 && ROWS >= 8 ? 4 : 1;   // rows over which a k-tile's DMA is issued
    static_assert(STAGES >= 2 && STAGES <= 4, "wait counts below are written for 2 to 4 stages");
    // rows at which the B fragments of the next k-step / of the next k-tile are fetched: after the
    // last use of the buffer they go to, and (for this tile's) before the hand-over point
    constexpr int B_NEXT_STEP = FM16 > 2 ? FM16 / 2 : 0;
    constexpr int B_NEXT_TILE = ROWS - 3 > FM16 * (SPW - 1) ? ROWS - 3 : FM16 * (SPW - 1);
    auto load_a = [&](const uint16_t *tile, int row) {   // row of the walk -> fragment
        const int q = row / FM16, i = row % FM16;
        const int r = wm * TM + i * 16 + c16;
        return *reinterpret_cast<const bf16x8_t *>(tile + lds_off(r, (q + zero) * 4 + q16));
    };
    auto load_b = [&](const uint16_t *tile, int q, bf16x8_t *b) {
        if constexpr (BKM) {
            // lane l needs column 16j + l%16 at the k-values 8*(l/16) .. +7 of the k-step.  The
            // transposing load hands lane i of a 16-lane group element i%4 of the 8-byte chunks
            // that lanes 4t + i/4 (t = 0..3) point at: lane l points at k-row 8*(l/16) + (l%16)/4
            // (+4 for the second half) and at columns 16j + 4*(l%4) .. +3.
            typedef short bkm_shortx4_t __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) bkm_shortx4_t lds_shortx4_t;
            const int kr = (q + zero) * 32 + 8 * q16 + (c16 >> 2);
#pragma unroll
            for (int j = 0; j < FN16; ++j) {
                const int chunk = (wn * TN + j * 16) / 8 + ((c16 & 3) >> 1);
                const uint16_t *src = tile + BM * BK + kr * BN + ((chunk ^ bkm_swz(kr)) << 3) + (c16 & 1) * 4;
                const bkm_shortx4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t *)src);
                const bkm_shortx4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t *)(src + 4 * BN));
                b[j] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        } else {
#pragma unroll
            for (int j = 0; j < FN16; ++j) {
                const int r = wn * TN + j * 16 + c16;
                b[j] = *reinterpret_cast<const bf16x8_t *>(tile + BM * BK + lds_off(r, (q + zero) * 4 + q16));
            }
        }
    };

    if (KG == 1 || nk > 0) issue(0, 0);
    if (nk > 1) issue(1, 1);
    if (STAGES >= 3 && nk > 2) issue(2, 2);
    if (STAGES >= 4 && nk > 3) issue(3, 3);
    if (KG == 1 ? nk == 1 : nk <= 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (STAGES >= 4 && nk > 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NG) : "memory");
    else if (STAGES >= 3 && nk > 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NG) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NG) : "memory");
    __syncthreads();

    bf16x8_t ring[4], bb[2][FN16];
    load_b(lds, 0, bb[0]);
#pragma unroll
    for (int t = 0; t < 3; ++t) ring[t] = load_a(lds, t);
    int stage = 0;                                       // stage holding k-tile kt
    for (int kt = 0; kt < steps; ++kt) {
        if (KG > 1 && kt >= nk) break;                   // the last trip has no k-tile for this group
        const uint16_t *cur = lds + stage * (STAGE_BYTES / 2);
        const int nstage = stage + 1 == STAGES ? 0 : stage + 1;
        const uint16_t *nxt = lds + nstage * (STAGE_BYTES / 2);
        const bool more = kt + 1 < steps;                // uniform
#pragma unroll
        for (int row = 0; row < ROWS; ++row) {
            const int q = row / FM16, i = row % FM16;
            if (row == ROWS - 3 && more) {
                // own reads of this stage are complete before the barrier says so
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                // k-tile kt+1 has landed once only the requests of the tiles after it are outstanding
                if (STAGES >= 4 && kt + 3 < nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NG) : "memory");
                else if (STAGES >= 3 && kt + 2 < nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NG) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
            }
            if (row == B_NEXT_TILE && more) load_b(nxt, 0, bb[0]);
            // The DMA of k-tile kt+STAGES into the stage that the hand-over frees is issued a few
            // instructions per row over the SPREAD rows that follow the hand-over (they run into
            // the next k-tile): a burst of all NG instructions from all wavefronts at once fills
            // the CU's vector-memory queue and holds up the MFMAs queued behind them.
            if (row >= ROWS - 3) {
                const int w = row - (ROWS - 3);
                if (w < SPREAD && more && kt + STAGES < nk)
                    issue_part(kt + STAGES, stage, w * NG / SPREAD, (w + 1) * NG / SPREAD);
            } else if (row + 3 < SPREAD) {
                const int w = row + 3;
                if (kt >= 1 && kt - 1 + STAGES < nk)
                    issue_part(kt - 1 + STAGES, stage == 0 ? STAGES - 1 : stage - 1, w * NG / SPREAD,
                               (w + 1) * NG / SPREAD);
            }
            if (row + 3 < ROWS) ring[(row + 3) & 3] = load_a(cur, row + 3);
            else if (more) ring[(row + 3) & 3] = load_a(nxt, row + 3 - ROWS);
            // B fragments of the next k-step of this tile
            if (i == B_NEXT_STEP && q + 1 < SPW) load_b(cur, q + 1, bb[(q + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < FN16; ++j)
                acc[i >> 1][j >> 1][i & 1][j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    ring[row & 3], bb[q & 1][j], acc[i >> 1][j >> 1][i & 1][j & 1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (CHAINS && ((kt + 1) & (chain - 1)) == 0 && more) fold();
        stage = nstage;
    }
    if constexpr (CHAINS) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) acc[i][j][b >> 1][b & 1] += sum[i][j][b >> 1][b & 1];
    }
    // the stage buffers are reused below: every wavefront must be past its last operand read
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    // every request has landed and every wavefront is past its last operand read (barrier above):
    // the stage buffers are free for the groups' exchange and the epilogue's staging.
    // Each group takes a KG-th of every wavefront's sub-tile to the end: KGM x KGN pieces of EM x EN fragments.
    constexpr int KGM = FM % KG == 0 ? KG : FM % 2 == 0 && KG % 2 == 0 ? 2 : 1, KGN = KG / KGM;
    constexpr int EM = FM / KGM, EN = FN / KGN, EWM = WM * KGM, EWN = WN * KGN;
    static_assert(FM % KGM == 0 && FN % KGN == 0, "pieces of whole fragments");
    floatx4_t own[KG > 1 ? EM : 1][KG > 1 ? EN : 1][2][2];
    if constexpr (KG > 1) {
        floatx4_t *xch = reinterpret_cast<floatx4_t *>(lds_raw);
        auto slot = [&](int to, int from, int q) {           // quad q of a piece on its way between groups
            return (((to * (KG - 1) + from) * NW + wave) * (EM * EN * 4) + q) * 64 + lane;
        };
#pragma unroll
        for (int o = 0; o < KG; ++o)
#pragma unroll
            for (int q = 0; q < EM * EN * 4; ++q) {
                const floatx4_t v = acc[o / KGN * EM + q / 4 / EN][o % KGN * EN + q / 4 % EN][(q >> 1) & 1][q & 1];
                if (kg == o) own[q / 4 / EN][q / 4 % EN][(q >> 1) & 1][q & 1] = v;      // uniform
                else xch[slot(o, kg < o ? kg : kg - 1, q)] = v;
            }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < KG - 1; ++g)
#pragma unroll
            for (int q = 0; q < EM * EN * 4; ++q) own[q / 4 / EN][q / 4 % EN][(q >> 1) & 1][q & 1] += xch[slot(kg, g, q)];
        __syncthreads();
    }
    auto &res = [&]() -> auto & { if constexpr (KG > 1) return own; else return acc; }();
    // row and column of the piece in the tile (not variables: with one group that changes the addressing of the
    // whole epilogue, 1 % of a block; with several these expressions in place of them cost 3 % of a projection)
    const int piece_row = wm * TM + kg / KGN * (EM * 32), piece_col = wn * TN + kg % KGN * (EN * 32);
    auto prow = [&] { if constexpr (KG > 1) return piece_row; else return wm * TM; };
    auto pcol = [&] { if constexpr (KG > 1) return piece_col; else return wn * TN; };
    if (ranges > 1) {
        // partial tile, fp32: 16 neighbouring lanes cover 64 contiguous bytes of a row.
        // Divided problem: [range][batch][rows][N]; divided tail: [tail tile][range][BM][BN].
        const bool tail = tail_split > 1;
        float *dst = tail ? part + ((size_t)(tile_id - full_tiles) * tail_split + split) * (BM * BN)
                          : part + ((size_t)split * nbatch + bidx) * rows * N;
        const size_t pitch = tail ? BN : N;
        const int rbase = tail ? 0 : row0, cbase = tail ? 0 : col0;
#pragma unroll
        for (int jj = 0; jj < 2 * EN; ++jj) {
            const int lcol = pcol() + jj * 16 + c16;
            if (col0 + lcol >= N) continue;
#pragma unroll
            for (int ii = 0; ii < 2 * EM; ++ii)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int lrow = prow() + ii * 16 + 4 * q16 + e;
                    if (row0 + lrow < rows)
                        dst[(size_t)(rbase + lrow) * pitch + cbase + lcol] = res[ii >> 1][jj >> 1][ii & 1][jj & 1][e];
                }
        }
        return;
    }
    // per-wavefront staging region; the piece passes through it a few fragments at a time (fewer per pass
    // when the output is fp32)
    constexpr int FE = epi_frags(EM), FE32 = epi_frags_f32(BM, BN, EWM, EWN);
    static_assert(epi_bytes_f32(BN, EWM, EWN, FE32) <= kLdsLimit, "fp32 staging");
    char *stage_base = reinterpret_cast<char *>(lds_raw);
    constexpr bool kAhead = BM * BN < 320 * 256;
    if (ep.out_f32 || ep.residual) {
        uint16_t *wlds = reinterpret_cast<uint16_t *>(stage_base + all_wave * (FE32 * 32 * (EN * 32 + 4) * 4));
#pragma unroll
        for (int f0 = 0; f0 < EM; f0 += FE32) {
            if (f0 + FE32 <= EM)
                store_tile_epilogue<FE32, EN, true, kAhead>(res + f0, ep, rows, N, row0 + prow() + f0 * 32, col0 + pcol(),
                                                    lane, wlds);
            else
                store_tile_epilogue<(EM % FE32 ? EM % FE32 : FE32), EN, true, kAhead>(
                    res + f0, ep, rows, N, row0 + prow() + f0 * 32, col0 + pcol(), lane, wlds);
        }
        return;
    }
    uint16_t *wlds = reinterpret_cast<uint16_t *>(stage_base + all_wave * (FE * 32 * (EN * 32 + 8) * 2));
    store_tile_epilogue<FE, EN, false, false>(res, ep, rows, N, row0 + prow(), col0 + pcol(), lane, wlds);
    if constexpr (FE < EM)
        store_tile_epilogue<EM - FE, EN, false, false>(res + FE, ep, rows, N, row0 + prow() + FE * 32, col0 + pcol(), lane,
                                                wlds);
}

// Sum of the partial tiles of the divided tail + the epilogue (bias, GELU, residual, bf16 or fp32
// output, K and V columns to the cache).  One thread per 4 consecutive columns of one tile row.
__global__ __launch_bounds__(256) void gemm_tail_epilogue_kernel(const float *__restrict__ part,
                                                                 int ranges, int full_tiles,
                                                                 int tiles_m, int tiles_n, int group_m,
                                                                 int BM, int BN, int rows, int N,
                                                                 long total, EpiParams ep)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;       // over tail tiles * BM * BN/4
    if (idx >= total) return;
    const int cpr = BN / 4;
    const int lcol = (int)(idx % cpr) * 4;
    const long tr = idx / cpr;
    const int lrow = (int)(tr % BM), tt = (int)(tr / BM), pid = full_tiles + tt;
    const int group = pid / (group_m * tiles_n);
    const int first_m = group * group_m;
    const int gsize = min(tiles_m - first_m, group_m);
    const int tm = first_m + (pid % (group_m * tiles_n)) % gsize;
    const int tn = (pid % (group_m * tiles_n)) / gsize;
    const int row = tm * BM + lrow, col = tn * BN + lcol;
    if (row >= rows || col >= N) return;
    const float *src = part + (size_t)tt * ranges * BM * BN + (size_t)lrow * BN + lcol;
    float4 v = *reinterpret_cast<const float4 *>(src);
    for (int s = 1; s < ranges; ++s) {
        const float4 p = *reinterpret_cast<const float4 *>(src + (size_t)s * BM * BN);
        v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    finish_quad(ep, row, col, v);
}

// tail > 1: the tiles beyond the last full round of 256 are divided into `tail` ranges of the
// contraction axis each (nsplit must be 1 then)
template <int BM, int BN, int WM, int WN, int STAGES, int KG = 1>
static void launch_gemm_bf16_cfg(const void *A, const void *W, int rows, int N, int K,
                                 const EpiParams &ep, hipStream_t st, int nsplit = 1,
                                 float *part = nullptr, int tail = 1)
{
    const int tiles_m = (rows + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int ntiles = tiles_m * tiles_n;
    const int full_tiles = tail > 1 ? ntiles / 256 * 256 : ntiles;
    const int tail_units = (ntiles - full_tiles) * tail;
    const int grid = tail > 1 ? full_tiles + (tail_units + 7) / 8 * 8 : (ntiles * nsplit + 7) / 8 * 8;
    constexpr size_t lds = gemm_lds_bytes(BM, BN, WM, WN, STAGES, KG);
    static_assert(lds <= kLdsLimit, "LDS of a CU");
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, STAGES, KG>;
    // set on every launch: the attribute belongs to the current device's copy of the kernel
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    // patch height that minimises what one XCD has to pull through its own L2: a patch of g x c
    // tiles reads g row strips (BM x K) and c column strips (BN x K), with g * c = tiles / 8
    int group_m = (int)lround(sqrt((double)ntiles * BN / (8.0 * BM)));
    group_m = group_m < 1 ? 1 : (group_m > tiles_m ? tiles_m : group_m);
    launch(kern, dim3(grid), dim3(64 * WM * WN * KG), lds, st, (const uint16_t *)A,
                       (const uint16_t *)W, rows, N, K, tiles_m, tiles_n, group_m, ep, nsplit, part,
                       full_tiles, tail, 1, (size_t)0, (size_t)0, (size_t)0, NoJob{});
    if (tail > 1) {
        const long total = (long)(ntiles - full_tiles) * BM * (BN / 4);
        launch(gemm_tail_epilogue_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
               (const float *)part, tail, full_tiles, tiles_m, tiles_n, group_m, BM, BN, rows, N, total, ep);
    }
}

// out[b] = A[b] X[b] for nbatch problems with the second operand k-major (X[b]: [K][N], A[b]:
// [rows][K], `a_bstride` elements apart or shared when 0), bf16 output, no epilogue terms.
template <int BM, int BN, int WM, int WN, int STAGES, int KG = 1>
static void launch_kmajor_cfg(const void *A, size_t a_bstride, const void *X, int nbatch, int rows,
                              int N, int K, void *out, hipStream_t st)
{
    EpiParams ep{};
    ep.out0 = out; ep.ld0 = N; ep.split = N; ep.N = N; ep.rows_per_sample = 1;
    const int tiles_m = (rows + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int ntiles = tiles_m * tiles_n * nbatch;
    const int grid = (ntiles + 7) / 8 * 8;
    constexpr size_t lds = gemm_lds_bytes(BM, BN, WM, WN, STAGES, KG);
    static_assert(lds <= kLdsLimit, "LDS of a CU");
    auto kern = K % BK ? gemm_bf16_kernel<BM, BN, WM, WN, STAGES, KG, true, false, true>
                       : gemm_bf16_kernel<BM, BN, WM, WN, STAGES, KG, true>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int group_m = (int)lround(sqrt((double)tiles_m * tiles_n * BN / (8.0 * BM)));
    group_m = group_m < 1 ? 1 : (group_m > tiles_m ? tiles_m : group_m);
    launch(kern, dim3(grid), dim3(64 * WM * WN * KG), lds, st, (const uint16_t *)A, (const uint16_t *)X, rows,
           N, K, tiles_m, tiles_n, group_m, ep, 1, (float *)nullptr, ntiles, 1, nbatch, a_bstride,
           (size_t)K * N, (size_t)rows * N, NoJob{});
}

// out[p][b] = share p of the contraction of A[b] W[b]^T, in fp32, for nbatch problems of one shape (A[b]:
// [rows][K], W[b]: [N][K], both bf16 and `rows*K` / `N*K` elements apart; out[p][b]: [rows][N]), on the
// tiled MFMA kernel.  K a multiple of 64, N <= 128.  The number of shares is batched_f32_parts().
// Error against 64 bits of positive values at K = 1024, 2048, 4096 (two shares, at 2048 three) and
// 4096 (one share): 4.3, 4.2, 4.0 and 3.2e-8, with one chain per share 9.2, 9.2, 17 and 34e-8; 25.6 -> 28.3 us at
// 4 x (4096 x 4096 x 128).
template <int BM, int BN, int WM, int WN, int STAGES, int KG = 1>
static void launch_batched_f32_cfg(const void *A, const void *W, int nbatch, int rows, int N, int K,
                                   int parts, float *out, const InverseJob &inv, hipStream_t st)
{
    EpiParams ep{};
    ep.out0 = out; ep.ld0 = N; ep.split = N; ep.N = N; ep.rows_per_sample = 1; ep.out_f32 = 1;
    const int tiles_m = (rows + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int ntiles = tiles_m * tiles_n * nbatch;
    const int grid = (nbatch + 7) / 8 * 8 + (ntiles * parts + 7) / 8 * 8;
    constexpr size_t lds = gemm_lds_bytes(BM, BN, WM, WN, STAGES, KG);
    static_assert(lds >= spd_inverse_lds(BN > 64 ? 8 : 4), "the inverse's tables fit the rings");
    static_assert(lds <= kLdsLimit, "LDS of a CU");
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, STAGES, KG, false, true>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int group_m = (int)lround(sqrt((double)tiles_m * tiles_n * BN / (8.0 * BM)));
    group_m = group_m < 1 ? 1 : (group_m > tiles_m ? tiles_m : group_m);
    launch(kern, dim3(grid), dim3(64 * WM * WN * KG), lds, st, (const uint16_t *)A, (const uint16_t *)W, rows,
           N, K, tiles_m, tiles_n, group_m, ep, parts, out, ntiles, 1, nbatch,
           (size_t)rows * K, (size_t)N * K, (size_t)rows * N, inv);
}

// Output rows, over all shares and problems, that a plan never exceeds: the shares it may take (each at
// least 4 k-tiles; two are always counted, the least this has ever been), as long as their partial
// results stay below 96K rows.  Never falls as the problem grows, which the shares themselves do.
size_t batched_f32_room(int nbatch, int rows, int K)
{
    const size_t R = (size_t)nbatch * rows, kt = K / BK, shares = kt < 8 ? 2 : kt < 16 ? kt / 4 : 4;
    const size_t divided = shares * R < (96u << 10) ? shares * R : (96u << 10);
    return R > divided ? R : divided;
}

// Tile height (256, 128 or 64 rows; one tile spans all N <= 128 columns) and shares of the contraction,
// by the same prediction as tile_plan; the consumer sums the shares, so they cost it a read each.
struct BatchedPlan { int bm, parts; };
static BatchedPlan batched_f32_plan(int nbatch, int rows, int N, int K)
{
    // (64 rows of the narrow tile run in four groups, but are priced without: as linear layers are, 0.237 and 0.46,
    // takes more shares and makes handovers of 144 sizes 0.1 % slower, at rank 32 up to 4.6)
    const bool narrow = N <= 64;
    const struct { int bm; double k_us, tile_us; } cands[3] = {
        {256, 0.896, 1.9}, {128, narrow ? 0.364 : 0.537, narrow ? 0.3 : 0.95}, {64, narrow ? 0.274 : 0.375, 0.3}};
    const int kt = K / BK;
    // operands beyond the 256 MB of last-level cache (the caller has just read them) take the time they
    // need from HBM at 5.5 TB/s; among equals the largest tile, which is then the fastest (40 x
    // (4096 x 4096 x 128): 280 us with 256 rows, 306 with 128; with 64 columns of G 87 and 92)
    const double bytes = nbatch * (2.0 * ((double)rows + N) * K + 4.0 * rows * N);
    const double hbm_us = bytes > 256e6 ? bytes / 5.5e6 : 0.0;
    // the inverse of the same launch takes that long in any case, and a CU per problem (4 samples at rank 128:
    // one share instead of two for the kernel that reads them, 132.8 -> 128.1 us in all)
    const double inverse_us = (N <= 64 ? 0.22 : 0.39) * N;
    const int cus = nbatch <= 32 ? 256 - nbatch : 256;
    BatchedPlan best{256, 1};
    double best_us = 1e300;
    for (const auto &c : cands)
        for (int parts = 1; parts <= 4; ++parts) {
            const int per = (kt + parts - 1) / parts;
            if (parts > 1 && (kt / parts < 4 || (parts - 1) * per >= kt ||
                              (size_t)parts * nbatch * rows > batched_f32_room(nbatch, rows, K)))
                continue;
            const long tiles = (long)((rows + c.bm - 1) / c.bm) * nbatch;
            const double rounds = (double)((tiles * parts + cus - 1) / cus);
            const double us = fmax(fmax(hbm_us, inverse_us), rounds * (c.tile_us + c.k_us * per)) +
                              (parts - 1) * (1.0 + 8.0 * nbatch * rows * N / kMergeRate);
            if (us < best_us) { best_us = us; best = {c.bm, parts}; }
        }
    return best;
}
int batched_f32_parts(int nbatch, int rows, int N, int K) { return batched_f32_plan(nbatch, rows, N, K).parts; }
int batched_f32_tile_rows(int nbatch, int rows, int N, int K) { return batched_f32_plan(nbatch, rows, N, K).bm; }

void launch_gemm_bf16_batched_f32(const void *A, const void *W, int nbatch, int rows, int N, int K,
                                  float *out, const InverseJob &inv, hipStream_t st)
{
    const BatchedPlan p = batched_f32_plan(nbatch, rows, N, K);
    const bool narrow = N <= 64;
    if (p.bm == 256) launch_batched_f32_cfg<256, 128, 4, 2, 3>(A, W, nbatch, rows, N, K, p.parts, out, inv, st);
    else if (p.bm == 128 && narrow) launch_batched_f32_cfg<128, 64, 4, 2, 4>(A, W, nbatch, rows, N, K, p.parts, out, inv, st);
    else if (p.bm == 128) launch_batched_f32_cfg<128, 128, 2, 4, 4>(A, W, nbatch, rows, N, K, p.parts, out, inv, st);
    else if (narrow) launch_batched_f32_cfg<64, 64, 1, 1, 2, 4>(A, W, nbatch, rows, N, K, p.parts, out, inv, st);
    else launch_batched_f32_cfg<64, 128, 2, 4, 4>(A, W, nbatch, rows, N, K, p.parts, out, inv, st);
}

// Whether the 64x128 tiles of a projection run with wavefront groups: from 8 k-tiles on, in one round, and as long
// as no more than 160 column strips of x, which the tiles above each other share, are read at once.  Where every
// CU reads a strip of its own the loop waits for memory and the groups' longer first fill comes on top.  Time of one
// group over time of two: 16 or 128 strips, 2 k-tiles 0.95, 5 and 7 0.99 to 1.01, 14 1.04, 36 1.08, 64 1.12; 192
// strips, 8 to 64 k-tiles 0.93 to 0.98; 512 strips and more, 1 to 8 k-tiles 0.85 to 0.92, 16 0.95, 64 0.98.
bool kmajor_in_groups(int B, int M, int rows, int d)
{
    const long strips = (long)((d + 127) / 128) * B;
    return (M + BK - 1) / BK >= 8 && strips <= 160 && (rows + 63) / 64 * strips <= 256;
}

// Runs out[b] = qt[b] x[b] (qt: [rows][M] per sample or shared, x[b]: [M][d]) on the tiled MFMA
// kernel (M a multiple of 8, d of 64).  Where not even 64 rows of qt fit 32-bit byte offsets (M of 2^25 and more),
// as many rows at a time as do, sample by sample (8 rows of 2^25 tokens, width 64: 0.20 s; 15.8 by a thread per
// column).  Tile by predicted time, constants as in tile_plan plus
// a tenth for the transposing reads (no 320x256 tile: with them it would not fit the 256 registers).  Even a
// few tiles here beat many of a kernel that turns X around through registers, whose 64-token chunk takes
// 1.7 us against 0.4 us of a 64x128 k-tile: 692 x 2304 x 2048 61 -> 17 us, 4 x (128 x 4096 x 4096)
// 123 -> 39 us; ragged, 692 x 2312 x 2048 51.5 -> 18.6, 4 x (2000 x 6392 x 4096) 720 -> 368 us.
void launch_gemm_bf16_kmajor(const void *qt, size_t q_stride, const void *x, int B, int M, int rows,
                             int d, void *out, hipStream_t st)
{
    const struct { int bm, bn; double k_us, tile_us; } cands[] = {
        {256, 256, 1.64, 3.4}, {192, 256, 1.43, 2.0}, {256, 128, 0.98, 1.9}, {128, 256, 0.98, 1.9},
        {192, 128, 0.77, 1.3}, {128, 128, 0.59, 0.95}, {64, 128, 0.41, 0.3}};
    int best = -1;
    double best_us = 1e300;
    const int kt = (M + BK - 1) / BK;
    const double bytes = 2.0 * B * ((double)M * d + (double)rows * d + (q_stride ? (double)rows * M : 0));
    for (int i = 0; i < 7; ++i) {
        const auto &c = cands[i];
        if ((size_t)c.bm * M * sizeof(uint16_t) >= ((size_t)1 << 32)) continue;   // 32-bit operand offsets
        const long tiles = (long)((rows + c.bm - 1) / c.bm) * ((d + c.bn - 1) / c.bn) * B;
        // what the operands' way from HBM adds: 0.040 us/MB in rows of 512 bytes, 0.058 in rows of 256 (40
        // samples of 4096 x 4096 to 128 rows: 247 us with 128x256 tiles, 271 with 128x128, of which the
        // tiles' own time is 194 each; 24 samples 153 and 163)
        const double us = (double)((tiles + 255) / 256) * (c.tile_us + c.k_us * kt) +
                          bytes * (c.bn >= 256 ? 4.0e-8 : 5.8e-8);
        if (us < best_us) { best_us = us; best = i; }
    }
    switch (best) {
    case 0: launch_kmajor_cfg<256, 256, 2, 4, 2>(qt, q_stride, x, B, rows, d, M, out, st); break;
    case 1: launch_kmajor_cfg<192, 256, 2, 4, 2>(qt, q_stride, x, B, rows, d, M, out, st); break;
    case 2: launch_kmajor_cfg<256, 128, 4, 2, 3>(qt, q_stride, x, B, rows, d, M, out, st); break;
    case 3: launch_kmajor_cfg<128, 256, 2, 4, 3>(qt, q_stride, x, B, rows, d, M, out, st); break;
    case 4: launch_kmajor_cfg<192, 128, 2, 4, 3>(qt, q_stride, x, B, rows, d, M, out, st); break;
    case 5: launch_kmajor_cfg<128, 128, 2, 4, 4>(qt, q_stride, x, B, rows, d, M, out, st); break;
    case 6:
        if (kmajor_in_groups(B, M, rows, d)) launch_kmajor_cfg<64, 128, 2, 2, 3, 2>(qt, q_stride, x, B, rows, d, M, out, st);
        else launch_kmajor_cfg<64, 128, 2, 4, 4>(qt, q_stride, x, B, rows, d, M, out, st);
        break;
    default: {
        const int n = (int)(((1u << 31) - BK) / (unsigned)M) + 1;
        for (int b = 0; b < B; ++b)
            for (int t = 0; t < rows; t += n)
                launch_kmajor_cfg<64, 128, 2, 4, 4>((const uint16_t *)qt + b * q_stride + (size_t)t * M, 0,
                                                    (const uint16_t *)x + (size_t)b * M * d, 1, n < rows - t ? n : rows - t,
                                                    d, M, (uint16_t *)out + ((size_t)b * rows + t) * d, st);
    }
    }
}

// Sum of the partial tiles of a split contraction + the epilogue (bias, GELU, residual, bf16 or
// fp32 output, K and V columns to the cache).  One thread per 4 consecutive columns.
__global__ __launch_bounds__(256) void gemm_splitk_epilogue_kernel(const float *__restrict__ part,
                                                                   int nsplit, int rows, int N,
                                                                   EpiParams ep)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const int cpr = N / 4;
    if (idx >= (long)rows * cpr) return;
    const int row = (int)(idx / cpr), col = (int)(idx % cpr) * 4;
    const size_t off = (size_t)row * N + col;
    float4 v = *reinterpret_cast<const float4 *>(part + off);
    for (int s = 1; s < nsplit; ++s) {
        const float4 p = *reinterpret_cast<const float4 *>(part + (size_t)s * rows * N + off);
        v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    finish_quad(ep, row, col, v);
}

// ------------------------------------------------------------------------------ fp32
// Same epilogue for fp32 storage.
__device__ __forceinline__ void finish_quad_f32(const EpiParams &ep, int row, int col, float4 v)
{
    if (ep.bias) {
        const float4 b = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(ep.bias) + col);
        v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
    }
    if (ep.gelu) {
        const auto gelu = [](float x) {
            return 0.5f * x * (1.0f + tanhf(0.7978845608028654f * (x + 0.044715f * x * x * x)));
        };
        v.x = gelu(v.x); v.y = gelu(v.y); v.z = gelu(v.z); v.w = gelu(v.w);
    }
    if (ep.residual) {
        const float4 r = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(ep.residual) +
                                                           (size_t)row * ep.N + col);
        v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
    }
    *reinterpret_cast<float4 *>(epi_dst<float>(ep, row, col)) = v;
}

__global__ __launch_bounds__(256) void gemm_f32_merge_kernel(const float *__restrict__ part, int nsplit,
                                                             int rows, int N, EpiParams ep)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const int cpr = N / 4;
    if (idx >= (long)rows * cpr) return;
    const int row = (int)(idx / cpr), col = (int)(idx % cpr) * 4;
    const float *src = part + (size_t)row * N + col;
    float4 v = *reinterpret_cast<const float4 *>(src);
    for (int s = 1; s < nsplit; ++s) {
        const float4 p = *reinterpret_cast<const float4 *>(src + (size_t)s * rows * N);
        v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    finish_quad_f32(ep, row, col, v);
}

// Linear layer of a few rows (bf16), or of any number (fp32).  A workgroup owns 16*FT output features and 16*TT rows; its
// NW wavefronts take NW shares of the contraction axis, each with a ring of its own in LDS, so there is no
// barrier before the end, where the partial tiles meet in LDS.  Weights are the A operand of the MFMA: a lane ends up
// with 4 consecutive features of one row.
// What bounds it: at few rows the operands' way through the CU's vector L1 (the rows are read again by
// every feature tile, L2 hits), so the DMA fetches whole 128-byte lines.  Loads in the MFMA's own lane order, a row
// per lane, would save the LDS but reach only 38 GB/s per CU where these reach 150: only neighbouring lanes'
// addresses are taken together.  Rings of 64-byte rows are 20 to 30 % slower too.  Two to four steps in flight are the
// same within 3 % (16x16: 16 rows, 7680 to 1920 12.1, 12.0 and 11.9 us, fp32 1024 to 1024 4.2, 4.3 and 4.5); the larger instances
// have LDS for two or three.  us, weights from HBM, against loads straight to registers or 64x64 tiles, whichever was
// faster: 64 rows, hidden 2048, QKV 13.6 -> 8.9, O 10.8 -> 6.0, FC1 14.9 -> 11.0, FC2 15.5 -> 14.2 (the weights alone
// take 7.2, 4.8, 8.9 and 8.9 in launches by themselves, an empty one 2.4); 16 rows QKV 10.5 -> 7.2, FC1 10.9 -> 8.6.
// fp32, bound by the MFMA's rate (157 TFLOP/s, as the vector units) from a few hundred rows on, so what counts is
// that every CU gets the same share: hidden 1024, 128 rows QKV 16.9 -> 10.4, O 10.9 -> 6.4, FC1 17.8 -> 14.7,
// FC2 21.1 -> 14.4, 2048 rows FC1 254 -> 190.
template <typename T, int FT, int TT, int NW, int STAGES>
__global__ __launch_bounds__(64 * NW) void gemm_rows_kernel(
    const T *__restrict__ A, const T *__restrict__ W, int rows, int N, int K, int row_tiles,
    int nsplit, EpiParams ep, float *__restrict__ part)
{
    constexpr int NF = FT + TT;                         // fragments of 16 rows
    constexpr int IPF = 2, NI = NF * IPF;               // DMA instructions (8 rows x 128 bytes) per fragment and step
    constexpr int KE = 128 / sizeof(T);                 // contraction indices per step: two MFMA k-steps
    static_assert(FT * TT <= STAGES * NI, "a wavefront's result fits its ring");
    extern __shared__ uint4 lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q16 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD takes one contiguous share of the (feature tile, split, row tile) units
    const int units = row_tiles * nsplit * (N / (16 * FT));
    const int per_xcd = (units + 7) / 8;
    int pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (pid >= units || (int)(blockIdx.x >> 3) >= per_xcd) return;
    const int rt = pid % row_tiles; pid /= row_tiles;
    const int split = pid % nsplit, n0 = pid / nsplit * (16 * FT), row0 = rt * (16 * TT);

    // steps of this wavefront: the first `extra` of all shares take one more
    const int steps = K / KE, parts = nsplit * NW, pi = split * NW + wave;
    const int per = steps / parts, extra = steps - per * parts;
    const int s0 = pi * per + min(pi, extra), n = per + (pi < extra ? 1 : 0);
    // lane l of a DMA instruction fills physical chunk l%8 of row l/8; chunks are swizzled as in lds_off()
    const T *Wb = W + (size_t)n0 * K + (size_t)s0 * KE, *Ab = A + (size_t)row0 * K + (size_t)s0 * KE;
    uint32_t off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int r = (i % IPF) * 8 + lane / 8, f = i / IPF;
        const int row = f < FT ? 16 * f + r : min(row0 + 16 * (f - FT) + r, rows - 1) - row0;
        off[i] = (uint32_t)((size_t)row * K * sizeof(T)) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    constexpr int RING = STAGES * NI * 1024;
    const uint32_t ring = (uint32_t)(uintptr_t)lds_raw + wave * RING;
    const uint4 *mine = lds_raw + wave * (RING / 16);
    auto issue = [&](int s) {
        const uint32_t dst = ring + (uint32_t)(s % STAGES) * (NI * 1024);
#pragma unroll
        for (int i = 0; i < NI; ++i)
            dma_b128((i / IPF < FT ? Wb : Ab) + (size_t)s * KE, off[i], dst + i * 1024);
    };
    // waits until only the `after` steps requested last are outstanding
    auto landed = [&](int after) {
        if (STAGES > 3 && after == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STAGES > 3 ? 3 * NI : 0) : "memory");
        else if (STAGES > 2 && after == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STAGES > 2 ? 2 * NI : 0) : "memory");
        else if (after == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    static_assert(STAGES >= 2 && STAGES <= 4, "wait counts are written for 2 to 4 stages");

    floatx4_t acc[FT][TT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int t = 0; t < TT; ++t) acc[f][t] = floatx4_t{0};
    // fp32: no accumulation runs over more than a step's 32 products; what these chains give is added up in a second
    // set of registers.  (One chain per wavefront is as fast, but the block of 128 rows, hidden 1024, is then off by 3.0e-7 with
    // four wavefronts and by 2.2e-7 with eight, against 1.35e-7.)
    constexpr bool CHAINS = sizeof(T) == 4;
    floatx4_t sum[CHAINS ? FT : 1][CHAINS ? TT : 1] = {};
    uint4 frag[2][NF];
    // fragments of MFMA k-step u of step s
    auto fetch = [&](int s, int u, uint4 *dst) {
        const uint4 *src = mine + (s % STAGES) * (NI * 64) + c16 * 8 + ((u * 4 + q16) ^ (c16 >> 1));
#pragma unroll
        for (int i = 0; i < NF; ++i) dst[i] = src[i * 128];
    };
    auto mac = [&](const uint4 *v) {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int f = 0; f < FT; ++f)
#pragma unroll
                for (int t = 0; t < TT; ++t)
                    acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, v[f]), __builtin_bit_cast(bf16x8_t, v[FT + t]), acc[f][t], 0, 0, 0);
        } else {
            // a chunk holds four consecutive k of a row: the k-slots of four MFMAs
#define FVAR_MAC(c)                                                                                       \
            _Pragma("unroll") for (int f = 0; f < FT; ++f) _Pragma("unroll") for (int t = 0; t < TT; ++t) \
                acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(v[f].c),                 \
                                                                 __uint_as_float(v[FT + t].c), acc[f][t], 0, 0, 0)
            FVAR_MAC(x); FVAR_MAC(y); FVAR_MAC(z); FVAR_MAC(w);
#undef FVAR_MAC
        }
    };
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < n) issue(s);
    if (n > 0) {
        landed(min(n, STAGES) - 1);
        fetch(0, 0, frag[0]);
    }
    for (int s = 0; s < n; ++s) {
        fetch(s, 1, frag[1]);
        __builtin_amdgcn_sched_barrier(0);
        mac(frag[0]);
        __builtin_amdgcn_sched_barrier(0);
        // the stage is free once its last fragments are in registers
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (s + STAGES < n) issue(s + STAGES);
        if (s + 1 < n) {
            landed(min(n - 2 - s, STAGES - 1));
            fetch(s + 1, 0, frag[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        mac(frag[1]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (CHAINS)
#pragma unroll
            for (int f = 0; f < FT; ++f)
#pragma unroll
                for (int t = 0; t < TT; ++t) { sum[f][t] += acc[f][t]; acc[f][t] = floatx4_t{0}; }
    }
    if constexpr (CHAINS)
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int t = 0; t < TT; ++t) acc[f][t] += sum[f][t];
    // the wavefronts' partial tiles meet in LDS, each in its own ring
    float4 *red = reinterpret_cast<float4 *>(lds_raw);
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int t = 0; t < TT; ++t)
            red[wave * (RING / 16) + (f * TT + t) * 64 + lane] =
                make_float4(acc[f][t][0], acc[f][t][1], acc[f][t][2], acc[f][t][3]);
    __syncthreads();
    for (int blk = wave; blk < FT * TT; blk += NW) {
        float4 v = red[blk * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const float4 p = red[w * (RING / 16) + blk * 64 + lane];
            v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
        }
        const int row = row0 + (blk % TT) * 16 + c16, col = n0 + (blk / TT) * 16 + 4 * q16;
        if (row >= rows) continue;
        if (nsplit > 1) *reinterpret_cast<float4 *>(part + ((size_t)split * rows + row) * N + col) = v;
        else if constexpr (sizeof(T) == 2) finish_quad(ep, row, col, v);
        else finish_quad_f32(ep, row, col, v);
    }
}

// ------------------------------------------------------------------------------ plan
// Which kernel, tile and division of the contraction axis a bf16 problem gets: the candidate with
// the lowest predicted time.  The prediction is
//     launch + rounds x (per tile + per k-tile x k-tiles of a workgroup) [+ merge of the partials]
// with rounds of workgroups over the 256 CUs, never below the time in which the operands and the
// output cross HBM.  Its constants are a least-squares fit to 8200 timings of every tile with every
// division on 344 problems (rows 7 .. 15360, hidden 1024 .. 4096, the four layers of a block):
// residual 4 % rms.  Of 63000 timings of the kernels as they are now, on 1320 problems, its picks are on average
// 2.7 % (19 in 20 at most 15 %, worst 34 %) slower than the best candidate of each; constants of the small tiles
// refitted on half of them gain 0.2 % on the other half.  One rate per tile and no small tiles cost 30 % (worst 3x).
// The undivided timings are in profiles/linear_layer_tile_times.txt, divisions in linear_layer_divisions.txt.
// With wavefront groups the last three tiles have constants of their own (kGroupedTiles), used exactly where the
// launch takes them.  With these for the kernels without groups too, 320 workgroups of 64x64 looked 10 % cheaper than
// they are: on 115 of 3000 problems where the picks differ 17.1 us in geometric mean instead of 15.9, at worst 1536 x 6144
// with 703 rows 40.5 instead of 28.1, and 128x64 divided eight ways took more workspace than 64x64 in five.
constexpr double kLaunchUs = 3.6;      // a launch by itself

struct TileCfg { int bm, bn; double k_us, tile_us; };   // us per k-tile and per tile with all CUs at work
constexpr TileCfg kTiles[] = {
    {320, 256, 1.745, 4.9}, {256, 256, 1.491, 3.4}, {192, 256, 1.304, 2.0}, {256, 192, 1.289, 2.0},
    {256, 128, 0.896, 1.9}, {128, 256, 0.891, 1.9}, {192, 128, 0.704, 1.3}, {128, 128, 0.537, 0.95},
    {64, 128, 0.375, 0.3},  {128, 64, 0.364, 0.3},  {64, 64, 0.274, 0.1}};
constexpr TileCfg kGroupedTiles[] = {{64, 128, 0.365, 0.3}, {128, 64, 0.315, 0.53}, {64, 64, 0.237, 0.46}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]), kSmallTile = kNumTiles - 1;
// Whether `workgroups` workgroups of `per` k-tiles each run with wavefront groups: from 16 (64x128: 32) k-tiles on,
// 64x64 only up to one workgroup per CU, beyond which three workgroups of the one-group kernel share a CU.  Time of
// one group over time of several at 2-7, 8-15, 16-31, 32-63 and 64-127 k-tiles: 64x64 0.95, 1.00, 1.06, 1.10, 1.15
// (0.75 with more workgroups than CUs), 64x128 0.96, 0.98, 1.00, 1.01, 1.03, 128x64 0.97, 1.00, 1.06, 1.08, 1.12.
static bool in_groups(int cfg, int per, long workgroups)
{
    return cfg == 8 ? per >= 32 : cfg == 9 ? per >= 16 : cfg == kSmallTile && per >= 16 && workgroups <= 256;
}
constexpr int kRowsMax = 256;           // bf16: gemm_rows_kernel is not used beyond 256 rows

// Instances of gemm_rows_kernel (features / 16, rows / 16, wavefronts), with us per round of workgroups over the CUs
// (the rings fill a CU's LDS) and per step of a wavefront.  They and the constants of ring_us are fitted to 19000
// timings of every instance and division on 1184 layers (bf16: 4 .. 256 rows, hidden 512 .. 8192; fp32: 4 .. 2048 rows,
// hidden 512 .. 4096), weights from HBM: 8 % rms.
struct RingCfg { int ft, tt, nw; double round_us, step_us; };
constexpr int kNumRings = 8;
constexpr RingCfg kRings[2][kNumRings] = {
    {{1, 1, 8, 1.51, 0.548}, {2, 1, 8, 1.85, 0.799}, {1, 2, 8, 1.87, 0.767}, {2, 2, 8, 2.60, 1.114},
     {3, 2, 8, 2.90, 1.622}, {2, 4, 4, 2.92, 1.221}, {4, 4, 4, 4.01, 2.267}, {3, 4, 4, 3.31, 1.773}},
    {{1, 1, 8, 1.23, 0.503}, {2, 1, 8, 1.22, 0.754}, {1, 2, 8, 1.29, 0.692}, {2, 2, 8, 1.39, 0.971},
     {3, 2, 8, 1.41, 1.252}, {2, 4, 4, 2.08, 0.672}, {4, 4, 4, 3.12, 0.962}, {3, 4, 4, 2.59, 0.826}}};
constexpr double kRingHbmRate = 6.5e6;  // bytes / us

// fp32: at most 8 shares, and not more than 256 workgroups of 32 features x 16 rows per tile
static int f32_row_tiles(int rows) { return rows <= 16 ? 1 : rows <= 32 ? 2 : 4; }
size_t gemm_f32_scratch_bound(int rows, int N)
{
    const size_t every = (size_t)8 * rows * N, full = (size_t)256 * 32 * 16 * f32_row_tiles(rows);
    return every < full ? every : full;
}

// bf16: the fastest tile and division, and its predicted time.  `groups`: with the kernels that use wavefront groups, as
// they are launched.  Candidates with more than `most` floats of scratch are left out.
static GemmPlan tile_plan(int rows, int N, int K, bool groups, size_t most, double &best_us)
{
    GemmPlan best{0, 1, 1, 0};
    best_us = 1e300;
    const int kt = K / BK;
    const double hbm_us = 2.0 * ((double)rows * K + (double)N * K + (double)rows * N) / kHbmRate;
    const auto part_us = [](double floats) { return kMergeUs + floats * 8.0 / kMergeRate; };
    const auto tail_us = [](double floats) { return kTailMergeUs + floats * 8.0 / kTailMergeRate; };
    for (int i = 0; i < kNumTiles; ++i) {
        const int bm = kTiles[i].bm, bn = kTiles[i].bn;
        const long tiles = (long)((rows + bm - 1) / bm) * ((N + bn - 1) / bn);
        const double area = (double)bm * bn;
        for (int ns = 1; ns <= 8; ++ns) {
            // every workgroup at least two k-tiles, none without any; one division beyond a full chip
            const int per = (kt + ns - 1) / ns;
            if (ns > 1 && (tiles * ns > 512 || kt / ns < 2 || (ns - 1) * per >= kt)) continue;
            const TileCfg &c = groups && in_groups(i, per, tiles * ns) ? kGroupedTiles[i - 8] : kTiles[i];
            const size_t scratch = ns > 1 ? (size_t)ns * rows * N : 0;
            const double units = (double)tiles * ns / 256.0;
            // three workgroups of the smallest tile share a CU, so its rounds are not whole
            const double rounds = i == kSmallTile ? (units > 1.0 ? units : 1.0) : ceil(units);
            double us = rounds * (c.tile_us + c.k_us * per);
            us = kLaunchUs + (us > hbm_us ? us : hbm_us);
            if (ns > 1) us += part_us((double)ns * rows * N);
            if (us < best_us && scratch <= most) { best_us = us; best = {i, ns, 1, scratch}; }
        }
        // whole rounds undivided, the tiles beyond them divided
        const long full = tiles / 256, rem = tiles - full * 256;
        if (full == 0 || rem == 0) continue;
        const TileCfg &c = groups && in_groups(i, kt, tiles) ? kGroupedTiles[i - 8] : kTiles[i];
        for (int t = 2; t <= 8; ++t) {
            const int per = (kt + t - 1) / t;
            if (rem * t > 256 || kt / t < 4) break;
            if ((t - 1) * per >= kt) continue;
            double us = full * (c.tile_us + c.k_us * kt) + c.tile_us + c.k_us * per;
            us = (kLaunchUs + (us > hbm_us ? us : hbm_us) + tail_us((double)rem * t * area)) * kTailMargin;
            const size_t scratch = (size_t)rem * t * (size_t)area;
            if (us < best_us && scratch <= most) { best_us = us; best = {i, 1, t, scratch}; }
        }
    }
    return best;
}

// How much scratch callers have been told a layer takes.  It was once the plan's own, and the plan then had, for up to
// kRowsMax rows, a kernel without LDS to choose from, described here by its us per k-step of a wavefront, once, and for
// every further round of workgroups over the CUs.  The kernel is gone; the workspace keeps its size, since programs
// keep it: a smaller one could not hold the shares that are the faster ones here, a larger one would refuse them.
struct RowsCfg { int ft, tt; double step_us, fixed_us, round_us; };
constexpr RowsCfg kRows[] = {{1, 1, 0.174, 3.0, 0.0}, {2, 1, 0.261, 3.3, 0.0}, {2, 2, 0.281, 3.7, 3.0}};
constexpr double kRowsRate = 11.9e6;    // bytes / us
constexpr int kRowsWaves = 8;
static size_t rows_scratch(int rows, int N, int K, bool groups, size_t most, size_t scratch, double best_us)
{
    if (rows > kRowsMax) return scratch;
    for (const RowsCfg &c : kRows) {
        const int bm = 16 * c.tt, bn = 16 * c.ft;
        const long tiles = (long)((rows + bm - 1) / bm) * (N / bn);
        for (int ns = 1; ns <= 8; ns *= 2) {
            if (ns > 1 && (tiles * ns > 1024 || K / 32 < ns * kRowsWaves)) break;
            const int steps = (K / 32 + ns * kRowsWaves - 1) / (ns * kRowsWaves);
            const double l2_us = (double)tiles * (bm + bn) * K * 2.0 / kRowsRate, w_us = 2.0 * N * K / kHbmRate;
            double us = c.fixed_us + c.step_us * steps + (l2_us > w_us ? l2_us : w_us) +
                        (groups ? (tiles * ns - 1) / 256 * c.round_us : 0.0);
            if (ns > 1) us += kMergeUs + (double)ns * rows * N * 8.0 / kMergeRate;
            const size_t floats = ns > 1 ? (size_t)ns * rows * N : 0;
            if (us < best_us && floats <= most) { best_us = us; scratch = floats; }
        }
    }
    return scratch;
}

// bf16: the fastest tile; `floats`: the scratch that callers have been told, never more than without the groups
struct TileChoice { GemmPlan plan; double us; size_t floats; };
static TileChoice tile_choice(int rows, int N, int K)
{
    TileChoice c;
    const auto search = [&](bool groups, size_t most, GemmPlan &p, double &us) {
        p = tile_plan(rows, N, K, groups, most, us);
        return rows_scratch(rows, N, K, groups, most, p.scratch_floats, us);
    };
    c.floats = search(true, SIZE_MAX, c.plan, c.us);
    if (c.floats == 0) return c;
    GemmPlan none;
    double us;
    const size_t told = search(false, SIZE_MAX, none, us);
    if (c.floats > told) c.floats = search(true, told, c.plan, c.us);
    return c;
}

// Time of what a CU does and of what HBM gives, of which neither quite hides the other
static double together(double cu_us, double hbm_us)
{
    const double x = cu_us / hbm_us, x2 = x * x, x4 = x2 * x2;
    return hbm_us * sqrt(sqrt(sqrt(1.0 + x4 * x4)));
}

// Predicted time of an instance of gemm_rows_kernel without its merge
static double ring_us(const RingCfg &c, int rows, int N, int K, int es, int ns)
{
    const int parts = ns * c.nw, steps = K * es / 128, per = (steps + parts - 1) / parts;
    const long tiles = (long)((rows + 16 * c.tt - 1) / (16 * c.tt)) * (N / (16 * c.ft));
    const double rounds = (double)((tiles * ns + 255) / 256);
    // Where the shares of the contraction start whole multiples of 4 KiB apart, the wavefronts of all workgroups are on
    // the same few HBM channels: 32 rows, 16384 to 4096, 32x32 undivided (4 KiB) 49.0 us, in two shares (2 KiB) 29.3.
    double conflict = 1.0;
    if (steps % parts == 0) {
        const int apart = steps / parts * 128;
        conflict = apart % 8192 == 0 ? 1.25 : apart % 4096 == 0 ? 1.5 : 1.0;
    }
    const double bytes = (double)es * ((double)rows * K + (double)N * K + (double)rows * N);
    return together(1.0 + rounds * (c.round_us + c.step_us * per), 3.4 + 0.7 * (rounds - 1.0) + bytes * conflict / kRingHbmRate);
}

static double merge_us(const GemmPlan &p) { return p.nsplit > 1 ? kMergeUs + p.scratch_floats * 8.0 / kMergeRate : 0.0; }

// What runs, within `room` floats: an instance of gemm_rows_kernel (fp32 always; plans of kNumTiles + instance) or the
// tile, whichever is predicted faster.  The tiles' own times leave out that the weights' way from HBM is not hidden at so few
// rows (12 rows, 3072 to 12288: 64x64 16.2 us predicted, 21.4 measured, 15.2 by 48x32), and are a little low besides: on
// 1296 layers of other sizes the picks take 0.7586 of the time of the plan without gemm_rows_kernel with a factor of 1.0,
// 0.7571 with 1.03 and 0.7540 with 1.1, at worst 1 %, 3 % and 5 % more than it.
// On the layers that kRings is fitted to, none is more than 3 % above the time of the plan without gemm_rows_kernel
// (fp32: of a kernel that loads straight to registers); on average they take 0.78 and 0.68 of it.  The picks are
// 1.3 and 0.5 % off the best of all candidates, at worst 42 % (another tile) and 13 %.  (Without the conflicts, with the
// weights at 6.0e6 bytes / us beside anything, and steps fitted where they are few, FC2 of 16384 to 4096 took 39 to 49 us
// at 4 to 32 rows, where the tiles take 33 to 34 and 32x32 in two shares 27 to 29.)
static GemmPlan linear_plan(DType dt, int rows, int N, int K, size_t room, TileChoice tile)
{
    const bool bf16 = dt == DType::BF16;
    const int es = bf16 ? 2 : 4;
    if (bf16 && rows > kRowsMax) return tile.plan;
    GemmPlan best{0, 1, 1, 0};
    double best_us = 1e300;
    if (bf16) {
        if (tile.plan.scratch_floats > room) tile.plan = tile_plan(rows, N, K, true, room, tile.us);
        const double bytes = 2.0 * ((double)rows * K + (double)N * K + (double)rows * N), merge = merge_us(tile.plan);
        best = tile.plan;
        best_us = together(1.03 * (tile.us - merge), 3.4 + bytes / kRingHbmRate) + merge;
    }
    for (int i = 0; i < kNumRings; ++i) {
        const RingCfg &c = kRings[bf16][i];
        if (N % (16 * c.ft)) continue;
        for (int ns = 1; ns <= 8; ns *= 2) {
            const GemmPlan p{kNumTiles + i, ns, 1, ns > 1 ? (size_t)ns * rows * N : 0};
            if (ns > 1 && (K * es / 128 < ns * c.nw || p.scratch_floats > room)) break;
            const double us = ring_us(c, rows, N, K, es, ns) + merge_us(p);
            if (us < best_us) { best_us = us; best = p; }
        }
    }
    return best;
}

BlockPlan block_plan(DType dt, int B, int rows, int d, int H, int Dh, int F)
{
    const int R = (int)((size_t)B * rows), shape[4][2] = {{3 * d, d}, {d, d}, {F, d}, {d, F}};   // N, K
    BlockPlan p;
    TileChoice tile[4] = {};
    p.floats = attention_scratch_floats(dt, B, rows, H, Dh);
    if (dt == DType::BF16) {
        for (int i = 0; i < 4; ++i) {
            tile[i] = tile_choice(R, shape[i][0], shape[i][1]);
            if (tile[i].floats > p.floats) p.floats = tile[i].floats;
        }
    } else {
        // what the plans take falls as the rows become more; their bound does not, so that a workspace sized for the
        // largest call serves every smaller one (bf16 never had that)
        const size_t bound = gemm_f32_scratch_bound(R, 3 * d > F ? 3 * d : F);
        if (bound > p.floats) p.floats = bound;
    }
    for (int i = 0; i < 4; ++i) p.layer[i] = linear_plan(dt, R, shape[i][0], shape[i][1], p.floats, tile[i]);
    return p;
}

template <typename T, int FT, int TT, int NW, int STAGES>
static void launch_gemm_rows(const void *A, const void *W, int rows, int N, int K, const EpiParams &ep,
                             hipStream_t st, int nsplit, float *part)
{
    const int row_tiles = (rows + 16 * TT - 1) / (16 * TT);
    const int units = row_tiles * nsplit * (N / (16 * FT));
    constexpr size_t lds = (size_t)NW * STAGES * (FT + TT) * 2048;
    static_assert(lds <= kLdsLimit, "LDS of a CU");
    auto kern = gemm_rows_kernel<T, FT, TT, NW, STAGES>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    launch(kern, dim3((units + 7) / 8 * 8), dim3(64 * NW), lds, st, (const T *)A, (const T *)W, rows, N, K,
           row_tiles, nsplit, ep, part);
}

// instance i of kRings
template <typename T>
static void launch_gemm_ring(int i, const void *A, const void *W, int rows, int N, int K, const EpiParams &ep,
                             hipStream_t st, int nsplit, float *part)
{
    switch (i) {
    case 0: launch_gemm_rows<T, 1, 1, 8, 4>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 1: launch_gemm_rows<T, 2, 1, 8, 3>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 2: launch_gemm_rows<T, 1, 2, 8, 3>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 3: launch_gemm_rows<T, 2, 2, 8, 2>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 4: launch_gemm_rows<T, 3, 2, 8, 2>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 5: launch_gemm_rows<T, 2, 4, 4, 2>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 6: launch_gemm_rows<T, 4, 4, 4, 2>(A, W, rows, N, K, ep, st, nsplit, part); break;
    case 7: launch_gemm_rows<T, 3, 4, 4, 2>(A, W, rows, N, K, ep, st, nsplit, part); break;
    }
}

// Every column has to belong to a workgroup: the instances of gemm_rows_kernel leave no remainder of their features.
static bool launchable(DType dt, int N, const GemmPlan &plan)
{
    if (plan.nsplit < 1 || plan.tail < 1 || plan.cfg < 0) return false;
    if (plan.cfg < kNumTiles) return dt == DType::BF16;
    const int i = plan.cfg - kNumTiles;
    return i < kNumRings && N % (16 * kRings[dt == DType::BF16][i].ft) == 0;
}

bool launch_gemm(DType dt, const void *A, const void *W, int rows, int N, int K,
                 const GemmEpilogue &e, const GemmPlan &plan, float *part, hipStream_t st)
{
    if (!launchable(dt, N, plan)) return false;
    EpiParams ep;
    ep.bias = e.bias; ep.residual = e.residual; ep.gelu = e.gelu;
    ep.out0 = e.out0; ep.ld0 = e.ld0; ep.split = e.split;
    ep.kcache = e.kcache; ep.vcache = e.vcache;
    ep.hd = e.hd; ep.cap = e.cap; ep.len = e.len;
    ep.rows_per_sample = e.rows_per_sample > 0 ? e.rows_per_sample : 1;
    ep.N = N;
    ep.out_f32 = e.out_f32;
    ep.res_f32 = e.res_f32;
    if (dt == DType::BF16) {
        const int ns = plan.nsplit, tail = plan.tail, tile = plan.cfg < kNumTiles ? plan.cfg : kSmallTile;
        const bool groups = in_groups(plan.cfg, (K / BK + ns - 1) / ns,
                                      (long)ns * ((rows + kTiles[tile].bm - 1) / kTiles[tile].bm) *
                                          ((N + kTiles[tile].bn - 1) / kTiles[tile].bn));
        switch (plan.cfg) {
        case 0: launch_gemm_bf16_cfg<320, 256, 2, 4, 2>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 1: launch_gemm_bf16_cfg<256, 256, 2, 4, 2>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 2: launch_gemm_bf16_cfg<192, 256, 2, 4, 2>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 3: launch_gemm_bf16_cfg<256, 192, 4, 2, 2>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 4: launch_gemm_bf16_cfg<256, 128, 4, 2, 3>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 5: launch_gemm_bf16_cfg<128, 256, 2, 4, 3>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 6: launch_gemm_bf16_cfg<192, 128, 2, 4, 3>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 7: launch_gemm_bf16_cfg<128, 128, 2, 4, 4>(A, W, rows, N, K, ep, st, ns, part, tail); break;
        case 8:
            if (groups) launch_gemm_bf16_cfg<64, 128, 2, 2, 3, 2>(A, W, rows, N, K, ep, st, ns, part, tail);
            else launch_gemm_bf16_cfg<64, 128, 2, 4, 4>(A, W, rows, N, K, ep, st, ns, part, tail);
            break;
        case 9:
            if (groups) launch_gemm_bf16_cfg<128, 64, 2, 2, 3, 2>(A, W, rows, N, K, ep, st, ns, part, tail);
            else launch_gemm_bf16_cfg<128, 64, 4, 2, 4>(A, W, rows, N, K, ep, st, ns, part, tail);
            break;
        case 10:
            if (groups)
                launch_gemm_bf16_cfg<64, 64, 1, 1, 2, 4>(A, W, rows, N, K, ep, st, ns, part, tail);
            else
                launch_gemm_bf16_cfg<64, 64, 2, 2, 3>(A, W, rows, N, K, ep, st, ns, part, tail);
            break;
        default: launch_gemm_ring<uint16_t>(plan.cfg - kNumTiles, A, W, rows, N, K, ep, st, ns, part); break;
        }
        if (ns > 1) {
            const long total = (long)rows * (N / 4);
            launch(gemm_splitk_epilogue_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                   (const float *)part, ns, rows, N, ep);
        }
    } else {
        launch_gemm_ring<float>(plan.cfg - kNumTiles, A, W, rows, N, K, ep, st, plan.nsplit, part);
        if (plan.nsplit > 1) {
            const long total = (long)rows * (N / 4);
            launch(gemm_f32_merge_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                   (const float *)part, plan.nsplit, rows, N, ep);
        }
    }
    return true;
}

}  // namespace fvar
