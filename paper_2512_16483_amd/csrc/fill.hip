// Restoration of the full token map (paper, Eq. "redefine"; cached rows in the rank-r restored
// form W_r F_r of Sec. "Random Projection (RP) for Low-Rank Feature" / Eq. "lstsq").
//
//   kept rows    y[b, idx_keep[b,j], :] = y_keep[b,j,:]         one wavefront per row, 16 B/lane
//   pruned rows  y[b, i, :] = w_c[b,i,:] . g_c[b]               thin GEMM, K = r
//
// The pruned part writes (M-k)*d elements per sample and does 2*r flops for each: at r = 64 that
// is 64 flop per written byte in bf16, far above what the vector ALUs can feed at HBM speed, so
// the bf16 path runs it on MFMA with fp32 accumulation and stays bound by the output write.
// A workgroup owns a 128-column slab of g_c[b]: the slab travels global -> LDS by DMA once, in
// its own row-major layout, and the workgroup streams its share of the pruned rows past it.
// The product is formed transposed (slab columns are the MFMA rows, token rows the MFMA columns)
// so that a lane ends up with 4 consecutive output columns of one token row: the slab operand,
// which the MFMA wants k-contiguous, is fetched with the transposing LDS load
// (ds_read_b64_tr_b16), the w_c rows go straight from global memory into the other operand, one
// row group ahead of the MFMAs that use them.
//
// Optionally every workgroup also leaves, per output row, the sum of squares of the values it
// stored (exact products of the stored elements, fp64 sum): the row energies of the map, i.e. the
// selection scores of the NEXT block (paper, Sec. "Representative Token Restoration"), so that
// the next block does not have to read the map again.
#include <type_traits>

#include "common.h"

namespace fvar {

// sum over the `width` (power of two, <= 64) consecutive lanes of a group
__device__ __forceinline__ double group_sum(double v, int width)
{
    for (int o = width >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// 16 bytes of the restored map; PAST: past the caches (nontemporal), see map_past_caches
template <bool PAST> __device__ __forceinline__ void store_map(void *dst, const uint4 &v)
{
    typedef uint32_t uintx4_t __attribute__((ext_vector_type(4)));
    if constexpr (PAST) __builtin_nontemporal_store(uintx4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<uintx4_t *>(dst));
    else *reinterpret_cast<uint4 *>(dst) = v;
}

// Whether a restored map of that many bytes is written past the caches.  What counts is the map's next reader, the
// score pass (scored fills: the gather) of the next block: from 20 % more than the 256 MB of last-level cache on
// next to nothing of the map is still there when it comes, and stores past the caches spare y_keep, w_c and the
// weights; a small map's dirty lines leave the L2s sooner that way.  In between, the reader finds the map in
// the cache.  Score + LayerNorm gather + fill in a chain of blocks, ordinary -> past the caches, us: 9 MB 13.6 -> 13.1,
// 19 16.4 -> 15.5, 38 27.0 -> 28.2, 105 60.0 -> 61.1, 164 95.1 -> 103.6, 210 115.5 -> 126.7, 268 146.8 -> 151.2,
// 302 173.8 -> 179.3, 333 211 -> 204, 380 233 -> 215, 537 342 -> 294; with scores (no score pass) 9 MB 13.6 -> 13.0,
// 38 26.2 -> 24.9 and 31.3 -> 31.7, 75 37.4 -> 41.4, 210 89.0 -> 98.1, 268 115.2 -> 115.9, 333 156.5 -> 157.4,
// 419 183.6 -> 174.0.  Fills that follow each other without a reader see it otherwise (210 MB 63.6 -> 48.0).
bool map_past_caches(size_t bytes, bool scored)
{
    return bytes <= (scored ? 40u : 24u) * 1000000 || bytes > (size_t)256 * 1024 * 1024 / 5 * 6;
}

// sum of squares of the 8 bf16 (4 fp32) elements of a 16-byte chunk, in fp64
template <typename T> __device__ __forceinline__ double chunk_energy(const uint4 &c)
{
    float f[Elem<T>::kPerChunk];
    Elem<T>::unpack(c, f);
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < Elem<T>::kPerChunk; ++e) acc = fma((double)f[e], (double)f[e], acc);
    return acc;
}

// ------------------------------------------------------------------ kept rows: scatter
// Workgroup `blk` of the scatter part: four rows, one per wavefront.  With `parts` the row's
// energy goes to part 0 of the row and zeros to its other parts.
template <typename T, bool PAST>
__device__ __forceinline__ void scatter_rows(int blk, const T *__restrict__ y_keep,
                                             const int32_t *__restrict__ idx_keep, int M, int k,
                                             int total_rows, int d, T *__restrict__ y,
                                             double *__restrict__ parts, int nparts)
{
    constexpr int E = Elem<T>::kPerChunk;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blk * 4 + wave;
    if (row >= total_rows) return;
    const int b = row / k;
    const int dst_row = idx_keep ? idx_keep[row] : row - b * k;
    const uint4 *src = reinterpret_cast<const uint4 *>(y_keep + (size_t)row * d);
    uint4 *dst = reinterpret_cast<uint4 *>(y + ((size_t)b * M + dst_row) * d);
    const int nchunk = d / E;
    double e = 0.0;
    int c = lane;
    for (; c + 192 < nchunk; c += 256) {            // four chunks in flight per lane
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[c + 64 * u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            store_map<PAST>(dst + c + 64 * u, v[u]);
            if (parts) e += chunk_energy<T>(v[u]);
        }
    }
    for (; c < nchunk; c += 64) {
        const uint4 v = src[c];
        store_map<PAST>(dst + c, v);
        if (parts) e += chunk_energy<T>(v);
    }
    if (parts) {
        e = group_sum(e, 64);
        double *pr = parts + ((size_t)b * M + dst_row) * nparts;
        if (lane < nparts) pr[lane] = lane == 0 ? e : 0.0;
    }
}

// ------------------------------------------------------------------ pruned rows, bf16 MFMA
constexpr int kFillCols = 128;              // column slab per workgroup (16 chunks of 16 B per row)
constexpr int kFillStage = 64;              // row pitch (elements) of the per-wavefront output staging

typedef short fill_shortx4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void fill_dma_b128(const void *base, uint32_t byte_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}

// Bound by the output's way to memory, as long as every wavefront keeps stores in flight: 4 x 6400 rows of 4096,
// keep 1/4, rank 128: 68.4 -> 57.9 us in a chain of blocks, 73.3 -> 63.6 one after the other (a plain fill of the
// same map takes 33 and its kept rows' copy 20), 32 x 1600 of 2048, keep 0.3, rank 64: 56.7 -> 52.0 and
// 63.1 -> 58.2.  Before, a group's stores waited for indices that
// queued behind the stores of the group before it, every MFMA for its own LDS read, and 30 % of the LDS cycles
// were bank conflicts (21 % with the staging tile swizzled, which is worth 0.88 of the time over 224 shapes).
// Workgroups are numbered so that an XCD gets all slabs of its rows: it then writes whole rows (slabs dealt
// round robin put every eighth slab of all rows on one XCD: 13.6 -> 12.0 us with scores, 4096 rows of 2048).
// One launch does both parts: workgroups [0, fill_blocks) restore pruned rows (slab, row share and
// sample decoded from the block id), the workgroups after them copy kept rows.
// KSTEPS >= ceil(r / 16): 16-wide steps of the contraction, of which the first kFillWholeSteps are whole at
// every rank that gets this KSTEPS.
template <int KSTEPS>
constexpr int kFillWholeSteps = KSTEPS <= 4 ? KSTEPS - 1 : KSTEPS == 6 ? 4 : KSTEPS == 8 ? 6 : KSTEPS == 12 ? 8 : 12;
template <int KSTEPS, bool SCORED, bool PAST>
__global__ __launch_bounds__(256, KSTEPS + SCORED <= 8 ? 3 : 2) void fill_bf16_kernel(const uint16_t *__restrict__ y_keep,
                                                        const int32_t *__restrict__ idx_keep,
                                                        const int32_t *__restrict__ idx_drop, int M,
                                                        int k, int B, int r, int d,
                                                        const uint16_t *__restrict__ w_c,
                                                        const uint16_t *__restrict__ g_c,
                                                        uint16_t *__restrict__ y, int slabs,
                                                        int row_split, int fill_blocks,
                                                        double *__restrict__ parts)
{
    if ((int)blockIdx.x >= fill_blocks) {
        scatter_rows<uint16_t, PAST>(blockIdx.x - fill_blocks, y_keep, idx_keep, M, k, B * k, d, y, parts, slabs);
        return;
    }
    constexpr int RP = KSTEPS * 16;                           // slab rows in LDS (k extent, padded)
    const int nd = M - k;
    const int unit = xcd_contiguous(blockIdx.x, fill_blocks);
    const int slab = unit % slabs, share = (unit / slabs) % row_split;
    const int b = unit / (slabs * row_split);
    extern __shared__ uint4 lds_raw[];
    uint16_t *gs = reinterpret_cast<uint16_t *>(lds_raw);     // [RP][kFillCols], chunks swizzled
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds_raw;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rl = lane & 31, g = lane >> 5;
    uint16_t *wl = gs + RP * kFillCols + wave * (32 * kFillStage);   // output staging of this wavefront
    const int col0 = slab * kFillCols;
    const uint16_t *G = g_c + (size_t)b * r * d;
    const uint16_t *W = w_c + (size_t)b * M * r;
    const int32_t *drop = idx_drop + (size_t)b * nd;
    uint16_t *Y = y + (size_t)b * M * d;

    // ---- the slab: rows t of g_c[b], columns col0 .. col0+127, 4 rows (1 KiB) per DMA instruction.
    // Lane l fills physical chunk l%16 of row 4*group + l/16 with the logical chunk that the
    // swizzle (chunk ^ 4*(row%4)) maps there.  Rows past r repeat row r-1 (their products meet
    // zeros of the other operand), columns past d repeat the last chunk (never stored).
    for (int grp = wave; grp < RP / 4; grp += 4) {
        const int t = min(grp * 4 + lane / 16, r - 1);
        const int lc = (lane % 16) ^ ((t & 3) << 2);
        const int col = min(col0 + lc * 8, d - 8);
        fill_dma_b128(G, (uint32_t)(((size_t)t * d + col) * 2), lds_base + grp * 1024);
    }

    // ---- operand addressing
    // transposing read of the slab: lane l = 16*Gq + 4*j + a points at slab row 8*(Gq/2) + j (+ 16s,
    // + 4 for the second read) and columns 16*(Gq%2) + 4*a .. +3 (+ 32*cb); it receives, for
    // MFMA row (slab column) 16*(Gq%2) + l%16 of block cb, the k-slots 8*(Gq/2) + 0..3 (+4)
    const int tG = lane >> 4, tj = (lane >> 2) & 3, ta = lane & 3;
    const int g_lane = (8 * (tG >> 1) + tj) * kFillCols + ((2 * (tG & 1) + (ta >> 1)) << 3) + (ta & 1) * 4;
    // rows of this workgroup: 32-row groups it, it + row_split*4 ... per wavefront
    const int groups = (nd + 31) / 32;
    const int gstep = row_split * 4;
    int grp_row = share * 4 + wave;                             // this wavefront's current group

    // other operand: lane (row rl, half g) holds w_c[row][16s + 8g .. +8), zeros past r.
    // The token row of a slot comes from idx_drop: that index is fetched two groups ahead of the
    // MFMAs (one group ahead of the w_c fragments it addresses), so neither the fragment loads nor
    // the stores wait for an index at the moment they are issued.
    // Loads and stores of a wavefront complete in one order, so a load that is waited for in the group that
    // issues it, or whose place among the stores the compiler does not know, waits for all stores before it
    // to reach memory.  Hence no branch around a load or a store: slots past the last row repeat that row,
    // result and all.
    uint4 afrag[2][KSTEPS];
    auto load_row = [&](int grpi) { return drop[min(grpi * 32 + rl, nd - 1)]; };
    auto load_a = [&](int row, uint4 *dst) {
        const uint16_t *wrow = W + (size_t)row * r;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            const int t = 16 * s + 8 * g;
            dst[s] = *reinterpret_cast<const uint4 *>(wrow + (s < kFillWholeSteps<KSTEPS> ? t : min(t, r - 8)));
        }
    };
    int row_cur = load_row(grp_row), row_next = load_row(grp_row + gstep);   // token row of this lane
    load_a(row_cur, afrag[0]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // one 32-row group: af holds its w_c fragments, af_next receives those of the next group
    auto group = [&](int grp_row, const uint4 *af, uint4 *af_next) {
        // destination rows of the 4 row-chunks this lane stores per half (rows it*8 + lane/8)
        int orow[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) orow[it] = __shfl(row_cur, it * 8 + (lane >> 3));
        row_cur = row_next;
        load_a(row_next, af_next);
        row_next = load_row(grp_row + 2 * gstep);
        double erow[4] = {0.0, 0.0, 0.0, 0.0};
        // two halves of 64 columns (one, where the row ends in between): 2 x 32-column accumulator tiles each
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half == 1 && col0 + 64 >= d) break;            // uniform
            typedef __attribute__((address_space(3))) fill_shortx4_t lds_shortx4_t;
            // slab fragments, one step ahead of the MFMAs that use them
            bf16x8_t gf[2][2];
            auto load_g = [&](int s, bf16x8_t *dst) {
#pragma unroll
                for (int c2 = 0; c2 < 2; ++c2) {
                    const int cb = half * 2 + c2;
                    const uint16_t *src = gs + g_lane + 16 * s * kFillCols + ((cb ^ tj) << 5);
                    const fill_shortx4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t *)src);
                    const fill_shortx4_t hi =
                        __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t *)(src + 4 * kFillCols));
                    dst[c2] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            };
            floatx16_t acc[2] = {floatx16_t{0}, floatx16_t{0}};
            load_g(0, gf[0]);
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                if (s + 1 < KSTEPS) load_g(s + 1, gf[(s + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                const uint4 av = s < kFillWholeSteps<KSTEPS> || 16 * s + 8 * g < r ? af[s] : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int c2 = 0; c2 < 2; ++c2)
                    acc[c2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        gf[s & 1][c2], __builtin_bit_cast(bf16x8_t, av), acc[c2], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // accumulator entry e of tile c2: token row rl, slab column 32*cb + 8*(e/4) + 4*g + e%4.
            // Pack 4 consecutive columns and park them row-major in this wavefront's staging tile, whose
            // 16-byte chunks are swizzled (chunk ^ (row / 2) % 8) and, from row 16 on, have their halves
            // swapped: 32 lanes that write (8 bytes of 32 rows) and 16 that read (two rows) then cover all 64
            // banks once.  (The conflicts that the counters still show are the slab's reads or lanes served in
            // another order; which, they do not say.)
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint2 pk;
                    pk.x = pack_bf16x2(acc[c2][4 * q], acc[c2][4 * q + 1]);
                    pk.y = pack_bf16x2(acc[c2][4 * q + 2], acc[c2][4 * q + 3]);
                    *reinterpret_cast<uint2 *>(wl + rl * kFillStage + (((c2 * 4 + q) ^ ((rl >> 1) & 7)) << 3) +
                                               4 * (g ^ (rl >> 4))) = pk;
                }
            // same wavefront wrote and reads the region: LDS operations of a wavefront stay in order
            // in hardware; the compiler is told not to move them across these points (the stores
            // and loads use different vector types).
            // 8 lanes cover the 128 bytes of one row half: 8 rows per store instruction.
            asm volatile("" ::: "memory");
            uint4 v[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int lrow = it * 8 + (lane >> 3);
                v[it] = *reinterpret_cast<const uint4 *>(wl + lrow * kFillStage +
                                                         (((lane & 7) ^ ((lrow >> 1) & 7)) << 3));
                if (it >= 2) v[it] = make_uint4(v[it].z, v[it].w, v[it].x, v[it].y);
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                store_map<PAST>(Y + (size_t)orow[it] * d + col0 + half * 64 + (lane & 7) * 8, v[it]);
                if (SCORED) erow[it] += chunk_energy<uint16_t>(v[it]);
            }
            asm volatile("" ::: "memory");
        }
        // the 8 lanes of a group hold the pieces of one row; the lane at their head owns rows
        // it*8 + lane/8 of the group
        if constexpr (SCORED) {
            double e8[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) e8[it] = group_sum(erow[it], 8);
            if ((lane & 7) == 0) {
#pragma unroll
                for (int it = 0; it < 4; ++it) parts[((size_t)b * M + orow[it]) * slabs + slab] = e8[it];
            }
        }
    };
    for (; grp_row < groups; grp_row += 2 * gstep) {
        group(grp_row, afrag[0], afrag[1]);
        if (grp_row + gstep < groups) group(grp_row + gstep, afrag[1], afrag[0]);
    }
}

// ------------------------------------------------------------------ pruned rows, fp32 FMA
__global__ __launch_bounds__(256) void fill_f32_kernel(const float *__restrict__ y_keep,
                                                       const int32_t *__restrict__ idx_keep,
                                                       const int32_t *__restrict__ idx_drop, int M,
                                                       int k, int B, int r, int d,
                                                       const float *__restrict__ w_c,
                                                       const float *__restrict__ g_c,
                                                       float *__restrict__ y, int fill_blocks,
                                                       double *__restrict__ parts)
{
    __shared__ float wrow[256];
    __shared__ double esum[4];
    if ((int)blockIdx.x >= fill_blocks) {
        scatter_rows<float, false>(blockIdx.x - fill_blocks, y_keep, idx_keep, M, k, B * k, d, y, parts, 1);
        return;
    }
    const int nd = M - k;
    const int b = blockIdx.x / nd, j = blockIdx.x % nd;
    const int i = idx_drop[(size_t)b * nd + j];
    const float *W = w_c + ((size_t)b * M + i) * r;
    const float *G = g_c + (size_t)b * r * d;
    for (int t = threadIdx.x; t < r; t += 256) wrow[t] = W[t];
    __syncthreads();
    float *out = y + ((size_t)b * M + i) * d;
    double e = 0.0;
    for (int c = threadIdx.x * 4; c < d; c += 1024) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int t = 0; t < r; ++t) {
            const float w = wrow[t];
            const float4 gv = *reinterpret_cast<const float4 *>(G + (size_t)t * d + c);
            acc.x = fmaf(w, gv.x, acc.x); acc.y = fmaf(w, gv.y, acc.y);
            acc.z = fmaf(w, gv.z, acc.z); acc.w = fmaf(w, gv.w, acc.w);
        }
        *reinterpret_cast<float4 *>(out + c) = acc;
        e = fma((double)acc.x, (double)acc.x, e); e = fma((double)acc.y, (double)acc.y, e);
        e = fma((double)acc.z, (double)acc.z, e); e = fma((double)acc.w, (double)acc.w, e);
    }
    if (parts) {                                            // uniform
        e = group_sum(e, 64);
        if ((threadIdx.x & 63) == 0) esum[threadIdx.x >> 6] = e;
        __syncthreads();
        if (threadIdx.x == 0) parts[(size_t)b * M + i] = (esum[0] + esum[1]) + (esum[2] + esum[3]);
    }
}

// Row energies of the restored map from the per-slab parts: scores[row] = fl32(sum of the row's
// parts).  `width` neighbouring lanes (a power of two, at most 16) share a row: with one thread per row the
// 4096 rows of a single image are 16 workgroups, each a chain of 16 loads 128 bytes apart.
__global__ __launch_bounds__(256) void scores_from_parts_kernel(const double *__restrict__ parts,
                                                                int nparts, int width, long rows,
                                                                float *__restrict__ scores)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x, row = t / width;
    const int l = (int)(t % width);
    if (row >= rows) return;                               // the lanes of a row together
    const double *p = parts + (size_t)row * nparts;
    double acc = 0.0;
    for (int i = l; i < nparts; i += width) acc += p[i];
    acc = group_sum(acc, width);
    if (l == 0) scores[row] = (float)acc;
}

// ------------------------------------------------------------------ raw cached rows
// Eq. "redefine" as printed: kept rows come from the block output, every other row is the cached
// counterpart row itself.  One wavefront per output row: the first B*k rows of the launch scatter
// y_keep, the remaining B*(M-k) copy row idx_drop[b,j] of the cache to the same position of y.
// PAST: the kept rows are stored past the caches, where the map does not fit the last-level cache of 256 MB
// (score + fill in a chain, ordinary -> past, us: 16 MB 10.8 -> 11.5, 63 35.2 -> 36.5, 210 98.8 -> 98.5,
// 262 133.4 -> 129.6, 302 170.6 -> 165.1, 537 302.5 -> 293.0).
template <typename T, bool PAST>
__global__ __launch_bounds__(256) void cache_fill_kernel(const T *__restrict__ y_keep,
                                                         const int32_t *__restrict__ idx_keep,
                                                         const int32_t *__restrict__ idx_drop, int M,
                                                         int k, int B, int d,
                                                         const T *__restrict__ cache,
                                                         T *__restrict__ y)
{
    constexpr int E = Elem<T>::kPerChunk;
    const int kept_blocks = (B * k + 3) / 4;
    if ((int)blockIdx.x < kept_blocks) {
        scatter_rows<T, PAST>(blockIdx.x, y_keep, idx_keep, M, k, B * k, d, y, nullptr, 0);
        return;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nd = M - k;
    const int j = (blockIdx.x - kept_blocks) * 4 + wave;
    if (j >= B * nd) return;                       // also covers nd == 0
    const int b = j / nd;
    const size_t row = (size_t)b * M + idx_drop[j];
    const uint4 *src = reinterpret_cast<const uint4 *>(cache + row * d);
    uint4 *dst = reinterpret_cast<uint4 *>(y + row * d);
    const int nchunk = d / E;
    for (int c = lane; c < nchunk; c += 64) dst[c] = src[c];
}

void launch_cache_fill(DType dt, const void *y_keep, const int32_t *idx_keep, const int32_t *idx_drop,
                       int B, int M, int k, int d, const void *cache, void *y, hipStream_t st)
{
    // cache == y: the pruned rows are in place already and only the kept rows are written
    const int copy_rows = cache == y ? 0 : B * (M - k);
    const int blocks = (B * k + 3) / 4 + (copy_rows + 3) / 4;
    if (blocks == 0) return;
    const bool past = dt == DType::BF16 && (size_t)B * M * d * sizeof(uint16_t) > 256u * 1000000;
    auto run = [&](auto kern, auto *t) {
        typedef std::remove_pointer_t<decltype(t)> T;
        launch(kern, dim3(blocks), dim3(256), 0, st, (const T *)y_keep, idx_keep, idx_drop, M, k, B, d, (const T *)cache,
               (T *)y);
    };
    if (dt != DType::BF16) run(cache_fill_kernel<float, false>, (float *)nullptr);
    else if (past) run(cache_fill_kernel<uint16_t, true>, (uint16_t *)nullptr);
    else run(cache_fill_kernel<uint16_t, false>, (uint16_t *)nullptr);
}

// parts per output row that launch_fill leaves when row energies are requested
int fill_score_parts(DType dt, int d)
{
    return dt == DType::BF16 ? (d + kFillCols - 1) / kFillCols : 1;
}

// Workgroups that share the pruned rows of one slab: one round of the two that a CU holds at every rank, rounded
// down, and no more than there are 32-row groups for their four wavefronts.  Each stages its slab once.  Against 768
// in all, rounded up, which is one and a half rounds from rank 136 (with scores 104) on and a little over one where
// 768 is no multiple of the slabs: 6400 x 4096 rank 64 15.7 -> 13.9 us, rank 256 26.6 -> 23.5, 7 x 1600 x 4096
// rank 160 32.1 -> 27.8, 16 x 1024 x 4096 rank 128 49.6 -> 45.6, 4 x 6400 x 4096 rank 128 65.6 -> 64.6, on average
// over 168 shapes 0.967 (0.87 to 1.05); 1024 workgroups 1.007, 1536 1.02.
int fill_row_split(int slabs, int nd)
{
    const int most = ((nd + 31) / 32 + 3) / 4, round = slabs < 512 ? 512 / slabs : 1;
    return round < most ? round : most;
}

template <int KSTEPS>
static void launch_fill_bf16(const void *y_keep, const int32_t *idx_keep, const int32_t *idx_drop, int B,
                             int M, int k, int r, int d, const void *w_c, const void *g_c, void *y,
                             double *parts, bool past, hipStream_t st)
{
    const int nd = M - k;
    const int scatter_blocks = (B * k + 3) / 4;
    const int slabs = (d + kFillCols - 1) / kFillCols;
    const int row_split = fill_row_split(slabs * B, nd);
    const int fill_blocks = slabs * row_split * B;
    const size_t lds = nd > 0 ? ((size_t)KSTEPS * 16 * kFillCols + 4 * 32 * kFillStage) * sizeof(uint16_t) : 0;
    auto kern = parts ? past ? fill_bf16_kernel<KSTEPS, true, true> : fill_bf16_kernel<KSTEPS, true, false>
                      : past ? fill_bf16_kernel<KSTEPS, false, true> : fill_bf16_kernel<KSTEPS, false, false>;
    if (lds > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (fill_blocks + scatter_blocks == 0) return;
    launch(kern, dim3(fill_blocks + scatter_blocks), dim3(256), lds, st, (const uint16_t *)y_keep, idx_keep,
           idx_drop, M, k, B, r, d, (const uint16_t *)w_c, (const uint16_t *)g_c, (uint16_t *)y, slabs,
           row_split, fill_blocks, parts);
}

// parts: null, or B*M*fill_score_parts() doubles that receive the energy of every output row in
// parts; scores_out (with parts): [B*M] fp32 row energies, summed from the parts by a second kernel.  past: bf16
// maps are written past the caches
void launch_fill(DType dt, const void *y_keep, const int32_t *idx_keep, const int32_t *idx_drop,
                 int B, int M, int k, int r, int d, const void *w_c, const void *g_c, void *y,
                 double *parts, float *scores_out, bool past, hipStream_t st)
{
    const int nd = M - k;
    const int scatter_blocks = (B * k + 3) / 4;
    if (dt == DType::BF16) {
        const int ks = nd > 0 ? (r + 15) / 16 : 1;
#define FVAR_FILL(KS) launch_fill_bf16<KS>(y_keep, idx_keep, idx_drop, B, M, k, r, d, w_c, g_c, y, parts, past, st)
        if (ks <= 1) FVAR_FILL(1);
        else if (ks <= 2) FVAR_FILL(2);
        else if (ks <= 3) FVAR_FILL(3);
        else if (ks <= 4) FVAR_FILL(4);
        else if (ks <= 6) FVAR_FILL(6);
        else if (ks <= 8) FVAR_FILL(8);
        else if (ks <= 12) FVAR_FILL(12);
        else FVAR_FILL(16);
#undef FVAR_FILL
    } else {
        const int fill_blocks = nd * B;
        if (fill_blocks + scatter_blocks > 0)
            launch(fill_f32_kernel, dim3(fill_blocks + scatter_blocks), dim3(256), 0, st,
                   (const float *)y_keep, idx_keep, idx_drop, M, k, B, r, d, (const float *)w_c,
                   (const float *)g_c, (float *)y, fill_blocks, parts);
    }
    if (parts && scores_out) {
        const long rows = (long)B * M;
        const int nparts = fill_score_parts(dt, d);
        int width = 1;
        while (2 * width <= nparts && width < 16) width *= 2;
        launch(scores_from_parts_kernel, dim3((unsigned)((rows * width + 255) / 256)), dim3(256), 0, st,
               (const double *)parts, nparts, width, rows, scores_out);
    }
}

}  // namespace fvar
