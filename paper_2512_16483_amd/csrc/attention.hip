// Attention of the rows that pass through the block over the whole multi-scale KV cache
// (every cached scale is <= the current one, so all L rows are visible to every query).
//
// bf16 kernel, flash style, written for 64-wide wavefronts and 32x32x16 MFMA:
//   * the score tile is computed TRANSPOSED, S^T = K Q^T (keys are the MFMA rows, queries the
//     columns).  In the 32x32 accumulator layout a lane then owns one query column, so the
//     running max / sum of the online softmax are lane-local scalars (one exchange with lane^32
//     per tile), the rescale of the output accumulator is a per-lane multiply, and the
//     probabilities are already laid out as the B operand of the second product
//     O^T = V^T P^T -- no trip through LDS for P.
//   * K and V tiles travel global -> LDS directly (global_load_lds_dwordx4, no staging registers,
//     no LDS store instructions), both row-major with XOR-swizzled 16-byte chunks; the swizzle is
//     applied on the global side (which chunk a lane fetches), since the DMA writes LDS in lane
//     order.  K rows feed the A operand of S^T with one ds_read_b128.  The A operand of the second
//     product needs V transposed (8 consecutive keys of one head-dim column per lane): it is read
//     with the transposing LDS load (ds_read_b64_tr_b16), which hands a lane 4 elements of one
//     column out of the 16 row chunks its 16-lane group points at -- V is never transposed in
//     memory.  The rows each lane points at follow the order in which the accumulator layout
//     hands out the keys of P.
//   * LDS is double buffered: the DMA of the next tile runs under the MFMAs of the current one,
//     one barrier per tile.
//
// fp32 kernel: see there.
#include <type_traits>

#include "common.h"

namespace fvar {

constexpr int BT = 64;                       // keys per tile

typedef short shortx4_t __attribute__((ext_vector_type(4)));
typedef short shortx8_t __attribute__((ext_vector_type(8)));

// 16 bytes per lane global -> LDS; the wavefront fills 1 KiB starting at `lds_addr` in lane order.
// M0 carries the LDS base and is rewritten before every use; no other instruction of these
// kernels reads it.  The loads are counted by hand (s_waitcnt vmcnt) because the compiler does
// not see them.
__device__ __forceinline__ void attn_dma_b128(const void *base, uint32_t byte_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}

// Chunk swizzles (XOR on the 16-byte chunk index of a row).
//   K rows are read 16 rows at a time at one logical chunk (ds_read_b128): with 256-byte rows
//   (head_dim 128) all rows start at the same bank, so the 16 rows must land in 16 different
//   chunks; with 128-byte rows two neighbouring rows already differ by half the banks.
//   V rows are read by the transposing load 4 consecutive rows x 64 contiguous bytes at a time
//   (per 32 lanes): the 4 rows must land in different 64-byte quarters of the 256-byte bank span.
template <int DH> __device__ __forceinline__ int k_swz(int row)
{
    return DH == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int DH> __device__ __forceinline__ int v_swz(int row)
{
    return DH == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2);
}

// KG = 2: two groups of four wavefronts work on the same queries, each with half of the workgroup's key tiles and
// double buffers of its own, and meet in LDS at the end.
template <int DH, int NQ, int KG>
__global__ __launch_bounds__(256 * KG, 2) void attn_bf16_kernel(const uint16_t *__restrict__ q,
                                                        const uint16_t *__restrict__ Kc,
                                                        const uint16_t *__restrict__ Vc, int n, int L,
                                                        int cap, int H, float c_log2,
                                                        uint16_t *__restrict__ o, int nsplit,
                                                        int tiles_per_split,
                                                        float *__restrict__ part_o,
                                                        float *__restrict__ part_ml, int nqb,
                                                        int full_units, int tail_split)
{
    constexpr int KS = DH / 16;              // k16 steps of the QK product
    constexpr int DB = DH / 32;              // 32-row blocks of O^T
    constexpr int KCH = DH / 8;              // 16 B chunks per K / V row
    constexpr int RPD = 64 / KCH;            // tile rows filled by one DMA instruction (1 KiB)
    constexpr int NDMA = BT / RPD / 4;       // DMA instructions per wavefront per tile and tensor
    constexpr int KTILE = BT * DH, STAGE = 2 * KTILE;

    extern __shared__ uint4 lds_raw[];
    uint16_t *lds = reinterpret_cast<uint16_t *>(lds_raw);   // [stage][K tile | V tile]
    uint32_t lds_base = (uint32_t)(uintptr_t)lds_raw;

    const int tid = threadIdx.x, lane = tid & 63;
    const int all_wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KG > 1 ? all_wave >> 2 : 0, wave = KG > 1 ? all_wave & 3 : all_wave;    // group, wavefront in it
    if (KG > 1) { lds += kg * 2 * STAGE; lds_base += kg * 4 * STAGE; }
    const int rl = lane & 31, g = lane >> 5;
    // Work decomposition.  A unit is one (query block, head, sample) triple, numbered with the
    // query block fastest.  Two ways of dividing the key axis between workgroups exist:
    //  * nsplit > 1 (problems with too few units to fill the chip): every unit is divided into
    //    nsplit key ranges, workgroup id = (sample * nsplit + range) * H * nqb + head * nqb + block;
    //  * tail_split > 1 (many units, but the last round of workgroups would leave most of the chip
    //    idle): the first full_units units run whole, each later unit is divided into tail_split
    //    ranges.
    // A workgroup with a partial key range [tile0, tile1) leaves an unnormalised partial result
    // (O, running max, running sum) for a merge kernel.
    // Workgroups are handed to the 8 XCDs in turn (id % 8), each with an L2 of its own, so ids
    // are first renumbered to give every XCD one contiguous run of the numbering above: the query
    // blocks of a head, which stream the same keys and values, then share one L2 instead of
    // fetching them from memory once per XCD.  Whole units and the divided last round are
    // renumbered separately, so the last round is still made of the short pieces on every XCD.
    int unit = blockIdx.x, split = 0, ranges = 1;
    size_t prow_base = 0;                                    // partial row of query 0 of this unit
    int prow_stride = 0;
    if (nsplit > 1) {
        unit = xcd_contiguous(unit, (int)gridDim.x);
        const int per = H * nqb, zz = unit / per;
        split = zz % nsplit;
        ranges = nsplit;
        unit = (zz / nsplit) * per + unit % per;
    } else if (unit < full_units) {
        unit = xcd_contiguous(unit, full_units);
    } else {
        const int t = xcd_contiguous(unit - full_units, (int)gridDim.x - full_units);
        unit = full_units + t / tail_split;
        split = t % tail_split;
        ranges = tail_split;
    }
    const int qb = unit % nqb, h = (unit / nqb) % H, b = unit / (nqb * H);
    if (nsplit > 1) {
        prow_base = (size_t)(b * nsplit + split) * n * H + h;
        prow_stride = H;
    } else if (ranges > 1) {
        prow_base = (size_t)((unit - full_units) * tail_split + split) * (128 * NQ) -
                    (size_t)qb * (128 * NQ);
        prow_stride = 1;
    }
    const int q0 = qb * (128 * NQ) + wave * (32 * NQ);
    const bool wave_active = __builtin_amdgcn_readfirstlane(q0 < n ? 1 : 0) != 0;
    const size_t rowpitch = (size_t)H * DH;
    const uint16_t *Kb = Kc + ((size_t)b * cap * H + h) * DH;
    const uint16_t *Vb = Vc + ((size_t)b * cap * H + h) * DH;

    // ---- Q fragments (B operand: lane = query column, 8 consecutive head-dim values)
    bf16x8_t qf[NQ][KS];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        const int row = min(q0 + j * 32 + rl, n - 1);
        const uint16_t *src = q + ((size_t)b * n + row) * rowpitch + (size_t)h * DH + 8 * g;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            qf[j][s] = *reinterpret_cast<const bf16x8_t *>(src + 16 * s);
    }

    // ---- DMA assignment: wavefront w owns the 1 KiB row groups w, w+4, ... of each tile; lane l
    // fills physical chunk l % KCH of tile row RPD*group + l / KCH, i.e. it fetches the logical
    // chunk that the swizzle maps there.  Byte offsets from the tile's first row; a tile that
    // reaches past row L-1 recomputes them with the row clamped.
    int d_row[NDMA];
    uint32_t k_off[NDMA], v_off[NDMA];
#pragma unroll
    for (int i = 0; i < NDMA; ++i) {
        d_row[i] = (wave + 4 * i) * RPD + lane / KCH;
        const int pc = lane % KCH;
        k_off[i] = (uint32_t)(((size_t)d_row[i] * rowpitch + ((pc ^ k_swz<DH>(d_row[i])) << 3)) * 2);
        v_off[i] = (uint32_t)(((size_t)d_row[i] * rowpitch + ((pc ^ v_swz<DH>(d_row[i])) << 3)) * 2);
    }
    auto issue_tile = [&](int t0, int stage) {
        const uint32_t sk = lds_base + stage * (STAGE * 2) + wave * 1024, sv = sk + KTILE * 2;
        if (t0 + BT <= L) {                                  // uniform
            const uint16_t *kt = Kb + (size_t)t0 * rowpitch, *vtile = Vb + (size_t)t0 * rowpitch;
#pragma unroll
            for (int i = 0; i < NDMA; ++i) attn_dma_b128(kt, k_off[i], sk + i * 4096);
#pragma unroll
            for (int i = 0; i < NDMA; ++i) attn_dma_b128(vtile, v_off[i], sv + i * 4096);
            return;
        }
#pragma unroll
        for (int i = 0; i < NDMA; ++i) {
            const int t = min(t0 + d_row[i], L - 1), pc = lane % KCH;
            attn_dma_b128(Kb, (uint32_t)(((size_t)t * rowpitch + ((pc ^ k_swz<DH>(d_row[i])) << 3)) * 2),
                          sk + i * 4096);
        }
#pragma unroll
        for (int i = 0; i < NDMA; ++i) {
            const int t = min(t0 + d_row[i], L - 1), pc = lane % KCH;
            attn_dma_b128(Vb, (uint32_t)(((size_t)t * rowpitch + ((pc ^ v_swz<DH>(d_row[i])) << 3)) * 2),
                          sv + i * 4096);
        }
    };

    // ---- transposing V read: lane l = 16*G + 4*j + a points at key row 4*(G/2) + j (+ 16u + 8h) and
    // the 4 head-dim values 16*(G%2) + 4*a (+ 32*db); it receives, for the output row
    // 16*(G%2) + (l%16) of block db, the keys 4*(G/2) + 0..3 (+ 16u + 8h): the k-slots 4h..4h+3 of
    // half G/2, in the order the P fragments hold them
    const int tG = lane >> 4, tj = (lane >> 2) & 3, ta = lane & 3;
    const int v_row = 4 * (tG >> 1) + tj;                    // key row inside a 16-key step (h = 0)
    const int v_swq = v_swz<DH>(v_row) >> 2;                 // depends on the lane only (rows +8, +16 keep it)
    const int v_lane = v_row * DH + ((2 * (tG & 1) + (ta >> 1)) << 3) + (ta & 1) * 4;   // elements

    floatx16_t oacc[DB][NQ];
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int j = 0; j < NQ; ++j) oacc[i][j] = floatx16_t{0};
    float m_run[NQ], l_run[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) { m_run[j] = -INFINITY; l_run[j] = 0.f; }

    const int ntiles_all = (L + BT - 1) / BT;
    int tile0 = ranges > 1 ? split * tiles_per_split : 0;
    const int tile1 = ranges > 1 ? min(ntiles_all, tile0 + tiles_per_split) : ntiles_all;
    int nloc = tile1 - tile0;                                // tiles of this group
    const int trips = KG > 1 ? (nloc + 1) / 2 : nloc;
    if (KG > 1) {
        // the second group, which has the cache's ragged tail, takes the odd tile: it comes in the last trip
        const int first = nloc - trips;
        if (kg == 0) nloc = first;
        else { tile0 += first; nloc = trips; }
    }
    if (KG == 1 || nloc > 0) issue_tile(tile0 * BT, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // the Q fragments are consumed here once so that the compiler's own wait for their loads
    // sits in front of the loop instead of inside it (where it would also wait for the prefetch)
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[j][s]));
    __syncthreads();

    // one key tile (`it` counts from this workgroup's first tile); MASKED is set only for the
    // last tile, whose ragged tail must not contribute
    auto tile = [&](int lt, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        const int it = tile0 + lt;
        const uint16_t *ks = lds + (lt & 1) * STAGE;
        const uint16_t *vt = ks + KTILE;
        // next tile into the other stage: every wavefront finished reading it before the barrier
        // that ended the previous iteration
        if (lt + 1 < nloc) issue_tile((it + 1) * BT, (lt + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);

        // a wavefront whose queries all lie past the end only helps with the staging
        if (wave_active && (KG == 1 || lt < nloc)) {
        // ---- S^T = K Q^T : [64 keys] x [32*NQ queries]
        floatx16_t sacc[2][NQ];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int j = 0; j < NQ; ++j) sacc[tb][j] = floatx16_t{0};
        // operand fragments are fetched one step ahead of the MFMAs that use them
        auto load_k = [&](int s, bf16x8_t *dst) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                const int r = tb * 32 + rl;
                dst[tb] = *reinterpret_cast<const bf16x8_t *>(
                    ks + r * DH + (((2 * s + g) ^ k_swz<DH>(r)) << 3));
            }
        };
        auto load_v = [&](int u, bf16x8_t *dst) {
            typedef __attribute__((address_space(3))) shortx4_t lds_shortx4_t;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint16_t *vsrc = vt + v_lane + 16 * u * DH + ((db ^ v_swq) << 5);
                const shortx4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t *)vsrc);
                const shortx4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t *)(vsrc + 8 * DH));
                dst[db] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        bf16x8_t kf[2][2];
        load_k(0, kf[0]);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s + 1 < KS) load_k(s + 1, kf[(s + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int j = 0; j < NQ; ++j)
                    sacc[tb][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s & 1][tb], qf[j][s],
                                                                          sacc[tb][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the first V fragments travel under the softmax
        bf16x8_t vf[2][DB];
        load_v(0, vf[0]);
        __builtin_amdgcn_sched_barrier(0);
        // ---- mask the ragged tail of the cache
        if (MASKED) {
            const int t0 = it * BT;
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int t = t0 + tb * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
                    if (t >= L) {
#pragma unroll
                        for (int j = 0; j < NQ; ++j) sacc[tb][j][i] = -INFINITY;
                    }
                }
        }
        // ---- online softmax, one query column per lane
        bf16x8_t pf[4][NQ];
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            float mx = sacc[0][j][0];
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[tb][j][i]);
            // the other 32 lanes hold the other half of the keys: exchanged in registers (a shuffle
            // is an LDS round trip in the serial part of the tile; without it 1294 -> 1266 us at
            // 1600 rows x 12121 keys x 32 heads of 128, batch 4, 28.5 -> 27.0 us at head_dim 64)
            const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
            const float m_new = fmaxf(m_run[j], mx), m_fin = fmaxf(m_new, -1e30f);   // nothing finite yet: weights of 0
            const float alpha = __builtin_amdgcn_exp2f((m_run[j] - m_fin) * c_log2);
            const float mc = m_fin * c_log2;
            m_run[j] = m_new;
            float psum = 0.f;
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                float p[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    p[i] = __builtin_amdgcn_exp2f(fmaf(sacc[tb][j][i], c_log2, -mc));
                    psum += p[i];
                }
#pragma unroll
                for (int uu = 0; uu < 2; ++uu) {
                    uint4 pk;
                    pk.x = pack_bf16x2(p[8 * uu + 0], p[8 * uu + 1]);
                    pk.y = pack_bf16x2(p[8 * uu + 2], p[8 * uu + 3]);
                    pk.z = pack_bf16x2(p[8 * uu + 4], p[8 * uu + 5]);
                    pk.w = pack_bf16x2(p[8 * uu + 6], p[8 * uu + 7]);
                    pf[2 * tb + uu][j] = __builtin_bit_cast(bf16x8_t, pk);
                }
            }
            l_run[j] = l_run[j] * alpha + psum;
            if (__any(alpha != 1.0f)) {                       // wave-uniform: the max rarely moves
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[db][j][i] *= alpha;
            }
        }
        // ---- O^T += V^T P^T
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u + 1 < 4) load_v(u + 1, vf[(u + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int j = 0; j < NQ; ++j)
                    oacc[db][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u & 1][db], pf[u][j],
                                                                          oacc[db][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    for (int lt = 0; lt + 1 < trips; ++lt) tile(lt, std::false_type{});
    tile(trips - 1, std::true_type{});

    if constexpr (KG > 1) {
        // Each group takes half of the head-dim blocks to the end: it parks the other half, its running max and sum
        // where the other group finds them (the stages are free: the last tile ended with a barrier).
        constexpr int HB = DB / 2;
        float4 *xo = reinterpret_cast<float4 *>(lds_raw);                        // [group][wave][j][block, quad][lane]
        float2 *xm = reinterpret_cast<float2 *>(xo + 8 * NQ * HB * 4 * 64);      // [group][wave][j][lane]
        float m_own[NQ], l_own[NQ];
        auto slot = [&](int grp, int j, int q) { return (((grp * 4 + wave) * NQ + j) * (HB * 4) + q) * 64 + lane; };
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            m_own[j] = m_run[j];
            l_own[j] = l_run[j] + __shfl_xor(l_run[j], 32);
            xm[((kg * 4 + wave) * NQ + j) * 64 + lane] = make_float2(m_own[j], l_own[j]);
#pragma unroll
            for (int hb = 0; hb < HB; ++hb)
#pragma unroll
                for (int e = 0; e < 16; e += 4) {
                    const floatx16_t &v = kg ? oacc[hb][j] : oacc[HB + hb][j];
                    xo[slot(kg, j, hb * 4 + e / 4)] = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
                }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const float2 other = xm[(((1 - kg) * 4 + wave) * NQ + j) * 64 + lane];
            const float m = fmaxf(m_own[j], other.x), m_fin = fmaxf(m, -1e30f);   // as in the loop: no finite score, no weight
            const float wo = __builtin_amdgcn_exp2f((m_own[j] - m_fin) * c_log2);
            const float wx = __builtin_amdgcn_exp2f((other.x - m_fin) * c_log2);
            const float l = l_own[j] * wo + other.y * wx;
            const int row = q0 + j * 32 + rl;
            if (row >= n) continue;
            const float inv = 1.0f / l;
            const size_t prow = prow_base + (size_t)row * prow_stride;
#pragma unroll
            for (int hb = 0; hb < HB; ++hb)
#pragma unroll
                for (int e = 0; e < 16; e += 4) {
                    const floatx16_t &v = kg ? oacc[HB + hb][j] : oacc[hb][j];
                    const float4 x = xo[slot(1 - kg, j, hb * 4 + e / 4)];
                    const float4 r = make_float4(fmaf(x.x, wx, v[e] * wo), fmaf(x.y, wx, v[e + 1] * wo),
                                                 fmaf(x.z, wx, v[e + 2] * wo), fmaf(x.w, wx, v[e + 3] * wo));
                    const int dh = (kg * HB + hb) * 32 + 8 * (e >> 2) + 4 * g;
                    if (ranges > 1)
                        *reinterpret_cast<float4 *>(part_o + prow * DH + dh) = r;
                    else
                        *reinterpret_cast<uint2 *>(o + ((size_t)b * n + row) * rowpitch + (size_t)h * DH + dh) =
                            make_uint2(pack_bf16x2(r.x * inv, r.y * inv), pack_bf16x2(r.z * inv, r.w * inv));
                }
            if (ranges > 1 && kg == 0 && g == 0) *reinterpret_cast<float2 *>(part_ml + prow * 2) = make_float2(m, l);
        }
        return;
    }
    if (ranges > 1) {
        // partial result of this key range: unnormalised O (fp32), running max and sum
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const int row = q0 + j * 32 + rl;
            const float l = l_run[j] + __shfl_xor(l_run[j], 32);
            if (row >= n) continue;
            const size_t prow = prow_base + (size_t)row * prow_stride;
            float *dst = part_o + prow * DH;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int e = 0; e < 16; e += 4) {
                    const int dh = db * 32 + 8 * (e >> 2) + 4 * g;
                    *reinterpret_cast<float4 *>(dst + dh) = make_float4(
                        oacc[db][j][e], oacc[db][j][e + 1], oacc[db][j][e + 2], oacc[db][j][e + 3]);
                }
            if (g == 0) *reinterpret_cast<float2 *>(part_ml + prow * 2) = make_float2(m_run[j], l);
        }
        return;
    }

    // ---- normalise and store: lane = query, 4 consecutive head-dim values per accumulator group
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        const int row = q0 + j * 32 + rl;
        const float l = l_run[j] + __shfl_xor(l_run[j], 32);
        const float inv = 1.0f / l;
        if (row >= n) continue;
        uint16_t *dst = o + ((size_t)b * n + row) * rowpitch + (size_t)h * DH;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e = 0; e < 16; e += 4) {
                const int dh = db * 32 + 8 * (e >> 2) + 4 * g;
                uint2 pk;
                pk.x = pack_bf16x2(oacc[db][j][e] * inv, oacc[db][j][e + 1] * inv);
                pk.y = pack_bf16x2(oacc[db][j][e + 2] * inv, oacc[db][j][e + 3] * inv);
                *reinterpret_cast<uint2 *>(dst + dh) = pk;
            }
    }
}

// Merge of the key-range partials: o = sum_s O_s w_s / sum_s l_s w_s with w_s = 2^((m_s - max m) c).
// One thread per 4 consecutive head-dim values of one (sample, query row, head).
__global__ __launch_bounds__(256) void attn_merge_kernel(const float *__restrict__ part_o,
                                                         const float *__restrict__ part_ml, int n,
                                                         int H, int DH, int nsplit, float c_log2,
                                                         long total, uint16_t *__restrict__ o)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;       // over B * n * H * DH/4
    if (idx >= total) return;
    const int per_row = H * (DH / 4);
    const long brow = idx / per_row;                             // b * n + row
    const int rem = (int)(idx % per_row), h = rem / (DH / 4), c4 = rem % (DH / 4);
    const long b = brow / n, row = brow % n;
    float m = -INFINITY;
    for (int s = 0; s < nsplit; ++s)
        m = fmaxf(m, part_ml[((((size_t)b * nsplit + s) * n + row) * H + h) * 2]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f;
    for (int s = 0; s < nsplit; ++s) {
        const size_t prow = (((size_t)b * nsplit + s) * n + row) * H + h;
        const float2 ml = *reinterpret_cast<const float2 *>(part_ml + prow * 2);
        const float w = __builtin_amdgcn_exp2f((ml.x - m) * c_log2);
        const float4 v = *reinterpret_cast<const float4 *>(part_o + prow * DH + c4 * 4);
        acc.x = fmaf(v.x, w, acc.x); acc.y = fmaf(v.y, w, acc.y);
        acc.z = fmaf(v.z, w, acc.z); acc.w = fmaf(v.w, w, acc.w);
        den = fmaf(ml.y, w, den);
    }
    const float inv = 1.0f / den;
    uint2 pk;
    pk.x = pack_bf16x2(acc.x * inv, acc.y * inv);
    pk.y = pack_bf16x2(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2 *>(o + ((size_t)brow * H + h) * DH + c4 * 4) = pk;
}

// Merge for the units whose key axis was divided only in the last round of workgroups: partials
// are stored per (tail unit, range) as [BQ queries][DH] (+ [BQ][2] running max / sum).
// One thread per 4 consecutive head-dim values of one (tail unit, query).
__global__ __launch_bounds__(256) void attn_tail_merge_kernel(const float *__restrict__ part_o,
                                                              const float *__restrict__ part_ml, int n,
                                                              int H, int DH, int BQ, int nqb,
                                                              int full_units, int ranges, float c_log2,
                                                              long total, uint16_t *__restrict__ o)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;       // over tail units * BQ * DH/4
    if (idx >= total) return;
    const int c4 = (int)(idx % (DH / 4));
    const long uq = idx / (DH / 4);
    const int ql = (int)(uq % BQ), tu = (int)(uq / BQ), unit = full_units + tu;
    const int qb = unit % nqb, h = (unit / nqb) % H, b = unit / (nqb * H);
    const int row = qb * BQ + ql;
    if (row >= n) return;
    float m = -INFINITY;
    for (int s = 0; s < ranges; ++s) m = fmaxf(m, part_ml[((size_t)(tu * ranges + s) * BQ + ql) * 2]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f;
    for (int s = 0; s < ranges; ++s) {
        const size_t prow = (size_t)(tu * ranges + s) * BQ + ql;
        const float2 ml = *reinterpret_cast<const float2 *>(part_ml + prow * 2);
        const float w = __builtin_amdgcn_exp2f((ml.x - m) * c_log2);
        const float4 v = *reinterpret_cast<const float4 *>(part_o + prow * DH + c4 * 4);
        acc.x = fmaf(v.x, w, acc.x); acc.y = fmaf(v.y, w, acc.y);
        acc.z = fmaf(v.z, w, acc.z); acc.w = fmaf(v.w, w, acc.w);
        den = fmaf(ml.y, w, den);
    }
    const float inv = 1.0f / den;
    uint2 pk;
    pk.x = pack_bf16x2(acc.x * inv, acc.y * inv);
    pk.y = pack_bf16x2(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2 *>(o + (((size_t)b * n + row) * H + h) * DH + c4 * 4) = pk;
}

// Query rows per workgroup and workgroups that a CU holds at once for a problem (the variant the
// launcher picks), and the plan for the last round of workgroups: with `units` workgroups on
// `slots` places, the units beyond the last full round are divided into `ranges` key ranges each
// when that round would leave more than a quarter of the places empty.
struct AttnPlan { int bq, slots, nqb, units, full_units, tail_ranges; };
static AttnPlan attention_plan(int B, int n, int H, int Dh)
{
    AttnPlan p;
    const bool wide = Dh == 64 && ((n % 256 == 0) || (n % 256 > 128));
    p.bq = wide ? 256 : 128;
    p.slots = 256 * ((Dh == 64 && !wide) ? 4 : 2);
    p.nqb = (n + p.bq - 1) / p.bq;
    p.units = p.nqb * H * B;
    p.full_units = p.units / p.slots * p.slots;
    const int rem = p.units - p.full_units;
    p.tail_ranges = 1;
    if (p.full_units > 0 && rem > 0 && rem * 4 <= p.slots * 3) {
        int r = p.slots / rem;
        p.tail_ranges = r > 8 ? 8 : r;
    }
    if (p.tail_ranges < 2) { p.tail_ranges = 1; p.full_units = p.units; }
    return p;
}

// Number of key ranges for a problem, from the launch geometry alone (not the cache length, so
// that the workspace can be sized from it; the launcher lowers it when the cache is short).
// The kernel is throughput-bound per CU, so what counts is rounds of workgroups over the 256 CUs:
// s ranges cost ceil(wgs*s/256)/s rounds of full-length work, plus about 8 % per extra range for
// the partial results and their merge (12 % when the problem already fills the chip once: its
// partials are larger); fitted to sweeps of the head_dim-128 shapes with 64..640 workgroups.
int attention_max_splits(DType dt, int B, int n, int H, int Dh)
{
    if (dt != DType::BF16) return 1;
    const bool wide = Dh == 64 && ((n % 256 == 0) || (n % 256 > 128));
    const long wgs = (long)((n + (wide ? 255 : 127)) / (wide ? 256 : 128)) * H * B;
    int best = 1;
    double best_cost = 1e300;
    const double per_split = wgs >= 256 ? 0.12 : 0.08;
    for (int s = 1; s <= 8; ++s) {
        const double rounds = (double)((wgs * s + 255) / 256);
        const double cost = rounds / s * (1.0 + per_split * (s - 1));
        if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
    }
    return best;
}

// Floats of scratch the bf16 attention of a problem may need for partial results (either way of
// dividing the key axis); 0 when every workgroup sees the whole cache.
size_t attention_scratch_floats(DType dt, int B, int n, int H, int Dh)
{
    if (dt != DType::BF16) return 0;
    const int ns = attention_max_splits(dt, B, n, H, Dh);
    if (ns > 1) return (size_t)ns * B * n * H * (Dh + 2);
    const AttnPlan p = attention_plan(B, n, H, Dh);
    if (p.tail_ranges > 1) return (size_t)(p.units - p.full_units) * p.tail_ranges * p.bq * (Dh + 2);
    return 0;
}

// How an attention is run: wavefront groups per workgroup, key ranges of every unit, key ranges of the units beyond
// the last whole round.
struct AttnRun { int kg, nsplit, tail; };

// Predicted time: rounds of workgroups over the places that a CU has for them, each with a fixed part and a pace per
// key tile that depends on how many share the CU and, up to one per CU, on how many CUs are at work; once a part that
// grows with the wavefronts of a workgroup that have queries (they load, merge and store); the partial results and
// their merge.  One row per variant (head_dim 128, 64 with 256 and with 128 queries), fitted to 3000 timings of 570
// problems (1 to 20 samples, 2 to 2500 queries, 70 to 11000 keys): 5 to 7 % rms.
struct AttnTimes { double once, active, groups, round, merge, merge_mb, pace[2][4], crowd[2]; };
constexpr AttnTimes kAttnTimes[3] = {
    {3.93, 1.64, 0.75, 1.90, 3.91, 0.14, {{1.06, 2.12, 0, 0}, {1.78, 0, 0, 0}}, {0.33, 0.68}},
    {2.89, 3.63, 0.88, 1.26, 3.62, 0.16, {{1.20, 2.16, 0, 0}, {1.90, 0, 0, 0}}, {0.22, 0.58}},
    {3.04, 1.37, 0.77, 0.52, 3.80, 0.15, {{0.72, 1.18, 1.80, 2.22}, {1.10, 2.24, 0, 0}}, {0.17, 0.32}}};
static double attention_us(int B, int n, int L, int H, int Dh, const AttnPlan &p, const AttnRun &run)
{
    const AttnTimes &c = kAttnTimes[Dh == 128 ? 0 : p.bq == 256 ? 1 : 2];
    const int ntiles = (L + BT - 1) / BT, tps = (ntiles + run.nsplit - 1) / run.nsplit, ns = (ntiles + tps - 1) / tps;
    const int trips = (tps + run.kg - 1) / run.kg, per = p.slots / 256 / run.kg;
    const int waves = n >= p.bq ? 4 : (4 * n + p.bq - 1) / p.bq;         // that have queries
    const long wgs = (long)p.units * ns, full = wgs / (256 * per), rem = wgs % (256 * per);
    const double *pace = c.pace[run.kg - 1];
    const auto tile_us = [&](int k, double busy) { return k == 1 ? pace[0] + c.crowd[run.kg - 1] * busy : pace[k - 1]; };
    double us = c.once + c.active * (waves - 1) / 3.0 + (run.kg > 1 ? c.groups : 0.0);
    us += full * (c.round + trips * tile_us(per, 1.0)) - (full && !rem ? c.round : 0.0);     // between rounds only
    if (rem && run.tail > 1) {
        us += c.round + (double)((trips + run.tail - 1) / run.tail) * tile_us(per, 1.0) + c.merge;
    } else if (rem) {
        const int k = (int)((rem + 255) / 256);
        us += (full ? c.round : 0.0) + trips * tile_us(k, rem / 256.0);
    }
    return ns > 1 ? us + c.merge + c.merge_mb * (2.0e-6 * ns * B * n * H * (Dh + 2) * sizeof(float)) : us;
}

// The division by key ranges that the workspace is sized for, unless fewer ranges, or two wavefront groups per
// workgroup with at most as many, promise 3 % and 0.9 us less: two groups fill a CU as two workgroups do, without
// partial results in memory.  us, one group and the ranges above -> here: 2 x 1024 queries, 2521 keys, 16 heads of 128
// 65.4 -> 50.6, 2000 x 6000 122.8 -> 105.8, 3 x 400 x 1500 42.8 -> 29.7, 2 x 576 x 1216, 30 heads of 64 33.5 -> 26.0;
// over the 570 problems 6 % on average, at worst 2 % more.  (With 3 % alone, and fixed parts that do not know how many
// wavefronts have queries, 24 of them were 3 to 18 % slower, all with few queries and a short cache: 2 x 2 queries,
// 635 keys, 32 heads of 128 12.7 us in two ranges, 15.0 by two groups.)
static AttnRun attention_run(int B, int n, int L, int H, int Dh, bool scratch)
{
    const AttnPlan p = attention_plan(B, n, H, Dh);
    const int ntiles = (L + BT - 1) / BT, longest = ntiles / 4 > 0 ? ntiles / 4 : 1;   // ranges of at least 4 tiles
    AttnRun run{1, scratch ? attention_max_splits(DType::BF16, B, n, H, Dh) : 1, 1};
    if (run.nsplit > longest) run.nsplit = longest;
    if (scratch && run.nsplit == 1) run.tail = p.tail_ranges;
    if (run.tail > longest) run.tail = longest;
    const int most = run.nsplit;
    const double sized = attention_us(B, n, L, H, Dh, p, run);
    double best = fmin(0.97 * sized, sized - 0.9);
    for (int kg = 1; kg <= 2; ++kg)
        for (int ns = 1; ns <= most; ++ns) {
            if (kg == 1 ? ns == most : ntiles < 6 * ns) continue;
            const AttnRun other{kg, ns, 1};
            const double us = attention_us(B, n, L, H, Dh, p, other);
            if (us < best) { best = us; run = other; }
        }
    return run;
}

int attention_ways(int B, int n, int L, int H, int Dh)
{
    const AttnRun run = attention_run(B, n, L, H, Dh, true);
    return 100 * run.kg + run.nsplit;
}

template <int DH, int NQ, int KG>
static void launch_attn_bf16(const void *q, const void *K, const void *V, int B, int n, int L,
                             int cap, int H, float scale, void *o, float *part, const AttnRun &run, hipStream_t st)
{
    constexpr int BQ = 128 * NQ;
    constexpr size_t stages = (size_t)KG * 2 * 2 * BT * DH * sizeof(uint16_t);
    constexpr size_t meet = KG > 1 ? (size_t)8 * NQ * 64 * (DH / 64 * 4 * sizeof(float4) + sizeof(float2)) : 0;
    constexpr size_t lds = stages > meet ? stages : meet;
    auto kern = attn_bf16_kernel<DH, NQ, KG>;
    if (lds > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    // no range is empty
    const int ntiles = (L + BT - 1) / BT;
    int nsplit = run.nsplit, tps = (ntiles + nsplit - 1) / nsplit;
    nsplit = (ntiles + tps - 1) / tps;
    const float c_log2 = scale * 1.4426950408889634f;
    AttnPlan plan = attention_plan(B, n, H, DH);
    int tail = nsplit == 1 ? run.tail : 1;
    if (tail > 1) {
        tps = (ntiles + tail - 1) / tail;
        tail = (ntiles + tps - 1) / tps;
    }
    if (tail < 2) { tail = 1; plan.full_units = plan.units; }
    const int tail_units = plan.units - plan.full_units;
    float *part_o = part, *part_ml = nullptr;
    if (nsplit > 1) part_ml = part + (size_t)nsplit * B * n * H * DH;
    else if (tail > 1) part_ml = part + (size_t)tail_units * tail * BQ * DH;
    const unsigned nwg = nsplit > 1 ? (unsigned)plan.units * nsplit
                                    : (unsigned)(plan.full_units + tail_units * tail);
    launch(kern, dim3(nwg), dim3(256 * KG), lds, st, (const uint16_t *)q, (const uint16_t *)K,
           (const uint16_t *)V, n, L, cap, H, c_log2, (uint16_t *)o, nsplit, tps, part_o, part_ml,
           plan.nqb, plan.full_units, tail);
    if (nsplit > 1) {
        const long total = (long)B * n * H * (DH / 4);
        launch(attn_merge_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
               (const float *)part_o, (const float *)part_ml, n, H, DH, nsplit, c_log2, total,
               (uint16_t *)o);
    } else if (tail > 1) {
        const long total = (long)tail_units * BQ * (DH / 4);
        launch(attn_tail_merge_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
               (const float *)part_o, (const float *)part_ml, n, H, DH, BQ, plan.nqb, plan.full_units,
               tail, c_log2, total, (uint16_t *)o);
    }
}

// ------------------------------------------------------------------------------ fp32
// Flash attention on the fp32 MFMA (16x16x4), for 16 queries per workgroup whose NW wavefronts take
// NW contiguous shares of the key tiles and meet in LDS at the end.  The MFMA is no faster than the
// vector units in fp32, but takes one operand register where they take an LDS read per few FMAs.  At the
// sizes of the fp32 configuration the chip is not filled: 128 rows x 16 heads are 128 workgroups of 8
// wavefronts, each with four or five key tiles in sequence (pipes busy 0.09 of the clocks).  Nothing is staged: S^T = K Q^T takes its operands as float4 of
// four consecutive head-dim values (the k-slots of four MFMAs), P stays in the registers S^T left
// it in, and V rows are read as float4 across the head dim, which only permutes the rows of O^T.
// 128 rows x 552 keys x 16 heads of 64: 109 us (one query row per 8 lanes, K / V through LDS) -> 11.9 us.
template <int DH, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(const float *__restrict__ q,
                                                           const float *__restrict__ Kc,
                                                           const float *__restrict__ Vc, int n, int L,
                                                           int cap, int H, float scale, int nqb,
                                                           float *__restrict__ o)
{
    constexpr int KS = DH / 16, VB = DH / 64;                // float4 per key row and lane; 64-wide V blocks
    __shared__ float4 red[NW][VB * 4][64];
    __shared__ float red_ml[NW][2][16];
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q16 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = xcd_contiguous(blockIdx.x, gridDim.x);  // query blocks of a head share an L2
    const int qb = unit % nqb, h = unit / nqb % H, b = unit / (nqb * H);
    const size_t pitch = (size_t)H * DH;
    const float *Kb = Kc + ((size_t)b * cap * H + h) * DH, *Vb = Vc + ((size_t)b * cap * H + h) * DH;
    float4 qf[KS];
    const int row = min(qb * 16 + c16, n - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s)
        qf[s] = *reinterpret_cast<const float4 *>(q + ((size_t)b * n + row) * pitch + (size_t)h * DH + 16 * s + 4 * q16);
    floatx4_t acc[VB * 4];
#pragma unroll
    for (int i = 0; i < VB * 4; ++i) acc[i] = floatx4_t{0};
    float m_run = -INFINITY, l_run = 0.f;
    const int tiles = (L + 15) / 16;
    const int t0 = (int)((long)tiles * wave / NW), t1 = (int)((long)tiles * (wave + 1) / NW);
    float4 kf[KS], vf[VB][4];
    auto load = [&](int t) {
        const float *kr = Kb + (size_t)min(t * 16 + c16, L - 1) * pitch + 4 * q16;
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[s] = *reinterpret_cast<const float4 *>(kr + 16 * s);
    };
    auto load_v = [&](int t) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *vr = Vb + (size_t)min(t * 16 + 4 * q16 + e, L - 1) * pitch + 4 * c16;
#pragma unroll
            for (int v = 0; v < VB; ++v) vf[v][e] = *reinterpret_cast<const float4 *>(vr + 64 * v);
        }
    };
    if (t0 < t1) { load(t0); load_v(t0); }
    for (int t = t0; t < t1; ++t) {
        // S^T: lane (c16, q16) ends up with keys 4 q16 .. +3 of query c16
        floatx4_t s = {0};
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i].x, qf[i].x, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i].y, qf[i].y, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i].z, qf[i].z, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i].w, qf[i].w, s, 0, 0, 0);
        }
        if (t + 1 < t1) load(t + 1);
        float p[4], mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = t * 16 + 4 * q16 + e < L ? s[e] * scale : -INFINITY;
            mx = fmaxf(mx, p[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float base = m_new == -INFINITY ? 0.f : m_new;     // nothing finite yet: weights of 0
        const float alpha = expf(m_run - base);
        m_run = m_new;
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) { p[e] = expf(p[e] - base); sum += p[e]; }
        l_run = l_run * alpha + sum;
        if (__any(alpha != 1.0f)) {
#pragma unroll
            for (int i = 0; i < VB * 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][e] *= alpha;
        }
        // O^T += V^T P^T: MFMA row c16 of block (v, j) is head-dim 64 v + 4 c16 + j
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < VB; ++v) {
                acc[4 * v + 0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][e].x, p[e], acc[4 * v + 0], 0, 0, 0);
                acc[4 * v + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][e].y, p[e], acc[4 * v + 1], 0, 0, 0);
                acc[4 * v + 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][e].z, p[e], acc[4 * v + 2], 0, 0, 0);
                acc[4 * v + 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][e].w, p[e], acc[4 * v + 3], 0, 0, 0);
            }
        if (t + 1 < t1) load_v(t + 1);
    }
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    // entry e of block (v, j): query c16, head-dim 64 v + 4 (4 q16 + e) + j; regrouped so that slot
    // (v, e) holds the four consecutive values j = 0..3
#pragma unroll
    for (int v = 0; v < VB; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            red[wave][4 * v + e][lane] = make_float4(acc[4 * v][e], acc[4 * v + 1][e], acc[4 * v + 2][e], acc[4 * v + 3][e]);
    if (q16 == 0) { red_ml[wave][0][c16] = m_run; red_ml[wave][1][c16] = l_run; }
    __syncthreads();
    if (qb * 16 + c16 >= n) return;
    float m = red_ml[0][0][c16];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, red_ml[w][0][c16]);
    float wgt[NW], den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { wgt[w] = expf(red_ml[w][0][c16] - m); den += red_ml[w][1][c16] * wgt[w]; }
    const float inv = 1.0f / den;
    for (int i = wave; i < VB * 4; i += NW) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 x = red[w][i][lane];
            v.x = fmaf(x.x, wgt[w], v.x); v.y = fmaf(x.y, wgt[w], v.y);
            v.z = fmaf(x.z, wgt[w], v.z); v.w = fmaf(x.w, wgt[w], v.w);
        }
        float *dst = o + ((size_t)b * n + row) * pitch + (size_t)h * DH + 64 * (i / 4) + 4 * (4 * q16 + i % 4);
        *reinterpret_cast<float4 *>(dst) = make_float4(v.x * inv, v.y * inv, v.z * inv, v.w * inv);
    }
}

void launch_attention(DType dt, const void *q, const void *K, const void *V, int B, int n, int L,
                      int cap, int H, int Dh, float scale, void *o, float *part, hipStream_t st)
{
    if (dt == DType::BF16) {
        // two 32-query blocks per wavefront halve the LDS operand traffic per MFMA; use the
        // single-block variant when that would leave most of a 256-query tile empty
        const bool wide = (n % 256 == 0) || (n % 256 > 128);
        const AttnRun run = attention_run(B, n, L, H, Dh, part != nullptr);
#define FVAR_ATTN(DH, NQ)                                                                                        \
    (run.kg == 2 ? launch_attn_bf16<DH, NQ, 2>(q, K, V, B, n, L, cap, H, scale, o, part, run, st)                \
                 : launch_attn_bf16<DH, NQ, 1>(q, K, V, B, n, L, cap, H, scale, o, part, run, st))
        if (Dh == 64) {
            if (wide) FVAR_ATTN(64, 2);
            else FVAR_ATTN(64, 1);
        } else {
            // head_dim 128 with two query blocks per wavefront does not fit the register budget of
            // two wavefronts per SIMD, which is what lets one wavefront's softmax overlap the
            // other's MFMAs
            FVAR_ATTN(128, 1);
        }
#undef FVAR_ATTN
    } else {
        const int nqb = (n + 15) / 16;
        const dim3 grid((unsigned)nqb * H * B), block(512);
        if (Dh == 64)
            launch(attn_f32_kernel<64, 8>, grid, block, 0, st, (const float *)q, (const float *)K,
                   (const float *)V, n, L, cap, H, scale, nqb, (float *)o);
        else
            launch(attn_f32_kernel<128, 8>, grid, block, 0, st, (const float *)q, (const float *)K,
                   (const float *)V, n, L, cap, H, scale, nqb, (float *)o);
    }
}

}  // namespace fvar
