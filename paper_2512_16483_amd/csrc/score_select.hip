// Representative-token scoring and selection (paper, Sec. "Representative Token Restoration").
//
//   score   s_i = fl32(sum_j x_ij^2): one wavefront per token row, 16-byte loads, products and
//           the sum carried in fp64 (exact products; the order of the adds then changes the
//           stored fp32 value only in double-rounding corner cases), butterfly reduction.
//   select  one workgroup per sample: histograms over the order-preserving integer image of the
//           scores yield the k-th largest key T and how many keys equal to T are still needed;
//           then an ordered sweep over the indices with prefix sums writes the kept and the
//           pruned indices, each ascending.  Ties at T go to the lower index.  No atomics touch
//           the outputs, so the result is deterministic.
#include "common.h"

namespace fvar {

template <typename T>
__global__ __launch_bounds__(256) void scores_kernel(const T *__restrict__ x, int rows, int d,
                                                     float *__restrict__ scores)
{
    constexpr int E = Elem<T>::kPerChunk;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const uint4 *src = reinterpret_cast<const uint4 *>(x + (size_t)row * d);
    const int nchunk = d / E;
    double acc0 = 0.0, acc1 = 0.0;
    int c = lane;
    // four chunks in flight per lane
    for (; c + 192 < nchunk; c += 256) {
        uint4 v0 = src[c], v1 = src[c + 64], v2 = src[c + 128], v3 = src[c + 192];
        float f[E];
        Elem<T>::unpack(v0, f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc0 = fma((double)f[e], (double)f[e], acc0);
        Elem<T>::unpack(v1, f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc1 = fma((double)f[e], (double)f[e], acc1);
        Elem<T>::unpack(v2, f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc0 = fma((double)f[e], (double)f[e], acc0);
        Elem<T>::unpack(v3, f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc1 = fma((double)f[e], (double)f[e], acc1);
    }
    for (; c < nchunk; c += 64) {
        uint4 v0 = src[c];
        float f[E];
        Elem<T>::unpack(v0, f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc0 = fma((double)f[e], (double)f[e], acc0);
    }
    double acc = wave_sum(acc0 + acc1);
    if (lane == 0) scores[row] = (float)acc;
}

void launch_scores(DType dt, const void *x, int rows, int d, float *scores, hipStream_t st)
{
    dim3 grid((rows + 3) / 4), block(256);
    if (dt == DType::BF16)
        launch(scores_kernel<uint16_t>, grid, block, 0, st, (const uint16_t *)x, rows, d,
                           scores);
    else
        launch(scores_kernel<float>, grid, block, 0, st, (const float *)x, rows, d,
                           scores);
}

// Order-preserving map float -> uint32 (larger float <=> larger key); -0 and +0 share a key.
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t b = __float_as_uint(s);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelBins = 4096;               // four per thread
constexpr int kSelKeysMax = 12;              // keys per thread that stay in registers

// Up to 12 * 1024 scores per sample: every thread keeps its KPT keys (tokens tid, tid + 1024, ...) in
// registers.  The first histogram spans the sample's own key range, so that neighbouring scores (a few
// binades in all, which one 8-bit digit throws into a handful of bins whose LDS atomics then run one by one)
// spread over its 4096 bins; the bin that holds the k-th largest key is divided in the same way until at most
// 64 keys are left, all of the bin is kept, or its keys are equal.  Those few are ranked by each wavefront for
// itself.  The sweep that follows counts all its pieces at once, for one barrier in all.
// Latency alone counts here: one workgroup per sample, six barriers where four 8-bit digits from LDS and a
// barrier per 1024 tokens of the sweep took 12 and more.  8 x 4096 scores 11.3 -> 6.6 us, 2304 scores 9 -> 5.9,
// 8 x 576 scores 5.0 -> 5.1.
template <int KPT>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const float *__restrict__ scores, int M,
                                                             int k, int32_t *__restrict__ idx_keep,
                                                             int32_t *__restrict__ idx_drop)
{
    __shared__ int hist[kSelBins];
    __shared__ uint32_t wave_min[kSelWaves], wave_max[kSelWaves], few[64];
    __shared__ int wave_sum_[kSelWaves], counts[KPT * kSelWaves];
    __shared__ int sh_bin, sh_remaining, sh_count, sh_few;

    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *s = scores + (size_t)b * M;

    uint32_t key[KPT], lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int i = j * kSelThreads + tid;
        key[j] = score_key(s[min(i, M - 1)]);            // a copy of the last key does not move the range
        lo = min(lo, key[j]);
        hi = max(hi, key[j]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, o));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, o));
    }
    if (lane == 0) { wave_min[wave] = lo; wave_max[wave] = hi; }
    reinterpret_cast<int4 *>(hist)[tid] = make_int4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) { lo = min(lo, wave_min[w]); hi = max(hi, wave_max[w]); }

    // ---- T: the k-th largest key; need_eq: how many keys equal to T are kept (the lowest indices).
    // `base` is the largest key of the range in question, `bins` its bins of 2^shift keys, largest first.
    uint32_t T, base = hi;
    int need_eq, remaining = k;
    uint32_t bins = kSelBins;
    int shift = max(0, 20 - __clz((int)(hi - lo)));      // hi == lo: clz 32
    for (;;) {
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const uint32_t bin = (base - key[j]) >> shift;
            // keys above the range wrap to a large difference, which at shift 0 and a base of few bits is the
            // only thing that tells them apart
            if (j * kSelThreads + tid < M && key[j] <= base && bin < bins) atomicAdd(&hist[bin], 1);
        }
        if (tid == 0) sh_few = 0;
        __syncthreads();
        const int4 c = reinterpret_cast<const int4 *>(hist)[tid];
        const int sum = c.x + c.y + c.z + c.w;
        int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wave_sum_[wave] = incl;
        __syncthreads();
        int run = incl - sum;                            // keys in larger bins
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) run += w < wave ? wave_sum_[w] : 0;
        if (run < remaining && remaining <= run + sum) { // one thread
            int bin = 4 * tid, n = c.x;
            if (remaining > run + n) { run += n; ++bin; n = c.y; }
            if (remaining > run + n) { run += n; ++bin; n = c.z; }
            if (remaining > run + n) { run += n; ++bin; n = c.w; }
            sh_bin = bin; sh_remaining = remaining - run; sh_count = n;
        }
        __syncthreads();
        const uint32_t bin = (uint32_t)sh_bin;
        const int count = sh_count;
        remaining = sh_remaining;
        base -= bin << shift;                            // the bin's largest key
        if (count == remaining || shift == 0) {          // all of it, or equal keys
            const uint32_t width = (1u << shift) - 1u;
            T = width > base ? 0u : base - width;
            need_eq = count == remaining ? M : remaining;
            break;
        }
        if (count <= 64) {
#pragma unroll
            for (int j = 0; j < KPT; ++j)
                if (j * kSelThreads + tid < M && key[j] <= base && (base - key[j]) >> shift == 0)
                    few[atomicAdd(&sh_few, 1)] = key[j];
            __syncthreads();
            const uint32_t mine = few[min(lane, count - 1)];
            const uint32_t one = (uint32_t)__builtin_amdgcn_readfirstlane((int)mine);
            if (__ballot(mine == one) == ~0ull) {        // equal scores: 48 of them ranked one by one take 3 us
                T = one;
                need_eq = remaining;
                break;
            }
            int above = 0, equal = 0;
            for (int i = 0; i < count; ++i) {
                const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
                above += other > mine;
                equal += other == mine;
            }
            // every lane with the wanted key agrees; take the first
            const int src = __ffsll(__ballot(above < remaining && remaining <= above + equal)) - 1;
            T = (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
            need_eq = remaining - __builtin_amdgcn_readlane(above, src);
            break;
        }
        // divide the bin; its counts were read before the last barrier
        const int next = max(0, shift - 12);
        bins = 1u << (shift - next);
        shift = next;
        reinterpret_cast<int4 *>(hist)[tid] = make_int4(0, 0, 0, 0);
        __syncthreads();
    }

    // ---- ordered sweep: stable compaction of kept and pruned indices.  Keys above T and keys equal to T are
    // counted together (low and high half): the kept keys before index i are those above T plus the first
    // need_eq of those equal to it.
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned long long mg[KPT], me[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const bool valid = j * kSelThreads + tid < M;
        mg[j] = __ballot(valid && key[j] > T);
        me[j] = __ballot(valid && key[j] == T);
        if (lane == 0) counts[j * kSelWaves + wave] = __popcll(mg[j]) | __popcll(me[j]) << 16;
    }
    __syncthreads();
    int32_t *keep_out = idx_keep + (size_t)b * k;
    int32_t *drop_out = idx_drop ? idx_drop + (size_t)b * (M - k) : nullptr;
    int carry = 0;
#pragma unroll
    for (int j0 = 0; j0 < KPT; j0 += 4) {                // 64 pieces of 64 tokens at a time
        const int mine = j0 * kSelWaves + lane < KPT * kSelWaves ? counts[j0 * kSelWaves + lane] : 0;
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        const int before = incl - mine + carry;
        carry += __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
        for (int j = j0; j < min(j0 + 4, KPT); ++j) {
            const int i = j * kSelThreads + tid;
            const int piece = __builtin_amdgcn_readlane(before, (j - j0) * kSelWaves + wave);
            const int gt_before = (piece & 0xffff) + __popcll(mg[j] & below);
            const int eq_before = (piece >> 16) + __popcll(me[j] & below);
            const bool keep = (mg[j] >> lane & 1) || ((me[j] >> lane & 1) && eq_before < need_eq);
            const int keep_pos = gt_before + min(eq_before, need_eq);
            if (i < M) {
                if (keep) keep_out[keep_pos] = i;
                else if (drop_out) drop_out[i - keep_pos] = i;
            }
        }
    }
}

// More scores than registers hold: MSB-first radix select in four passes of 8 bits, the keys read from
// memory in each.
__global__ __launch_bounds__(kSelThreads) void select_large_kernel(const float *__restrict__ scores, int M,
                                                                   int k, int32_t *__restrict__ idx_keep,
                                                                   int32_t *__restrict__ idx_drop)
{
    __shared__ int hist[256];
    __shared__ int2 wave_tot[2][kSelWaves];
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_remaining;

    const int b = blockIdx.x;
    const float *s = scores + (size_t)b * M;
    const int tid = threadIdx.x;

    auto key_at = [&](int i) -> uint32_t { return score_key(s[i]); };
    if (tid == 0) { sh_prefix = 0u; sh_remaining = k; }

    // ---- radix select of the k-th largest key
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        const uint32_t prefix = sh_prefix;
        const int remaining = sh_remaining;
        // keys whose already-fixed high bits equal the prefix
        const uint32_t himask = (pass == 0) ? 0u : (0xffffffffu << (shift + 8));
        for (int i = tid; i < M; i += kSelThreads) {
            uint32_t key = key_at(i);
            if ((key & himask) == prefix) atomicAdd(&hist[(key >> shift) & 0xffu], 1);
        }
        __syncthreads();
        if (tid < 64) {
            // lane l owns bins 255-4l .. 252-4l (descending); `above` = keys in higher bins
            int c[4], sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { c[j] = hist[255 - 4 * tid - j]; sum += c[j]; }
            int incl = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                int t = __shfl_up(incl, o);
                if (tid >= o) incl += t;
            }
            int run = incl - sum;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (run < remaining && remaining <= run + c[j]) {
                    sh_prefix = prefix | ((uint32_t)(255 - 4 * tid - j) << shift);
                    sh_remaining = remaining - run;
                }
                run += c[j];
            }
        }
        __syncthreads();
    }
    const uint32_t T = sh_prefix;      // k-th largest key
    const int need_eq = sh_remaining;  // how many keys == T are kept (the lowest indices)

    // ---- ordered sweep: stable compaction of kept and pruned indices.  Keys above T and keys equal to
    // T are counted together: the kept keys before index i are those above T plus the first need_eq of
    // those equal to it.  The wavefronts' counts alternate between two buffers, so a sweep takes one
    // barrier (four with a scan for each flag: 12.1 -> 11.3 us for 8 x 4096 scores, 5.4 -> 5.0 for 8 x 576).
    const int lane = tid & 63, wave = tid >> 6;
    int run_gt = 0, run_eq = 0;
    int32_t *keep_out = idx_keep + (size_t)b * k;
    int32_t *drop_out = idx_drop ? idx_drop + (size_t)b * (M - k) : nullptr;
    for (int base = 0, it = 0; base < M; base += kSelThreads, ++it) {
        const int i = base + tid;
        const bool valid = i < M;
        const uint32_t key = valid ? key_at(i) : 0u;
        const bool eq = valid && key == T, gt = valid && key > T;
        const unsigned long long me = __ballot(eq), mg = __ballot(gt), below = (1ull << lane) - 1ull;
        if (lane == 0) wave_tot[it & 1][wave] = make_int2(__popcll(mg), __popcll(me));
        __syncthreads();
        int gt_before = run_gt + __popcll(mg & below), eq_before = run_eq + __popcll(me & below);
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) {
            const int2 t = wave_tot[it & 1][w];
            if (w < wave) { gt_before += t.x; eq_before += t.y; }
            run_gt += t.x;
            run_eq += t.y;
        }
        const bool keep = gt || (eq && eq_before < need_eq);
        const int keep_pos = gt_before + min(eq_before, need_eq);
        if (valid) {
            if (keep) keep_out[keep_pos] = i;
            else if (drop_out) drop_out[i - keep_pos] = i;
        }
    }
}

void launch_select(const float *scores, int B, int M, int k, int32_t *idx_keep, int32_t *idx_drop,
                   hipStream_t st)
{
    const dim3 grid(B), block(kSelThreads);
    const int kpt = (M + kSelThreads - 1) / kSelThreads;
#define FVAR_SELECT(KPT) launch(select_kernel<KPT>, grid, block, 0, st, scores, M, k, idx_keep, idx_drop)
    if (kpt <= 1) FVAR_SELECT(1);
    else if (kpt <= 2) FVAR_SELECT(2);
    else if (kpt <= 4) FVAR_SELECT(4);
    else if (kpt <= 8) FVAR_SELECT(8);
    else if (kpt <= kSelKeysMax) FVAR_SELECT(kSelKeysMax);
    else launch(select_large_kernel, grid, block, 0, st, scores, M, k, idx_keep, idx_drop);
#undef FVAR_SELECT
}

}  // namespace fvar
