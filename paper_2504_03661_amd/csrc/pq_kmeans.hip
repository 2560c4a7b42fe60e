// Offline codebook training: k-means per (KV head, subspace) by Lloyd's iteration on sampled
// key / value vectors (Section II-C, training phase; Section III-A, "Offline PQ Codebook Training").
//
// One iteration = two kernels.
//   assign   every sample sub-vector goes to its nearest centroid — the rule and the arithmetic of
//            the encode kernel: squared Euclidean distance decided in IEEE double as
//            dist = fma(x_j - c_j, x_j - c_j, dist), equal distances to the lowest index — and is
//            added to that centroid's member sum and count.  fp16 values are integers times
//            2^-24, so the sums are kept as 64-bit integers: exact, and independent of the order in
//            which the atomics land (n_samples <= 2^20 keeps them below 2^61).
//   update   centroid = double(sum) * 2^-24 / count in IEEE double, rounded to float and from there
//            to fp16; a centroid without members keeps its value.  The kernel also clears the
//            accumulators for the next iteration.
// The paper does not say how it initialises, iterates or treats empty clusters; the initial
// centroids are the caller's, the iteration count too.
//
// Mapping of `assign`: one workgroup = (head, 4 neighbouring subspaces, slice of samples), one wavefront per
// subspace, lane = sample, 64 samples at a time.  Every wavefront keeps its subspace's codebook rows and partial sums
// in LDS (LDS atomics); the sums reach memory with one 64-bit atomic per touched entry and slice.  The 4 wavefronts
// read neighbouring words of the same rows, so a line of samples leaves L2 once for all of them.  Bound by the issue
// of vector instructions in the nearest-centroid filter, as the encode; 32 heads x 65536 samples, M = 64: 2.7 ms per
// iteration with one subspace per workgroup and the two-pass filter, 1.58 ms with the one-pass filter (two or four
// wavefronts per subspace on one set of sums, for more wavefronts per compute unit: 1.6 and 1.8 ms).  As many samples as
// that take the grids of pq_nearest_grid.h at M = 64 (pq_kmeans_grid_kernel): 0.44 ms
// (0.47 where the channels' scales go from 1/2 to 2).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "pq_internal.h"
#include "pq_nearest_filter.h"
#include "pq_nearest_grid.h"

namespace {

constexpr int KM_SUB = 4;  // neighbouring subspaces per workgroup, one wavefront each

template <int M, int DS>
__global__ __launch_bounds__(KM_SUB * 64) void pq_kmeans_assign_kernel(const __half *samples, const __half *codebook,
                                                                      unsigned long long *sums, unsigned int *counts,
                                                                      int n_samples, int n_slices, int rounds)
{
    __shared__ __attribute__((aligned(16))) unsigned char arow_all[KM_SUB][256 * pq_filter_row_bytes<_Float16>()];
    __shared__ unsigned long long sum_all[KM_SUB][256 * DS];
    __shared__ unsigned int cnt_all[KM_SUB][256];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char *arow = arow_all[wave];
    unsigned long long *part_sum = sum_all[wave];
    unsigned int *part_cnt = cnt_all[wave];
    const int head = blockIdx.x / n_slices;
    const int slice = blockIdx.x - head * n_slices;
    const int i = blockIdx.y * KM_SUB + wave;  // subspace

    // matrix-instruction rows of this (head, subspace)'s codebook for the nearest-centroid filter of the encode
    // (pq_nearest_filter.h); accumulators cleared
    const int64_t cb_base = ((int64_t)head * M + i) * 256 * DS;
    _Float16 y[4][DS];
    float c_max = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = lane + 64 * r;
#pragma unroll
        for (int j = 0; j < DS; ++j) {
            y[r][j] = ((const _Float16 *)codebook)[cb_base + c * DS + j];
            c_max = fmaxf(c_max, fabsf((float)y[r][j]));
            part_sum[c * DS + j] = 0ull;
        }
        part_cnt[c] = 0u;
    }
    const float scale =
        __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(pq_filter_scale<_Float16>(pq_filter_wave_max(c_max)))));
    bool cb_bad = false;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        pq_filter_build_row<DS>(y[r], scale, arow + (lane + 64 * r) * pq_filter_row_bytes<_Float16>(), cb_bad);
    cb_bad = __builtin_amdgcn_ballot_w64(cb_bad) != 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    // the slice's samples, 64 at a time, the next ones' loads in flight while these are assigned (the same rule and
    // arithmetic as the encode)
    const _Float16 *x = (const _Float16 *)samples + (int64_t)head * n_samples * PQ_HEAD_DIM + i * DS;
    const int s0 = slice * rounds * 64;
    const int s1 = s0 + rounds * 64 < n_samples ? s0 + rounds * 64 : n_samples;
    _Float16 next[DS];
    auto fetch = [&](int s) {
        const _Float16 *xp = x + (int64_t)(s < n_samples ? s : 0) * PQ_HEAD_DIM;
#pragma unroll
        for (int j = 0; j < DS; ++j)
            next[j] = xp[j];
    };
    int s = s0 + lane;
    fetch(s);
#pragma unroll 1
    for (; s - lane < s1; s += 64) {
        _Float16 xv[DS];
#pragma unroll
        for (int j = 0; j < DS; ++j)
            xv[j] = next[j];
        fetch(s + 64);
        const bool live = s < s1;
        const int code = pq_filter_code<DS, _Float16, _Float16>(arow, arow, scale, cb_bad, xv, live);
        if (live) {
#pragma unroll
            for (int j = 0; j < DS; ++j) {
                // exact: an fp16 value times 2^24 is an integer below 2^41 in magnitude
                const long long fixed = (long long)((float)xv[j] * 16777216.0f);
                atomicAdd(&part_sum[code * DS + j], (unsigned long long)fixed);
            }
            atomicAdd(&part_cnt[code], 1u);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    const int64_t acc_base = ((int64_t)head * M + i) * 256;
    for (int e = lane; e < 256 * DS; e += 64)
        if (part_sum[e] != 0ull)
            atomicAdd(&sums[acc_base * DS + e], part_sum[e]);
    for (int e = lane; e < 256; e += 64)
        if (part_cnt[e] != 0u)
            atomicAdd(&counts[acc_base + e], part_cnt[e]);
}

// Many samples at ds = 2: the same through the grid of pq_nearest_grid.h.  A workgroup is 4 neighbouring subspaces of a head and
// a slice of the samples; sums and counts of the 4 in LDS.  A coordinate enters its sum as the bits of the double
// x 2^24 + 1.5 2^52: an integer with a constant on top, which the count takes out again.
// The x sums of a subspace stand together, and so do the y sums: a 64-bit add then finds the 64 lanes on 32 pairs of banks (side
// by side x and y had 16 each: 32 heads x 64K samples, 2 iterations, normal data, 912 -> 872 us).
struct pq_sample {
    _Float16 x[GRID_SUB][2];
    bool live;
};

__global__ __launch_bounds__(GRID_WAVES * 64) void pq_kmeans_grid_kernel(const _Float16 *samples, const _Float16 *codebook,
                                                                         unsigned long long *sums, unsigned int *counts, const int n_heads,
                                                                         const int n_samples, const int slices, const int slice_chunks)
{
    constexpr int M = 64;
    __shared__ __attribute__((aligned(16))) pq_grids<_Float16> grids;
    __shared__ __attribute__((aligned(16))) pq_grid_scratch<false> scratch;
    __shared__ float2 box[GRID_SIDE];
    __shared__ unsigned long long sum[GRID_SUB][512];
    __shared__ unsigned int count[GRID_SUB][256];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // an XCD takes whole units of the 16 workgroups that share their samples, one after the other
    const int local = blockIdx.x >> 3;
    const int unit = (local >> 4) * 8 + (blockIdx.x & 7);
    if (unit >= n_heads * slices)
        return;
    const int i0 = (local & 15) * GRID_SUB;
    const int head = unit / slices, slice = unit - head * slices;
    const int n_chunks = (n_samples + 63) >> 6;
    const int first = slice * slice_chunks;
    const int last = first + slice_chunks < n_chunks ? first + slice_chunks : n_chunks;

    for (int e = threadIdx.x; e < GRID_SUB * 512; e += GRID_WAVES * 64)
        ((unsigned long long *)sum)[e] = 0ull;
    for (int e = threadIdx.x; e < GRID_SUB * 256; e += GRID_WAVES * 64)
        ((unsigned int *)count)[e] = 0u;
    pq_grid_build(grids, scratch.making, box, codebook + ((int64_t)head * M + i0) * 512);

    constexpr uint64_t BASE = 0x4338000000000000ull;  // the bits of 1.5 2^52
    const _Float16 *x = samples + (int64_t)head * n_samples * PQ_HEAD_DIM + i0 * 2;
    auto add = [&](int j, int code, _Float16 x0, _Float16 x1) {
        atomicAdd(&sum[j][code], (unsigned long long)__double_as_longlong(__builtin_fma((double)(float)x0, 16777216.0, 6755399441055744.0)));
        atomicAdd(&sum[j][256 + code], (unsigned long long)__double_as_longlong(__builtin_fma((double)(float)x1, 16777216.0, 6755399441055744.0)));
        atomicAdd(&count[j][code], 1u);
    };
    pq_grid_scan<_Float16, false, 0, pq_sample>(
        grids, scratch.queue, first, last,
        [&](int chunk, pq_sample &k) {
            const int s = chunk * 64 + lane;
            k.live = s < n_samples;
            const f16x8 row = *(const f16x8 *)(x + (int64_t)(k.live ? s : n_samples - 1) * PQ_HEAD_DIM);
            __builtin_memcpy(k.x, &row, sizeof(k.x));
        },
        [&](const pq_sample &k, int j, int code, bool decided) {
            if (decided)
                add(j, code, pq_grid_pick(j, k.x[0][0], k.x[1][0], k.x[2][0], k.x[3][0]), pq_grid_pick(j, k.x[0][1], k.x[1][1], k.x[2][1], k.x[3][1]));
        },
        [](const pq_sample &, uint32_t) {},
        [&](uint32_t id, _Float16 &x0, _Float16 &x1) {
            const _Float16 *xp = x + ((int64_t)(first + (int)(id >> 8)) * 64 + (id >> 2 & 63u)) * PQ_HEAD_DIM + (id & 3u) * 2;
            x0 = xp[0];
            x1 = xp[1];
        },
        [&](uint32_t id, _Float16 x0, _Float16 x1, int code) { add((int)(id & 3u), code, x0, x1); });
    __syncthreads();

    const int64_t acc = ((int64_t)head * M + i0) * 256;
    for (int e = threadIdx.x; e < GRID_SUB * 256; e += GRID_WAVES * 64) {
        const unsigned int n = ((const unsigned int *)count)[e];
        if (n == 0u)
            continue;
#pragma unroll
        for (int d = 0; d < 2; ++d)
            atomicAdd(&sums[(acc + e) * 2 + d], sum[e >> 8][d * 256 + (e & 255)] - n * BASE);
        atomicAdd(&counts[acc + e], n);
    }
}

// one thread per (head, subspace, centroid)
template <int DS>
__global__ void pq_kmeans_update_kernel(__half *codebook, unsigned long long *sums, unsigned int *counts, int64_t n)
{
#pragma clang fp contract(off)
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n)
        return;
    const unsigned int count = counts[e];
    if (count != 0u) {
#pragma unroll
        for (int j = 0; j < DS; ++j) {
            const double sum = (double)(long long)sums[e * DS + j];
            const double mean = sum * 5.9604644775390625e-08 / (double)count;  // 2^-24, then one division
            codebook[e * DS + j] = __float2half_rn((float)mean);
            sums[e * DS + j] = 0ull;
        }
        counts[e] = 0u;
    }
}

__global__ void pq_clear_words_kernel(uint32_t *p, int64_t n)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n)
        p[e] = 0u;
}

}  // namespace

hipError_t pq_launch_clear_words(void *p, int64_t words, hipStream_t s)
{
    hipLaunchKernelGGL(pq_clear_words_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, (uint32_t *)p, words);
    return hipGetLastError();
}

hipError_t pq_launch_kmeans_update(void *codebook, unsigned long long *sums, unsigned int *counts, int64_t n, int ds,
                                   hipStream_t s)
{
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    if (ds == 2)
        hipLaunchKernelGGL(pq_kmeans_update_kernel<2>, grid, block, 0, s, (__half *)codebook, sums, counts, n);
    else
        hipLaunchKernelGGL(pq_kmeans_update_kernel<4>, grid, block, 0, s, (__half *)codebook, sums, counts, n);
    return hipGetLastError();
}

int64_t pq_kmeans_accumulator_bytes(const pq_attn_ctx *ctx)
{
    if (pq_config_is_12bit(&ctx->cfg))
        return pq12_kmeans_workspace_bytes(ctx);
    const int64_t n = (int64_t)ctx->cfg.n_kv_heads * ctx->cfg.n_subspaces * 256;
    return n * ctx->ds * 8 + n * 4;
}

hipError_t pq_launch_kmeans(const pq_attn_ctx *ctx, const void *samples, int n_samples, void *codebook, int n_iters,
                            void *workspace, hipStream_t s)
{
    if (pq_config_is_12bit(&ctx->cfg))
        return pq12_launch_kmeans(ctx, samples, n_samples, codebook, n_iters, workspace, s);
    const int Hkv = ctx->cfg.n_kv_heads, M = ctx->cfg.n_subspaces, DS = ctx->ds;
    const int64_t n = (int64_t)Hkv * M * 256;
    unsigned long long *sums = (unsigned long long *)workspace;
    unsigned int *counts = (unsigned int *)(sums + n * DS);
    const int64_t words = pq_kmeans_accumulator_bytes(ctx) / 4;
    hipLaunchKernelGGL(pq_clear_words_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s,
                       (uint32_t *)workspace, words);
    // A wavefront takes several chunks of 64 samples in a row: one codebook set-up and one pass of up to 256 (ds + 1)
    // memory atomics for all of them.  Taken as resident are 3072 wavefronts, 3 workgroups per compute unit: few samples
    // make one round of them (8 heads x 2000: 31 us; 40 with 8192 wavefronts, 33 with one subspace per workgroup), many
    // between two and three (8 heads x 30000: 219 us; on a faster box 209, and 236 with 3072 wavefronts, whose last round
    // is a third full).
    const int n_chunks = (n_samples + 63) / 64;
    const int64_t waves = (int64_t)Hkv * n_chunks * M;
    const int64_t one_round = (waves + 3071) / 3072, several = waves / 8192;
    const int rounds = (int)(several > 64 ? 64 : several > 16 ? several : one_round < 16 ? one_round : 16);
    const int n_slices = (n_chunks + rounds - 1) / rounds;
    const dim3 grid((unsigned)(Hkv * n_slices), (unsigned)(M / KM_SUB)), block(KM_SUB * 64);
    // (its 16-byte loads ask for samples that start at such an address)
    const int grid_slices = M == 64 && ((uintptr_t)samples & 15) == 0 ? pq_grid_slices(n_chunks, n_chunks, (int64_t)Hkv * 16, ctx->n_cu) : 0;
    for (int it = 0; it < n_iters; ++it) {
        if (grid_slices > 0) {
            hipLaunchKernelGGL(pq_kmeans_grid_kernel, dim3((unsigned)((Hkv * grid_slices + 7) / 8 * 128)), dim3(GRID_WAVES * 64), 0, s,
                               (const _Float16 *)samples, (const _Float16 *)codebook, sums, counts, Hkv, n_samples, grid_slices,
                               (n_chunks + grid_slices - 1) / grid_slices);
            hipLaunchKernelGGL(pq_kmeans_update_kernel<2>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                               (__half *)codebook, sums, counts, n);
        } else if (M == 64) {
            hipLaunchKernelGGL((pq_kmeans_assign_kernel<64, 2>), grid, block, 0, s, (const __half *)samples,
                               (const __half *)codebook, sums, counts, n_samples, n_slices, rounds);
            hipLaunchKernelGGL(pq_kmeans_update_kernel<2>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                               (__half *)codebook, sums, counts, n);
        } else {
            hipLaunchKernelGGL((pq_kmeans_assign_kernel<32, 4>), grid, block, 0, s, (const __half *)samples,
                               (const __half *)codebook, sums, counts, n_samples, n_slices, rounds);
            hipLaunchKernelGGL(pq_kmeans_update_kernel<4>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                               (__half *)codebook, sums, counts, n);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipGetLastError();
}
