// 12-bit codes (M = 32 subspaces of 4 dims, 4096 centroids per subspace — the paper's 3-bit-per-
// dimension setting, Section IV-A): nearest-centroid encode and the conversions between the logical
// token-major form [B][Hkv][n][32] uint16 and the device layouts of pq_internal.h.
//
// Encode (Eq. 4 with Section II-C's nearest-centroid assignment) decides as the 8-bit encode: squared Euclidean
// distance in IEEE double as dist = fma(x_j - c_j, x_j - c_j, dist), equal distances to the lowest index.
// Two 12-bit codes share bytes, so the kernel for many tokens does not write the device layout itself: codes go to a
// token-major staging buffer and a second kernel packs them behind the current lengths, one thread per
// 12-byte unit (a V unit holds 8 tokens of one subspace: the thread keeps the codes of tokens it does
// not append).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "pq_internal.h"
#include "pq_device_utils.h"
#include "pq_nearest_filter.h"

namespace {

__device__ inline void pack8(const uint32_t (&c)[8], uint32_t (&w)[3])
{
    w[0] = c[0] | (c[1] << 12) | (c[2] << 24);
    w[1] = (c[2] >> 8) | (c[3] << 4) | (c[4] << 16) | (c[5] << 28);
    w[2] = (c[5] >> 4) | (c[6] << 8) | (c[7] << 20);
}

__device__ inline void unpack8(const uint32_t (&w)[3], uint32_t (&c)[8])
{
    c[0] = w[0] & 0xfffu;
    c[1] = (w[0] >> 12) & 0xfffu;
    c[2] = ((w[0] >> 24) | (w[1] << 8)) & 0xfffu;
    c[3] = (w[1] >> 4) & 0xfffu;
    c[4] = (w[1] >> 16) & 0xfffu;
    c[5] = ((w[1] >> 28) | (w[2] << 4)) & 0xfffu;
    c[6] = (w[2] >> 8) & 0xfffu;
    c[7] = w[2] >> 20;
}

// ---------------------------------------------------------------------------------------------------
// Codes of many tokens, with the matrix cores as a filter (pq_nearest_filter.h; the argument and the error bound are in
// pq_encode.hip).  A workgroup keeps the 4096 A rows of its (K or V, KV head, subspace) in LDS (64 KiB) and each of its
// 8 wavefronts takes 64-token chunks of the head's tokens over all sequences: 128 instructions of 32 centroids per 32
// tokens.  The group of values here is the block of 16 that one instruction leaves in a lane; the 128 blocks of a lane
// half form a grid of 16 rows and 8 columns, whose minima (24 numbers) name the blocks with a value near the smallest
// one.  Nearly always that is one block: its 16 centroids are evaluated in the defining fp64 arithmetic.  Otherwise the
// lane walks all blocks whose row and column are marked, and a codebook or token outside the bound's range the full fp64
// scan.  9.5 vector instructions per matrix instruction and tile, 3177 per 64 tokens and subspace counted with the 256 matrix
// instructions among them: 63 % of the issue slots, the matrix cores busy 40 % of the time (2048 tokens x 32 heads, K and V,
// 550 us).
// SPLIT (a head has at most 128 tokens in the call — a decoding step of a batch): all eight wavefronts take the SAME
// tokens and an eighth of the centroids each, keep their 16 block minima and exchange the smallest value and the
// marked blocks (one word per token and wavefront) through LDS; wavefront 0 refines.
// (16 x 32 heads x 64 tokens: 730 us with 4x4x4 instructions in two passes, 295 us now; 8192 tokens x 32
// heads 5.57 -> 1.74 ms; 17 x 32 x 1, SPLIT, 80 -> 48 us.)
// ---------------------------------------------------------------------------------------------------
typedef uint32_t u32x2e __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8e __attribute__((ext_vector_type(8)));

constexpr int F12_WAVES = 8;  // wavefronts that share one set of A rows
constexpr int F12_ROW = pq_filter_row_bytes<_Float16>();

template <bool SPLIT>
__global__ __launch_bounds__(F12_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void pq12_encode_fast_kernel(
    const __half *x0, const __half *x1, const __half *cb0, const __half *cb1, uint16_t *out0, uint16_t *out1, int B, int Hkv,
    int n_new, int groups_per_head, int rounds, int64_t x_head_stride)
{
#pragma clang fp contract(off)
    __shared__ __attribute__((aligned(16))) unsigned char arow[PQ12_CENTROIDS * F12_ROW];
    __shared__ uint32_t xchg[SPLIT ? F12_WAVES * 64 : 1];  // SPLIT: per wavefront and token
    __shared__ int any_bad;
    __shared__ float wave_c_max[F12_WAVES];
    typedef pq_filter_token<4, _Float16> token;
    typedef token::operand operand;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int which = blockIdx.z;  // 0: keys, 1: values
    const int i = blockIdx.y;      // subspace
    const int n_tok = B * n_new;   // tokens of one KV head over all sequences
    const int n_chunks = (n_tok + 63) >> 6;
    const int hkv = blockIdx.x / groups_per_head;
    const int group = blockIdx.x - hkv * groups_per_head;
    // SPLIT: the workgroup's eight wavefronts share the head's chunks; otherwise `rounds` chunks in a row each
    const int chunk0 = SPLIT ? 0 : (group * F12_WAVES + wave) * rounds;
    const int chunk1 = SPLIT ? n_chunks : (chunk0 + rounds < n_chunks ? chunk0 + rounds : n_chunks);
    const __half *x = which ? x1 : x0;
    const __half *cb = (which ? cb1 : cb0) + ((int64_t)hkv * PQ12_M + i) * PQ12_CENTROIDS * 4;
    uint16_t *out = which ? out1 : out0;

    // ---- A rows of the 4096 centroids
    constexpr int PER_THREAD = PQ12_CENTROIDS / (F12_WAVES * 64);
    f16x4 y[PER_THREAD];
    float c_max = 0.f;
#pragma unroll
    for (int r = 0; r < PER_THREAD; ++r) {
        y[r] = __builtin_bit_cast(f16x4, *(const u32x2e *)(cb + (tid + r * (F12_WAVES * 64)) * 4));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            c_max = fmaxf(c_max, fabsf((float)y[r][j]));
    }
    c_max = pq_filter_wave_max(c_max);
    if (lane == 0)
        wave_c_max[wave] = c_max;
    if (tid == 0)
        any_bad = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < F12_WAVES; ++w)
        c_max = fmaxf(c_max, wave_c_max[w]);
    const float scale = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(pq_filter_scale<_Float16>(c_max))));
    bool cb_bad = false;
#pragma unroll
    for (int r = 0; r < PER_THREAD; ++r) {
        const _Float16 c[4] = {y[r][0], y[r][1], y[r][2], y[r][3]};
        pq_filter_build_row<4>(c, scale, arow + (tid + r * (F12_WAVES * 64)) * F12_ROW, cb_bad);
    }
    if (cb_bad)
        any_bad = 1;
    __syncthreads();
    cb_bad = any_bad != 0;

    const unsigned char *my_row = arow + (lane & 31) * F12_ROW + (lane >> 5) * (F12_ROW / 2);
    const auto block_min = [](const f32x16e &d) {
        int b = min(__float_as_int(d[0]), __float_as_int(d[1]));
#pragma unroll
        for (int k = 2; k < 16; k += 2)
            b = min(min(b, __float_as_int(d[k])), __float_as_int(d[k + 1]));
        return b;
    };

#pragma unroll 1
    for (int chunk = chunk0; chunk < chunk1; ++chunk) {
        const int u = chunk * 64 + lane;
        const bool live = u < n_tok;
        const int uu = live ? u : 0;
        const int b = uu / n_new;
        const int t = uu - b * n_new;
        // x is [B][Hkv][x_head_stride >= n_new][d]
        const f16x4 v = __builtin_bit_cast(
            f16x4, *(const u32x2e *)(x + ((((int64_t)b * Hkv + hkv) * x_head_stride + t) * PQ_HEAD_DIM + i * 4)));
        const _Float16 xv[4] = {v[0], v[1], v[2], v[3]};
        token tok;
        tok.set(xv, scale);

        int code = 0;
        double bd = __builtin_huge_val();
        auto distance = [&](int c) {
            const f16x4 y = *(const f16x4 *)(arow + c * F12_ROW);
            double dist = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double diff = (double)tok.x[j] - (double)(float)y[j];
                dist = __builtin_fma(diff, diff, dist);
            }
            return dist;
        };
        // block m of lane half s: centroids c0 + 8 g + k, c0 = 32 m + 4 s, in ascending order; the smaller (distance,
        // index) stays (strict "<" inside a block, but the blocks of the two halves interleave)
        auto take_block = [&](int c0) {
            double d = __builtin_huge_val();
            int at = 0;
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double dist = distance(c0 + 8 * g + k);
                    at = dist < d ? 8 * g + k : at;
                    d = __builtin_fmin(d, dist);
                }
            at += c0;
            const bool closer = (d < bd) | ((d == bd) & (at < code));
            code = closer ? at : code;
            bd = closer ? d : bd;
        };

        uint32_t words[8];     // word w: the marked blocks 16 w + k of half 0 (bit k) and half 1 (bit 16 + k)
        bool many;             // this lane's token has several blocks to walk, in `words`
        bool none;             // no mark at all
        if constexpr (SPLIT) {
            int blocks[2][16], low[2], limit[2];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const operand A = *(const operand *)(my_row + (16 * wave + k) * (32 * F12_ROW));
#pragma unroll
                for (int tile = 0; tile < 2; ++tile)
                    blocks[tile][k] = block_min(tok.values(A, tile));
            }
#pragma unroll
            for (int tile = 0; tile < 2; ++tile) {
                low[tile] = blocks[tile][0];
#pragma unroll
                for (int k = 1; k < 16; ++k)
                    low[tile] = min(low[tile], blocks[tile][k]);
            }
            int best = tok.best_of(low[0], low[1]);
            xchg[wave * 64 + lane] = (uint32_t)best;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < F12_WAVES; ++w)
                best = min(best, (int)xchg[w * 64 + lane]);
            tok.limits(best, limit);
            uint32_t word[2] = {0u, 0u};
#pragma unroll
            for (int tile = 0; tile < 2; ++tile)
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    word[tile] |= blocks[tile][k] <= limit[tile] ? 1u << k : 0u;
            const auto halves = __builtin_amdgcn_permlane32_swap(word[0], word[1], false, false);
            __syncthreads();  // every wavefront has read the minima
            xchg[wave * 64 + lane] = halves[0] | (halves[1] << 16);
            __syncthreads();
            int count = 0, at = 0;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                words[w] = xchg[w * 64 + lane];
                count += __builtin_popcount(words[w]);
                at = words[w] ? 32 * w + __builtin_ctz(words[w]) : at;
            }
            __syncthreads();  // ... and the words
            many = count > 1;
            none = count == 0;
            if (wave == 0)  // wavefront 0 refines and stores for the workgroup
                take_block(32 * (16 * (at >> 5) + (at & 15)) + ((at & 16) ? 4 : 0));
        } else {
            int by_row[2][16], by_col[2][8], limit[2];
#pragma unroll
            for (int tile = 0; tile < 2; ++tile)
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    by_col[tile][c] = 0x7f800000;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
#pragma unroll
                for (int c = 0; c < 8; c += 2) {
                    const operand A0 = *(const operand *)(my_row + (8 * r + c) * (32 * F12_ROW));
                    const operand A1 = *(const operand *)(my_row + (8 * r + c + 1) * (32 * F12_ROW));
#pragma unroll
                    for (int tile = 0; tile < 2; ++tile) {
                        const int m0 = block_min(tok.values(A0, tile));
                        const int m1 = block_min(tok.values(A1, tile));
                        by_row[tile][r] = c == 0 ? min(m0, m1) : min(min(by_row[tile][r], m0), m1);
                        by_col[tile][c] = min(by_col[tile][c], m0);
                        by_col[tile][c + 1] = min(by_col[tile][c + 1], m1);
                    }
                }
            }
            int low[2];
#pragma unroll
            for (int tile = 0; tile < 2; ++tile) {
                low[tile] = by_col[tile][0];
#pragma unroll
                for (int c = 1; c < 8; ++c)
                    low[tile] = min(low[tile], by_col[tile][c]);
            }
            tok.limits(tok.best_of(low[0], low[1]), limit);
            pq_filter_marks<16, 8> marks;
#pragma unroll
            for (int tile = 0; tile < 2; ++tile)
                marks.add(tile, by_row[tile], by_col[tile], limit[tile]);
            take_block(marks.index(256, 32, 4));
            many = __builtin_amdgcn_inverse_ballot_w64(marks.several);
            none = !__builtin_amdgcn_inverse_ballot_w64(marks.some);
            if (marks.several != 0) {  // wave-uniform
                const auto halves = __builtin_amdgcn_permlane32_swap(pq_filter_mark_word(by_row[0], by_col[0], limit[0]),
                                                                     pq_filter_mark_word(by_row[1], by_col[1], limit[1]), false, false);
#pragma unroll
                for (int w = 0; w < 8; ++w) {  // rows 2 w and 2 w + 1
                    words[w] = 0u;
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        const uint32_t cols = halves[s] & 0xffu, rows = (halves[s] >> (8 + 2 * w)) & 3u;
                        words[w] |= ((rows & 1u ? cols : 0u) | (rows & 2u ? cols << 8 : 0u)) << (16 * s);
                    }
                }
            }
        }
        if (SPLIT && wave != 0)
            continue;
        const bool bad = cb_bad || tok.bad;
        many = many && live && !bad;
        if (__builtin_amdgcn_ballot_w64(many) != 0) {  // wave-uniform: every marked block of the lane's token
            const int code_one = code;
            const double bd_one = bd;
            code = 0;
            bd = __builtin_huge_val();
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                uint32_t left = many ? words[w] : 0u;
                while (__builtin_amdgcn_ballot_w64(left != 0u) != 0) {
                    const int k = left ? __builtin_ctz(left) : 0;
                    const int code_before = code;
                    const double bd_before = bd;
                    take_block(32 * (16 * w + (k & 15)) + ((k & 16) ? 4 : 0));
                    if (left == 0u) {  // this lane had nothing left: keep what it had
                        code = code_before;
                        bd = bd_before;
                    }
                    left &= left - 1u;
                }
            }
            if (!many) {
                code = code_one;
                bd = bd_one;
            }
        }
        if (__builtin_amdgcn_ballot_w64(live && (bad || none)) != 0) {  // wave-uniform: the defining scan for this chunk
            code = 0;
            bd = __builtin_huge_val();
            for (int c = 0; c < PQ12_CENTROIDS; ++c) {
                const double dist = distance(c);
                code = dist < bd ? c : code;  // ascending, strict "<": the lowest index among equal distances stays
                bd = __builtin_fmin(bd, dist);
            }
        }
        if (live)
            out[((((int64_t)b * Hkv + hkv) * n_new + t)) * PQ12_M + i] = (uint16_t)code;
    }
}

// ---------------------------------------------------------------------------------------------------
// A handful of tokens per KV head (one decoding step of a small batch): thread = CENTROIDS.  The filter kernel
// above would build 4096 rows for a wavefront with a few live lanes; here the 512 threads of a workgroup hold 8
// centroids each as fp16 in registers.  Two phases: fp32 distances, whose least over the workgroup bounds the
// centroids that can be the nearest (a bound relative to the distance itself), then the defining fp64 distances
// of those alone (ascending index per thread, strict "<"); the workgroup takes the lexicographic minimum of
// (distance, index): the lowest index among equal distances, as in the scan.  The floor is reading the codebooks
// once (64 MiB for K and V of 32 heads, 9.5 us at 7.05 TB/s).  At 50 registers and 8 wavefronts per workgroup all workgroups of 32 heads are
// resident in two rounds, with 128 KiB of loads under way per compute unit; 4 wavefronts per workgroup took 1.4 us
// longer.  An append of one token with the length update, 32 heads: 21.3 us when every distance was taken in fp64
// by 1024 threads, 17.4 us so; 4 tokens 39.2 and 27.6 us.  The code goes straight into the device layout — no staging, no
// packing kernels: a 12-bit field of a unit that other workgroups (K: the token's other subspaces) or nobody else in
// this call (V) writes, so it is cleared and set with two device-scope atomics per 32-bit word it touches;
// fields are disjoint, so the order of the workgroups does not matter.  Tokens beyond the capacity are not
// written (the length update flags them).
// ---------------------------------------------------------------------------------------------------
constexpr int FEW12_TOKENS = 8;  // tokens per head over all sequences
constexpr int FEW12_WAVES = 8;

__global__ __launch_bounds__(FEW12_WAVES * 64) __attribute__((amdgpu_waves_per_eu(8))) void pq12_encode_few_kernel(const __half *x0, const __half *x1,
                                                                          const __half *cb0, const __half *cb1,
                                                                          uint8_t *codes0, uint8_t *codes1,
                                                                          const int32_t *ctx_len, int B, int Hkv, int n_new,
                                                                          int64_t x_head_stride, int max_context,
                                                                          int64_t head_stride)
{
#pragma clang fp contract(off)
    static_assert(FEW12_WAVES == 8 && FEW12_TOKENS <= FEW12_WAVES, "lane u fetches token u, wavefront u finishes it");
    __shared__ float red_f[64 / FEW12_WAVES][FEW12_WAVES];
    __shared__ double red_d[FEW12_TOKENS][FEW12_WAVES];
    __shared__ int red_c[FEW12_TOKENS][FEW12_WAVES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int which = blockIdx.z;
    const int i = blockIdx.y;
    const int hkv = blockIdx.x;
    const int n_tok = B * n_new;  // <= FEW12_TOKENS
    const __half *x = which ? x1 : x0;
    const __half *cb = (which ? cb1 : cb0) + ((int64_t)hkv * PQ12_M + i) * PQ12_CENTROIDS * 4;
    uint8_t *codes = which ? codes1 : codes0;

    // vector r: centroids 2 * (64 * FEW12_WAVES * r + tid) and the next one, 16 bytes
    constexpr int NV = PQ12_CENTROIDS / (2 * 64 * FEW12_WAVES);
    f16x8e raw[NV];
#pragma unroll
    for (int r = 0; r < NV; ++r)
        raw[r] = *(const f16x8e *)(cb + (int64_t)(64 * FEW12_WAVES * r + tid) * 8);
    // lane u < n_tok of every wavefront fetches token u's sub-vector
    const int u_mine = lane < n_tok ? lane : 0;
    const int b_mine = u_mine / n_new;
    const int t_mine = u_mine - b_mine * n_new;
    const int p0_mine = ctx_len[b_mine];
    float x_mine[4];
    {
        const u32x2e raw_x = *(const u32x2e *)(x + ((((int64_t)b_mine * Hkv + hkv) * x_head_stride + t_mine) * PQ_HEAD_DIM + i * 4));
        const f16x4 v = __builtin_bit_cast(f16x4, raw_x);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            x_mine[j] = (float)v[j];
    }

    // fp32 distances: differences and sums of squares, each rounding relative to its own result, so that a distance is
    // within (2 + 4) * 2^-24 of its exact value; fp16 inputs reach neither the fp32 subnormals nor the overflow
    const auto token = [&](const int u, float (&xv)[4]) {
#pragma unroll
        for (int r = 0; r < NV; ++r)
            asm volatile("" : "+v"(raw[r]));  // converted for each token: held as fp32 the centroids would take 64 registers
#pragma unroll
        for (int j = 0; j < 4; ++j)
            xv[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x_mine[j]), u));
    };
    float minus_one = -1.f;  // not a constant to the compiler: v_fma_mix_f32 subtracts the fp16 value in one instruction
    asm("" : "+s"(minus_one));
    const auto rounded = [&](const int k, const float (&xv)[4]) {
        float d = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float diff = __builtin_fmaf((float)raw[k >> 1][4 * (k & 1) + j], minus_one, xv[j]);
            d = j == 0 ? diff * diff : __builtin_fmaf(diff, diff, d);
        }
        return d;
    };
    for (int u = 0; u < n_tok; ++u) {
        float xv[4];
        token(u, xv);
        float least = __builtin_huge_valf();
#pragma unroll
        for (int k = 0; k < 2 * NV; ++k)
            least = __builtin_fminf(least, rounded(k, xv));  // (a NaN is never the minimum)
        least = -wave_max(-least);
        if (lane == 0)
            red_f[u][wave] = least;
    }
    __syncthreads();
    // the defining distances of the centroids that can be the nearest: most wavefronts have none
    // lane 8 u + w: wavefront w's least for token u, the token's least over the 8 wavefronts, the limit
    const float leasts = (&red_f[0][0])[lane];
    float limits = leasts;
    limits = __builtin_fminf(limits, dpp_move<0xB1>(limits));   // quad_perm [1,0,3,2]
    limits = __builtin_fminf(limits, dpp_move<0x4E>(limits));   // quad_perm [2,3,0,1]
    limits = __builtin_fminf(limits, dpp_move<0x141>(limits));  // row_half_mirror
    // 16 * 2^-24 covers the error of both distances of a comparison (12 * 2^-24) and the roundings of the limit
    limits *= 1.f + 0x1p-20f;
    const int first = __builtin_amdgcn_readfirstlane(wave);
    for (int u = 0; u < n_tok; ++u) {
        const int limit_bits = __builtin_amdgcn_readlane(__float_as_int(limits), FEW12_WAVES * u);
        const float limit = __int_as_float(limit_bits);
        double bd = __builtin_huge_val();
        int bc = PQ12_CENTROIDS;
        if (__builtin_amdgcn_readlane(__float_as_int(leasts), FEW12_WAVES * u + first) <= limit_bits) {  // (both >= +0)
            float xv[4];
            token(u, xv);
            bc = 2 * tid;  // (no distance below infinity: the lowest index)
#pragma unroll
            for (int k = 0; k < 2 * NV; ++k) {
                if (rounded(k, xv) <= limit) {
                    double d = 0.0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double diff = (double)xv[j] - (double)(float)raw[k >> 1][4 * (k & 1) + j];
                        d = __builtin_fma(diff, diff, d);
                    }
                    // ascending index inside the thread, strict "<"
                    bc = d < bd ? 2 * (64 * FEW12_WAVES * (k >> 1) + tid) + (k & 1) : bc;
                    bd = __builtin_fmin(bd, d);
                }
            }
            wave_argmin(bd, bc);
        }
        if (lane == 0) {
            red_d[u][wave] = bd;
            red_c[u][wave] = bc;
        }
    }
    __syncthreads();
    // wavefront u finishes token u: the wavefronts' candidates are repeated over its lanes
    if (wave < n_tok) {
        double d = red_d[wave][lane & (FEW12_WAVES - 1)];
        int cc = red_c[wave][lane & (FEW12_WAVES - 1)];
        wave_argmin(d, cc);
        if (lane == 0) {
            const int b = wave / n_new;
            const int t = wave - b * n_new;
            int p0 = __builtin_amdgcn_readlane(p0_mine, wave);
            p0 = p0 < 0 ? 0 : p0;
            const int64_t pos = (int64_t)p0 + t;
            if (pos < max_context) {
                int slot;
                const int64_t unit = which ? pq12_v_unit(pos, i, &slot) : pq12_k_unit(pos, i, &slot);
                unsigned int *w = (unsigned int *)(codes + ((int64_t)b * Hkv + hkv) * head_stride + unit);  // 3 words
                const int bit = 12 * slot;  // the field: bits bit .. bit + 11 of the 96
                const uint64_t field = (uint64_t)((uint32_t)cc & 0xfffu) << (bit & 31);
                const uint64_t mask = (uint64_t)0xfffu << (bit & 31);
                unsigned int *w0 = w + (bit >> 5);
                __hip_atomic_fetch_and(w0, ~(unsigned int)mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_or(w0, (unsigned int)field, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((mask >> 32) != 0) {  // the field runs into the next word
                    __hip_atomic_fetch_and(w0 + 1, ~(unsigned int)(mask >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_or(w0 + 1, (unsigned int)(field >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
    }
}

// K units: one thread per (head, token j of the source, group of 8 subspaces)
__global__ void pq12_pack_k_kernel(const uint16_t *src, uint8_t *dst, const int32_t *pos0, int n, int Hkv, int max_context,
                                   int64_t head_stride, int64_t total)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= total)
        return;
    const int g = (int)(x & 3);
    const int64_t j = (x >> 2) % n;
    const int64_t head = (x >> 2) / n;
    int64_t p0 = pos0 ? pos0[head / Hkv] : 0;
    p0 = p0 < 0 ? 0 : p0;
    const int64_t pos = p0 + j;
    if (pos >= max_context)
        return;
    uint32_t c[8], w[3];
#pragma unroll
    for (int s = 0; s < 8; ++s)
        c[s] = src[(head * n + j) * PQ12_M + 8 * g + s] & 0xfffu;
    pack8(c, w);
    int slot;
    uint32_t *d = (uint32_t *)(dst + head * head_stride + pq12_k_unit(pos, 8 * g, &slot));
    d[0] = w[0];
    d[1] = w[1];
    d[2] = w[2];
}

// V units: one thread per (head, 128-token block touched by the source, group of 4 subspaces, lane)
__global__ void pq12_pack_v_kernel(const uint16_t *src, uint8_t *dst, const int32_t *pos0, int n, int Hkv, int max_context,
                                   int64_t cap_padded, int64_t head_stride, int n_vb, int64_t total)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= total)
        return;
    const int lane = (int)(x & 63);
    const int g = (int)((x >> 6) & 7);
    const int64_t vb_rel = (x >> 9) % n_vb;
    const int64_t head = (x >> 9) / n_vb;
    int64_t p0 = pos0 ? pos0[head / Hkv] : 0;
    p0 = p0 < 0 ? 0 : p0;
    const int64_t vblock = (p0 >> 7) + vb_rel;
    if (vblock * 128 >= cap_padded)
        return;
    const int sub = 4 * g + (lane & 3);
    bool any = false;
    int64_t jj[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t tok = vblock * 128 + (lane >> 2) + 16 * k;
        const int64_t j = tok - p0;
        jj[k] = (j >= 0 && j < n && tok < max_context) ? j : -1;
        any = any || jj[k] >= 0;
    }
    if (!any)
        return;
    int slot;
    uint32_t *d = (uint32_t *)(dst + head * head_stride + pq12_v_unit(vblock * 128 + (lane >> 2), sub, &slot));
    uint32_t w[3] = {d[0], d[1], d[2]}, c[8];
    unpack8(w, c);
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (jj[k] >= 0)
            c[k] = src[(head * n + jj[k]) * PQ12_M + sub] & 0xfffu;
    pack8(c, w);
    d[0] = w[0];
    d[1] = w[1];
    d[2] = w[2];
}

// one thread per code of the token-major tensor
__global__ void pq12_unpack_kernel(const uint8_t *packed, uint16_t *token_major, int kind, int n, int64_t head_stride,
                                   int64_t total)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= total)
        return;
    const int i = (int)(x % PQ12_M);
    const int64_t t = (x / PQ12_M) % n;
    const int64_t head = x / ((int64_t)PQ12_M * n);
    int slot;
    const int64_t unit = kind == PQ_CODES_K ? pq12_k_unit(t, i, &slot) : pq12_v_unit(t, i, &slot);
    const uint8_t *b = packed + head * head_stride + unit + ((3 * slot) >> 1);
    const uint32_t two = (uint32_t)b[0] | ((uint32_t)b[1] << 8);
    token_major[x] = (uint16_t)((two >> (4 * (slot & 1))) & 0xfffu);
}

// codes of tensors 0 .. n_tensors - 1 (K and V, or samples alone) into out [B][Hkv][n_new][32]
hipError_t launch_filter(const __half *x0, const __half *x1, const __half *cb0, const __half *cb1, uint16_t *out0, uint16_t *out1,
                         int n_tensors, int B, int Hkv, int n_new, int64_t x_rows, hipStream_t s)
{
    const int64_t n_tok = (int64_t)B * n_new;  // of a head over all sequences
    if (n_tok <= 128) {
        // a decoding step of a batch: the head's one or two chunks, the centroids split over the workgroup's wavefronts
        const dim3 grid((unsigned)Hkv, PQ12_M, (unsigned)n_tensors);
        hipLaunchKernelGGL(pq12_encode_fast_kernel<true>, grid, dim3(F12_WAVES * 64), 0, s, x0, x1, cb0, cb1, out0, out1, B, Hkv,
                           n_new, 1, 1, x_rows);
    } else {
        // up to 8 chunks in a row per wavefront while at least 1024 workgroups (two rounds of the chip) remain
        const int64_t chunks = (n_tok + 63) / 64;
        const int64_t groups1 = (chunks + F12_WAVES - 1) / F12_WAVES;
        const int64_t most = Hkv * groups1 * PQ12_M * n_tensors / 1024;
        const int rounds = (int)(most < 1 ? 1 : most > 8 ? 8 : most);
        const int groups = (int)((chunks + F12_WAVES * rounds - 1) / (F12_WAVES * rounds));
        const dim3 grid((unsigned)(Hkv * groups), PQ12_M, (unsigned)n_tensors);
        hipLaunchKernelGGL(pq12_encode_fast_kernel<false>, grid, dim3(F12_WAVES * 64), 0, s, x0, x1, cb0, cb1, out0, out1, B, Hkv,
                           n_new, groups, rounds, x_rows);
    }
    return hipGetLastError();
}

hipError_t launch_pack(const pq_attn_ctx *ctx, int kind, const uint16_t *src, int n, uint8_t *dst, const int32_t *pos0,
                       hipStream_t s)
{
    const int64_t heads = (int64_t)ctx->cfg.batch * ctx->cfg.n_kv_heads;
    const int64_t head_stride = ctx->cap_padded * PQ12_TOKEN_BYTES;
    if (n == 0)
        return hipSuccess;
    if (kind == PQ_CODES_K) {
        const int64_t total = heads * n * 4;
        hipLaunchKernelGGL(pq12_pack_k_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, src, dst, pos0, n,
                           ctx->cfg.n_kv_heads, ctx->cfg.max_context, head_stride, total);
    } else {
        const int n_vb = ((n + 127) >> 7) + 1;
        const int64_t total = heads * n_vb * 512;
        hipLaunchKernelGGL(pq12_pack_v_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, src, dst, pos0, n,
                           ctx->cfg.n_kv_heads, ctx->cfg.max_context, ctx->cap_padded, head_stride, n_vb, total);
    }
    return hipGetLastError();
}

}  // namespace

bool pq_config_is_12bit(const pq_attn_config *cfg) { return cfg->n_centroids == PQ12_CENTROIDS; }

hipError_t pq12_launch_pack_codes(const pq_attn_ctx *ctx, int kind, const uint16_t *token_major, int n_tokens,
                                  uint8_t *packed, bool unpack, hipStream_t s)
{
    if (!unpack)
        return launch_pack(ctx, kind, token_major, n_tokens, packed, nullptr, s);
    const int64_t heads = (int64_t)ctx->cfg.batch * ctx->cfg.n_kv_heads;
    const int64_t total = heads * n_tokens * PQ12_M;
    if (total == 0)
        return hipSuccess;
    hipLaunchKernelGGL(pq12_unpack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, packed,
                       const_cast<uint16_t *>(token_major), kind, n_tokens, ctx->cap_padded * PQ12_TOKEN_BYTES, total);
    return hipGetLastError();
}

hipError_t pq12_launch_encode_append(const pq_attn_ctx *ctx, const pq_encode_args &a, int64_t x_rows, int32_t *ctx_len,
                                     unsigned int *dev_err, hipStream_t s)
{
    const int64_t n_tok = (int64_t)a.B * a.n_new;  // tokens of a head over all sequences
    // 32 heads, one new token per sequence, with the length reset and all launches: 1 sequence 17 us, 2 20 us, 4 28 us, 8
    // 43 us with the kernel below; 44 .. 48 us for 1 .. 17 sequences with the split filter kernel.  8 heads, 8 sequences:
    // 19 us and 20 us
    if (n_tok <= FEW12_TOKENS) {
        // a decoding step: encode and write the device layouts in one kernel, then the lengths
        hipLaunchKernelGGL(pq12_encode_few_kernel, dim3((unsigned)a.Hkv, PQ12_M, 2), dim3(FEW12_WAVES * 64), 0, s,
                           (const __half *)a.x[0], (const __half *)a.x[1], (const __half *)a.codebook[0],
                           (const __half *)a.codebook[1], a.codes[0], a.codes[1], a.ctx_len, a.B, a.Hkv, a.n_new, x_rows,
                           a.max_context, ctx->cap_padded * PQ12_TOKEN_BYTES);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        return pq_launch_bump_len(ctx_len, a.B, a.n_new, a.max_context, dev_err, s);
    }
    const hipError_t enc = launch_filter((const __half *)a.x[0], (const __half *)a.x[1], (const __half *)a.codebook[0],
                                         (const __half *)a.codebook[1], ctx->stage[0], ctx->stage[1], 2, a.B, a.Hkv, a.n_new,
                                         x_rows, s);
    if (enc != hipSuccess)
        return enc;
    hipError_t e = launch_pack(ctx, PQ_CODES_K, ctx->stage[0], a.n_new, a.codes[0], a.ctx_len, s);
    if (e != hipSuccess)
        return e;
    e = launch_pack(ctx, PQ_CODES_V, ctx->stage[1], a.n_new, a.codes[1], a.ctx_len, s);
    if (e != hipSuccess)
        return e;
    // the lengths move only after both packing kernels have read the old ones (stream order)
    return pq_launch_bump_len(ctx_len, a.B, a.n_new, a.max_context, dev_err, s);
}

// ---------------------------------------------------------------------------------------------------
// Offline codebook training for 4096 centroids: the Lloyd iteration of pq_kmeans.hip with the assignment done
// by the encode kernel above (chunks of the samples, codes staged in the workspace) and the exact 64-bit
// integer member sums added straight to memory (a subspace has 4096 x 4 sums: they do not fit in LDS, and
// with that many addresses the atomics hardly collide).
// ---------------------------------------------------------------------------------------------------
namespace {

constexpr int KM12_CHUNK = 8192;  // samples per head and assignment launch

// one thread per (head, sample of the chunk, subspace)
__global__ void pq12_kmeans_accumulate_kernel(const __half *samples, const uint16_t *codes, unsigned long long *sums,
                                              unsigned int *counts, int64_t head_stride, int nc, int64_t total)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= total)
        return;
    const int i = (int)(x & (PQ12_M - 1));
    const int64_t tok = (x >> 5) % nc;
    const int64_t head = (x >> 5) / nc;
    const uint32_t c = codes[x] & 0xfffu;
    const __half *v = samples + (head * head_stride + tok) * PQ_HEAD_DIM + i * 4;
    const int64_t e = (head * PQ12_M + i) * PQ12_CENTROIDS + c;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // exact: an fp16 value times 2^24 is an integer below 2^41 in magnitude
        const long long fixed = (long long)(__half2float(v[j]) * 16777216.0f);
        atomicAdd(&sums[e * 4 + j], (unsigned long long)fixed);
    }
    atomicAdd(&counts[e], 1u);
}

}  // namespace

int64_t pq12_kmeans_workspace_bytes(const pq_attn_ctx *ctx)
{
    const int64_t n = (int64_t)ctx->cfg.n_kv_heads * PQ12_M * PQ12_CENTROIDS;
    return n * 4 * 8 + n * 4 + (int64_t)ctx->cfg.n_kv_heads * KM12_CHUNK * PQ12_M * 2;
}

hipError_t pq12_launch_kmeans(const pq_attn_ctx *ctx, const void *samples, int n_samples, void *codebook, int n_iters,
                              void *workspace, hipStream_t s)
{
    const int Hkv = ctx->cfg.n_kv_heads;
    const int64_t n = (int64_t)Hkv * PQ12_M * PQ12_CENTROIDS;
    unsigned long long *sums = (unsigned long long *)workspace;
    unsigned int *counts = (unsigned int *)(sums + n * 4);
    uint16_t *codes = (uint16_t *)(counts + n);
    hipError_t e = pq_launch_clear_words(workspace, (n * 4 * 8 + n * 4) / 4, s);
    if (e != hipSuccess)
        return e;
    for (int it = 0; it < n_iters; ++it) {
        for (int c0 = 0; c0 < n_samples; c0 += KM12_CHUNK) {
            const int nc = n_samples - c0 < KM12_CHUNK ? n_samples - c0 : KM12_CHUNK;
            const __half *x = (const __half *)samples + (int64_t)c0 * PQ_HEAD_DIM;
            // assignment = the encode's matrix-core filter (one sequence, one tensor)
            e = launch_filter(x, x, (const __half *)codebook, (const __half *)codebook, codes, codes, 1, 1, Hkv, nc,
                              (int64_t)n_samples, s);
            if (e != hipSuccess)
                return e;
            const int64_t total = (int64_t)Hkv * nc * PQ12_M;
            hipLaunchKernelGGL(pq12_kmeans_accumulate_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, x, codes,
                               sums, counts, (int64_t)n_samples, nc, total);
        }
        e = pq_launch_kmeans_update(codebook, sums, counts, n, 4, s);
        if (e != hipSuccess)
            return e;
    }
    return hipGetLastError();
}
