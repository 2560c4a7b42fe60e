// Nearest-centroid encode of new tokens, appended to the code tensors in place.
//
// Eq. 4 read with Section II-C ("assigned to the nearest centroid in its subspace"):
//   code[t][i] = argmin_c sum_j (x[t][i*ds + j] - C^i[c][j])^2,   ties -> lowest c.
// The comparison is decided in IEEE double: inputs widened exactly, and for
// j = 0 .. ds-1 in order dist = fma(x_j - c_j, x_j - c_j, dist): each difference and
// each fused multiply-add rounded once, nothing else contracted (this file is compiled
// with -ffp-contract=off and the loop below also pins it with a pragma).  fp64 vector
// arithmetic runs at the same rate as unpacked fp32 on gfx950, so exactness costs
// nothing here; a scan of all centroids costs 2 ds + 3 vector operations per (sub-vector, centroid).
//
// Appends of more than a few tokens reach the codes through pq_encode_fast_kernel, where the matrix cores find the
// few centroids that can be the nearest and the expression above decides among them; a handful of tokens per head
// through pq_encode_few_kernel, where the fp32 distances to all 256 do; thousands per head at M = 64 through
// pq_encode_grid_kernel, which looks the candidates up.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <string.h>

#include <type_traits>

#include "pq_internal.h"
#include "pq_device_utils.h"
#include "pq_nearest_filter.h"
#include "pq_nearest_grid.h"

namespace {

// ---------------------------------------------------------------------------------
// The codes of many tokens, found with the matrix cores as a filter (pq_nearest_filter.h); fp16 inputs first.
//
// With q(c) = n(c)/2 - x . c (n = |c|^2) the distance is |x|^2 + 2 q, so the nearest centroid minimises q.
// For fp16 inputs every product x_j c_j is exact in fp32, and v_mfma_f32_32x32x8_f16 evaluates
// v(c) = q(c) + off for 32 centroids (rows of A, from LDS) x 32 tokens (columns of B) per instruction, to within a
// bound e_c that follows from the magnitudes (below); off >= |x|^2/2 is a per-token number, itself one of the
// products, that makes every computed value positive, so that values compare as integers (v_min3_i32: half a vector
// operation per value, no NaN quieting).  That is a filter, not the decision:
//   values  every instruction leaves a lane with 16 of its token's values, in 4 "quads" of consecutive centroids.
//           Kept of the 8 instructions of a token are the minima over the quads of each instruction (8) and over the
//           instructions for each quad position (4).  Their minimum over both lane halves is the best value.
//   marks   the minima within tau of the best one.  A quad can hold a value that close only if its instruction AND
//           its position are marked: nearly always one of each, in one of the halves, and so one quad, found without
//           a second pass over the values.  The comparisons leave lane masks in scalar registers, where they are
//           combined.
//   refine  the distances of the marked quad's 4 centroids in the defining fp64 arithmetic (see the top of this
//           file), ascending, the smallest, lowest index first, is the code.  Where more than one instruction or
//           position is marked (ties, duplicated centroids, near-ties) the lane walks all quads that both marks allow.
//           A codebook or token outside the range the bound covers (norms beyond fp16, no mark, non-finite values):
//           the 64-token chunk runs the full fp64 scan.
// Either way the code is decided by the fp64 expression, so it is bit-exact by construction; the filter only has to be
// SAFE: every centroid outside the evaluated quads must have a strictly larger true distance.
// Bound: A row = (c_0 .. c_{ds-1}, h, l, 1, 2^15) with h + l = n/2 split into two fp16 (n summed in fp32: <= 3.5 x
// 2^-23 of n/2 in all, or the subnormal step 2^-25), B column = (-x_0 .. -x_{ds-1}, 1, 1, o_0, o_1); the at most 8
// terms are summed within 8 x 2^-23 of their magnitudes (measured over 2^-20 .. 2^15: at most 2.5 x 2^-23, and 7e-12
// absolute below 2^-14).  So e_c <= eps T_c, eps = 11.5 x 2^-23, T_c = n/2 + sum_j |x_j c_j| + off.  With d = |x - c|:
// |c| <= |x| + d, hence T_c <= 2.5 |x|^2 + 1.5 d^2 + off, and d^2 = 2 v(c) - 2 off + |x|^2 gives T_c <= 3 |x|^2 + 3 v(c):
// a centroid's error is bounded by its own value and the token, whatever outliers the codebook holds.  An unmarked
// c has computed v(c) > best + tau, so its true value exceeds that of the computed minimiser if
// tau >= 6 eps (|x|^2 + best) / (1 - 3 eps); tau = 1.05e-5 (|x|^2 + best) + 2^-22 is 1.27 times that, which is many
// orders above the rounding of the fp64 distances.  The same bound keeps every computed value positive:
// v(c) >= off - |x|^2/2 >= 0.0025 |x|^2 + 7e-7 > e_c.  (A tau from the largest norm of the codebook, some 7 times as
// wide, sent a quarter of all chunks through the walk over several quads.)
// The matrix instruction takes fp16 subnormals as they are (no flush: measured, and the default mode of a HIP kernel).
// Codebooks of small numbers: rows and offset carry a gain g = s^2 (pq_filter_scale), with which the above holds for s x and
// s c in the place of x and c — the products x_j (g c_j) are as exact, and no gain makes a coordinate of a row inexact.  The
// refinement compares the distances of g x and g c, g^2 times the true ones: the same order and the same ties.
//
// fp32 inputs run the same filter on split operands: coordinates are scaled by a power of two that brings the
// codebook's largest into [32, 64) and split into two fp16, v = v' + v'' (to 2^-22 of v, or 2^-25), and
// v_mfma_f32_32x32x16_f16 sums x'c' + x'c'' + x''c' and the same last four terms.  Against the fp16 bound: twice the
// terms of the sum (16 x 2^-23), 3 x 2^-22 of |x_j c_j| for what the split drops, 4 x 2^-23 for n/2 — eps = 26 x 2^-23 —
// and absolute terms 2^-25 (|x_j| + |c_j|), which with |c| <= |x| + d stay below 2^-24 (1.5 + |x|^2 + v): tau =
// 2.5e-5 (|x|^2 + best) + 2^-22 is 1.33 x 6 eps.  The refinement reads the unscaled fp32 coordinates.  A token longer
// than some 1000 times the codebook's largest coordinate leaves the range and sends its chunk through the full scan.
// (8192 tokens x 32 heads x (K, V), fp32: the full scan for every token 1.79 ms at M = 64 and 1.50 ms at M = 32, now
// 0.46 and 0.26 ms.)
//
// Cost per (sub-vector, centroid): 1.4 vector operations instead of 2 ds + 3 in fp64, the matrix instructions in
// parallel: 355 vector instructions per 64 tokens and subspace counted at M = 64, 16 of them matrix instructions, which
// fill 82 % of the issue slots at the 2.0 GHz the chip holds (M = 32: 394, 82 %; fp32, M = 64: 407, 78 %); what the
// wavefronts wait for in the rest is not known.  Prompt of 32K tokens x 32 heads x (K, V), M = 64: 2.75 ms with 4x4x4
// instructions in two passes (one for the best value, one for the marks), 1.54 ms in one; appends of that size go through
// the grids now (0.37 ms).
//
// A workgroup is 4 neighbouring subspaces of the same tokens, one wavefront each: a token's line of 64 subspaces is
// then fetched from L2 once for four wavefronts (one wavefront per workgroup 2.69 ms, two 2.35, four 1.75, eight 1.73
// on the same box and an earlier filter; eight run out of LDS at M = 32: 124 -> 175 us on 3 x 5000 tokens x 8 heads).
// fp16: a fp64 copy of the coordinates stays in LDS for ds = 2 (converting them at each use: 1.76 -> 1.89 ms); for ds = 4
// its 32 KiB cost more wavefronts than the conversions cost instructions (124 -> 111 us).
constexpr int FAST_WAVES = 4;

template <int M, int DS, typename T, bool PER_SEQ>
__global__ __launch_bounds__(FAST_WAVES * 64) void pq_encode_fast_kernel(const pq_encode_args a, const int rounds)
{
    // T: _Float16 or float; W: what the centroids' coordinates are kept as for the refinement
    typedef typename std::conditional<sizeof(T) == 4, float, typename std::conditional<DS == 2, double, _Float16>::type>::type W;
    constexpr int ROW = pq_filter_row_bytes<T>();
    __shared__ __attribute__((aligned(16))) unsigned char arow_all[FAST_WAVES][256 * ROW];
    __shared__ __attribute__((aligned(16))) W coord_all[FAST_WAVES][sizeof(W) == 2 ? 1 : 256 * DS];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char *arow = arow_all[wave];
    W *coord = coord_all[wave];
    const int which = blockIdx.z;                  // 0: keys, 1: values
    const int i = blockIdx.y * FAST_WAVES + wave;  // subspace
    // chunks of 64 tokens of one KV head over all sequences (they share its codebook): whole chunks of each sequence
    // (PER_SEQ: addresses and lengths are then scalar work), or the tokens of all sequences in a row
    const int seq_chunks = (a.n_new + 63) >> 6;
    const int n_chunks = PER_SEQ ? a.B * seq_chunks : (a.B * a.n_new + 63) >> 6;
    const int n_jobs = (n_chunks + rounds - 1) / rounds;  // a wavefront takes `rounds` chunks in a row: one codebook set-up
    const int hkv = blockIdx.x / n_jobs;
    const int chunk0 = (blockIdx.x - hkv * n_jobs) * rounds;
    const int chunk1 = chunk0 + rounds < n_chunks ? chunk0 + rounds : n_chunks;

    // ---- codebook of this subspace: A rows for the filter, coordinates for the exact evaluations
    const T *src = (const T *)a.codebook[which] + ((int64_t)hkv * M + i) * 256 * DS;
    T y[4][DS];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < DS; ++j)
            y[r][j] = src[(lane + 64 * r) * DS + j];
    float c_max = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < DS; ++j)
            c_max = fmaxf(c_max, fabsf((float)y[r][j]));
    const float scale = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(pq_filter_scale<T>(pq_filter_wave_max(c_max)))));
    bool cb_bad = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = lane + 64 * r;
        pq_filter_build_row<DS>(y[r], scale, arow + c * ROW, cb_bad);
        if constexpr (sizeof(W) > 2) {
#pragma unroll
            for (int j = 0; j < DS; ++j)
                coord[c * DS + j] = (W)(sizeof(T) == 2 ? (float)y[r][j] * scale : (float)y[r][j]);
        }
    }
    cb_bad = __builtin_amdgcn_ballot_w64(cb_bad) != 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    // ---- the tokens, one chunk ahead of the work.  All in 32 bits: sequences and heads are below 2^24, rows below
    // 2^32 (they fit the memory), a head's code bytes below 2^31.
    const uint32_t n_new = (uint32_t)a.n_new, Hkv = (uint32_t)a.Hkv, stride = (uint32_t)a.head_stride;
    const uint32_t cap = (uint32_t)a.max_context;
    const char *x = (const char *)a.x[which] + i * (DS * (int)sizeof(T));
    struct token {
        T x[DS];
        bool live;
        int n_old;
        uint32_t b, t;  // its sequence and position among the new tokens
    };
    // PER_SEQ: sequence and first token of the next chunk (scalars).  Otherwise this lane's own sequence, position and
    // input row (b Hkv + hkv) n_new + t: 64 tokens on are b_step sequences and t_step positions on, a sequence more
    // where t passes n_new.
    const uint32_t u0 = PER_SEQ ? (uint32_t)chunk0 : (uint32_t)chunk0 * 64u + (uint32_t)lane;
    uint32_t b = u0 / (PER_SEQ ? (uint32_t)seq_chunks : n_new);
    uint32_t t = PER_SEQ ? (u0 - b * (uint32_t)seq_chunks) * 64u : u0 - b * n_new;
    uint32_t row = (b * Hkv + (uint32_t)hkv) * n_new + t;
    const uint32_t b_step = 64u / n_new, t_step = 64u - b_step * n_new;
    const uint32_t row_step = b_step * Hkv * n_new + t_step, row_wrap = (Hkv - 1u) * n_new;
    auto fetch = [&](token &k) {
        const T *xp;
        if constexpr (PER_SEQ) {
            const bool any = b < (uint32_t)a.B;  // past the last chunk: the last sequence's last rows again
            k.b = any ? b : (uint32_t)a.B - 1u;
            const uint32_t first = any ? t : n_new - 1u;
            const uint32_t rest = n_new - first;  // at least 1
            const uint32_t l = (uint32_t)lane < rest ? (uint32_t)lane : rest - 1u;
            k.live = any && (uint32_t)lane < rest;
            k.t = first;
            const char *base = x + (uint64_t)((k.b * Hkv + (uint32_t)hkv) * n_new + first) * (PQ_HEAD_DIM * sizeof(T));
            xp = (const T *)(base + l * (uint32_t)(PQ_HEAD_DIM * sizeof(T)));
            t += 64u;
            if (t >= n_new) {
                t = 0u;
                ++b;
            }
        } else {
            k.live = b < (uint32_t)a.B;
            k.b = k.live ? b : 0u;
            k.t = t;
            xp = (const T *)(x + (uint64_t)(k.live ? row : (uint32_t)hkv * n_new) * (PQ_HEAD_DIM * sizeof(T)));
            b += b_step;
            t += t_step;
            row += row_step;
            if (t >= n_new) {
                t -= n_new;
                row += row_wrap;
                ++b;
            }
        }
#pragma unroll
        for (int j = 0; j < DS; ++j)
            k.x[j] = xp[j];
        k.n_old = a.ctx_len[k.b];
    };
    token next;
    fetch(next);
#pragma unroll 1
    for (int chunk = chunk0; chunk < chunk1; ++chunk) {
        const token k = next;
        fetch(next);  // in flight while this chunk is worked on
        const int code = pq_filter_code<DS, T, W>(arow, sizeof(W) == 2 ? arow : (const unsigned char *)coord, scale, cb_bad, k.x, k.live);
        const uint32_t n_old = (uint32_t)(k.n_old < 0 ? 0 : k.n_old);
        const uint32_t pos = (n_old < cap ? n_old : cap) + k.t + (PER_SEQ ? (uint32_t)lane : 0u);
        if (k.live && pos < cap) {
            const uint32_t off = which == 0 ? pq_k_code_offset(pos, i, M, a.k_skew) : pq_v_code_offset(pos, i, M);
            const uint32_t head = (PER_SEQ ? k.b * Hkv : __umul24(k.b, Hkv)) + (uint32_t)hkv;
            a.codes[which][(uint64_t)head * stride + off] = (uint8_t)code;
        }
    }
}

// ---------------------------------------------------------------------------------
// Long appends at ds = 2: the grid of pq_nearest_grid.h.  A workgroup is 4 neighbouring subspaces of one head (K or V) and a
// slice of the tokens: it builds their 4 grids and then walks the tokens, one 16-byte load (fp16; fp32: two) of a token for
// the 4 subspaces.  The 16 workgroups of the same tokens run on one XCD at about the same time, so a token's row comes from
// memory once.  Chunks are the 64-token blocks of the code layout: a lane's 4 offsets inside a block never change.
template <typename T> struct grid_token {
    T x[GRID_SUB][2];
    bool live;
    int64_t block;  // byte offset of the chunk's block of codes
};

// The grids of registered codebooks are the same in every append, so a context keeps them, once its appends have paid for
// building them (keep_grids), and a workgroup fetches the 80 KiB or so that are used of its four (fp16) instead of
// building for 66 us: 32 heads x 32K tokens 641 -> 392 us, and from some 1000 tokens on appends do better with kept grids than
// through the filter, where before 9000 had to pay for building them (32 heads x 4000 tokens 200 -> 84 us).  An image takes
// 25 KiB per subspace (32 heads, K and V: 105 MB of memory).
// A word per 4 subspaces holds the address of their image if it is that of the codebooks in force.  It is on the device, so that
// stream order and what a captured graph replays decide, not the host: registering codebooks puts it to 0, and a
// workgroup that finds that builds for itself and waits for nobody.  Images are written and read by agent-scope accesses, the
// word behind the image (the exchange of pq_device_utils.h): an append on another stream finds a whole image or none.

// words of a subspace's pool that are used
__device__ __forceinline__ int grid_pool_words(const pq_grid_map &m)
{
    return pq_grid_useless(m) || m.pool_used > GRID_POOL ? GRID_POOL : (int)m.pool_used;  // (useless: the wide coordinates)
}

// image -> grids in LDS, 8 bytes a thread and turn.  Requested together are coordinates, cells and maps and the first 512 words of
// every pool, which is all that most grids use of theirs.  The filter's rows are made anew, a thread each.
template <typename T> __device__ __forceinline__ void grid_fetch(pq_grids<T> &grids, const char *image)
{
    constexpr int THREADS = GRID_WAVES * 64, FRONT = (int)offsetof(pq_grids<T>, pool) / 8, TURNS = (FRONT + THREADS - 1) / THREADS;
    static_assert(THREADS == GRID_SUB * 256 && sizeof(pq_grid_map) % 16 == 0, "256 threads per pool, whole vectors");
    const int j = threadIdx.x >> 8, c = threadIdx.x & 255;
    const float *pool_from = (const float *)(image + offsetof(pq_grids<T>, pool) + j * (GRID_POOL * 4));
    float2 t[TURNS + 1];
#pragma unroll
    for (int k = 0; k < TURNS; ++k) {
        const int at = k * THREADS + (int)threadIdx.x;
        t[k] = fetch((const float *)image + 2 * (at < FRONT ? at : FRONT - 1));
    }
    t[TURNS] = fetch(pool_from + 2 * c);
#pragma unroll
    for (int k = 0; k < TURNS; ++k) {
        const int at = k * THREADS + (int)threadIdx.x;
        if (at < FRONT)
            ((float2 *)&grids)[at] = t[k];
    }
    ((float2 *)grids.pool[j])[c] = t[TURNS];
    __syncthreads();
    bool bad = false;
    const T mine[2] = {grids.coord[j][c][0], grids.coord[j][c][1]};
    const pq_grid_map &m = grids.map[j];
    pq_filter_build_row<2>(mine, m.scale, grids.arow[j] + c * pq_filter_row_bytes<T>(), bad);
    if ((m.again[c >> 5] >> (c & 31)) & 1u)
        pq_filter_hide_row<2, T>(grids.arow[j] + c * pq_filter_row_bytes<T>());
    const int words = grid_pool_words(m);
    for (int at = 256 + c; 2 * at < words; at += 256)
        ((float2 *)grids.pool[j])[at] = fetch(pool_from + 2 * at);
    __syncthreads();
}

// A workgroup: 4 subspaces, as the encode's workgroups, in the order of the images.
template <typename T>
__global__ __launch_bounds__(GRID_WAVES * 64) void pq_grid_image_kernel(const T *codebook_k, const T *codebook_v, const int groups_k, void *images,
                                                                        uint64_t *grid_state, uint64_t *found, const uint32_t generation)
{
    __shared__ __attribute__((aligned(16))) pq_grids<T> grids;
    __shared__ __attribute__((aligned(16))) pq_grid_scratch<false> scratch;
    __shared__ float2 box[GRID_SIDE];

    const int group = blockIdx.x;
    const T *src = group < groups_k ? codebook_k + (int64_t)group * (GRID_SUB * 512) : codebook_v + (int64_t)(group - groups_k) * (GRID_SUB * 512);
    pq_grid_build(grids, scratch.making, box, src);
    char *const image = (char *)images + (int64_t)group * pq_grid_image_bytes<T>();
    const auto write = [&](const int from, const int bytes, const int first, const int step) {
        for (int at = first * 8; at < bytes; at += step * 8) {
            const float2 v = *(const float2 *)((const char *)&grids + from + at);
            publish((float *)(image + from + at), v.x, v.y);
        }
    };
    write(0, (int)offsetof(pq_grids<T>, pool), threadIdx.x, GRID_WAVES * 64);
    const int j = threadIdx.x >> 8;
    write((int)offsetof(pq_grids<T>, pool) + j * (GRID_POOL * 4), 4 * grid_pool_words(grids.map[j]), threadIdx.x & 255, 256);
    publish_wait();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(grid_state + group, (uint64_t)image, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 64 && found != nullptr) {
        pq_grid_price sum = {0, 0};
        for (int k = 0; k < GRID_SUB; ++k) {
            const pq_grid_price price = pq_grid_price_of(grids.map[k]);
            sum.grid += price.grid;
            sum.filter += price.filter;
        }
        __hip_atomic_store(found + group, (uint64_t)generation << 32 | sum.grid << 16 | sum.filter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <typename T, bool WIDE>
__global__ __launch_bounds__(GRID_WAVES * 64) void pq_encode_grid_kernel(const pq_encode_args a, const int seq_chunks, const int slices,
                                                                         const int slice_chunks)
{
    constexpr int M = 64;
    __shared__ __attribute__((aligned(16))) pq_grids<T> grids;
    constexpr bool KEEP = sizeof(T) == 2;
    __shared__ __attribute__((aligned(16))) pq_grid_scratch<KEEP> scratch;
    __shared__ float2 box[GRID_SIDE];
    __shared__ uint64_t there;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // an XCD takes whole units of 16 workgroups, one after the other
    const int local = blockIdx.x >> 3;
    const int unit = (local >> 4) * 8 + (blockIdx.x & 7);
    if (unit >= 2 * a.Hkv * slices)
        return;
    const int i0 = (local & 15) * GRID_SUB;
    const int head = unit / slices, slice = unit - head * slices;
    const int which = head >= a.Hkv, hkv = which ? head - a.Hkv : head;
    const int n_chunks = a.B * seq_chunks;
    const int first = slice * slice_chunks;
    const int last = first + slice_chunks < n_chunks ? first + slice_chunks : n_chunks;

    const int group = head * (M / GRID_SUB) + i0 / GRID_SUB;
    if (threadIdx.x == 0)  // one look for all: the word may change
        there = a.grid_state != nullptr ? __hip_atomic_load(a.grid_state + group, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
    __syncthreads();
    const uint64_t image = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)there) |
                           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(there >> 32)) << 32;
    if (image != 0)
        grid_fetch<T>(grids, (const char *)image);
    else
        pq_grid_build(grids, scratch.making, box, (const T *)a.codebook[which] + ((int64_t)hkv * M + i0) * 512);

    const T *x = (const T *)a.x[which] + i0 * 2;
    uint8_t *codes = a.codes[which];
    const int n_new = a.n_new, cap = a.max_context;
    int in_block[GRID_SUB];
#pragma unroll
    for (int j = 0; j < GRID_SUB; ++j)
        in_block[j] = which == 0 ? (int)pq_k_code_offset((uint32_t)lane, i0 + j, M, a.k_skew) : (int)pq_v_code_offset((uint32_t)lane, i0 + j, M);
    // the next chunk: sequence b, block r of it
    int b = (first + wave) / seq_chunks;
    int r = first + wave - b * seq_chunks;
    auto length = [&](int seq) {
        const int n = a.ctx_len[seq];
        return n < 0 ? 0 : n < cap ? n : cap;
    };
    // (a sequence's length is loaded when its chunks begin, a chunk ahead: in front of every chunk's rows it was waited for,
    // and for the codes on their way to memory with it)
    auto fetch = [&, b, r, n_old = length(b < a.B ? b : a.B - 1)](int, grid_token<T> &k) mutable {
        const bool any = b < a.B;
        const int seq = any ? b : a.B - 1;
        const int t = r * 64 + lane - (n_old & 63);  // position among the new tokens
        const int pos = (n_old & ~63) + r * 64 + lane;
        k.live = any && t >= 0 && t < n_new && pos < cap;
        const int row = t < 0 ? 0 : t < n_new ? t : n_new - 1;
        const T *xp = x + (((int64_t)seq * a.Hkv + hkv) * n_new + row) * PQ_HEAD_DIM;
        typedef T quad __attribute__((ext_vector_type(16 / sizeof(T))));
        quad part[sizeof(T) / 2];
#pragma unroll
        for (int v = 0; v < (int)sizeof(T) / 2; ++v)
            part[v] = ((const quad *)xp)[v];
        __builtin_memcpy(k.x, part, sizeof(k.x));
        k.block = ((int64_t)seq * a.Hkv + hkv) * a.head_stride + (int64_t)((n_old >> 6) + r) * (64 * M);
        r += GRID_WAVES;
        if (r >= seq_chunks && any) {
            do {
                r -= seq_chunks;
                ++b;
            } while (r >= seq_chunks && b < a.B);
            n_old = length(b < a.B ? b : a.B - 1);
        }
    };
    const int n_old_first = length(0);
    auto place = [&](uint32_t id, int &seq, int &t, int &pos) {
        const uint32_t chunk = (uint32_t)first + (id >> 8);
        seq = a.B == 1 ? 0 : (int)(chunk / (uint32_t)seq_chunks);  // (a division is some 25 instructions)
        const int block = (int)(chunk - (uint32_t)seq * (uint32_t)seq_chunks);
        const int n_old = a.B == 1 ? n_old_first : length(seq);  // (no load on the way to a store)
        t = block * 64 + (int)((id >> 2) & 63u) - (n_old & 63);
        pos = n_old + t;
    };
    const auto block_of = [&](const grid_token<T> &k) {
        const uint64_t at = (uint64_t)codes + (uint64_t)k.block;
        const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at) |
                              (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) << 32;
        return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, 64 * M, 0x00020000);
    };
    // WIDE: 4 bytes a store.  Of V, four tokens' codes of a subspace stand together, and a transposition within four lanes
    // makes them so.  Of K, a token's codes of four subspaces do: at a multiple of 4 where the skew goes by quads of lanes, else
    // anywhere, and in 12 of the 64 lanes on both sides of a turn to the lane's next 16 bytes, 1 KiB on: three stores more.
    const bool is_k = which == 0;
    const bool apart = is_k && in_block[3] != in_block[0] + 3;
    const int in_front = in_block[1] != in_block[0] + 1 ? 1 : in_block[2] != in_block[1] + 1 ? 2 : 3;  // of the turn
    const int two_at = !apart ? -1 : in_front == 1 ? in_block[1] : in_block[0];
    const int one_at = !apart ? -1 : in_front == 1 ? in_block[0] : in_block[2];
    const int last_at = !apart ? -1 : in_block[3];
    const uint32_t two_of = apart && in_front == 1 ? 8u : 0u, one_of = apart && in_front == 1 ? 0u : 16u;
    const int four_at = apart ? -1 : is_k ? in_block[0] : (int)pq_v_code_offset((uint32_t)(lane & ~3), i0 + (lane & 3), M);
    const uint32_t turn_1 = (lane & 1) == 0 ? 0x06020400u : 0x03070105u, turn_2 = (lane & 2) == 0 ? 0x05040100u : 0x03020706u;
    const auto scan = [&](auto FOUR) {
        pq_grid_scan<T, KEEP, decltype(FOUR)::value, grid_token<T>>(
            grids, scratch.queue, first, last, fetch,
            [&](const grid_token<T> &k, int j, int code, bool decided) {
                const int off = pq_grid_pick(j, in_block[0], in_block[1], in_block[2], in_block[3]);
                if constexpr (sizeof(T) == 4) {  // (the other way 198 -> 202 us for 9000 tokens of 32 heads)
                    if (decided)
                        codes[k.block + (uint32_t)off] = (uint8_t)code;
                    return;
                }
                // A store for every lane, those beyond the block's bytes dropped: with stores in branches the compiler does not know how
                // many are on their way behind the next chunk's rows, and waits for all of them.
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)code, block_of(k), decided ? off : -1, 0, 0);
            },
            [&](const grid_token<T> &k, uint32_t w) {
                if (decltype(FOUR)::value == 1 && !is_k) {  // lane l of four: the four tokens' codes of subspace l
                    w = __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xf, 0xf, true), w, turn_1);
                    w = __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xf, 0xf, true), w, turn_2);
                }
                __builtin_amdgcn_raw_buffer_store_b32(w, block_of(k), four_at, 0, 0);
                if constexpr (decltype(FOUR)::value == 4) {
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(w >> two_of), block_of(k), two_at, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(w >> one_of), block_of(k), one_at, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(w >> 24), block_of(k), last_at, 0, 0);
                }
            },
            [&](uint32_t id, T &x0, T &x1) {
                int seq, t, pos;
                place(id, seq, t, pos);
                const T *xp = x + (((int64_t)seq * a.Hkv + hkv) * n_new + t) * PQ_HEAD_DIM + (id & 3u) * 2;
                x0 = xp[0];
                x1 = xp[1];
            },
            [&](uint32_t id, T, T, int code) {
                int seq, t, pos;
                place(id, seq, t, pos);
                const int i = i0 + (int)(id & 3u);
                const uint32_t off = which == 0 ? pq_k_code_offset((uint32_t)pos, i, M, a.k_skew) : pq_v_code_offset((uint32_t)pos, i, M);
                codes[((int64_t)seq * a.Hkv + hkv) * a.head_stride + off] = (uint8_t)code;
            });
    };
    if (!WIDE || pq_grid_useless_of(grids) != 0)
        scan(std::integral_constant<int, 0>());
    else if constexpr (WIDE) {
        if (is_k && a.k_skew == PQ_K_SKEW_LANE)
            scan(std::integral_constant<int, 4>());
        else
            scan(std::integral_constant<int, 1>());
    }
}

// ---------------------------------------------------------------------------------
// A handful of tokens per KV head (one decoding step of a small batch): lane = four CENTROIDS.  With one token per
// lane a wavefront would walk 256 centroids for a few live lanes; here every lane holds 4 neighbouring centroids in
// registers and the wavefront takes one token after the other, its sub-vector in scalar registers.
// The fp32 distances name the candidates: their relative error is at most 6 x 2^-24 (ds = 4: a difference twice, a product,
// three sums), so the nearest centroid's is within 12 x 2^-24 of the least, and all within 16 steps of the least
// distance's bits — at least 2^-20 of it — are kept.  One candidate, nearly always: it is the code, and naming it is scalar
// work.  Several (ties, near-ties), none, fp32 squares below 2^-100, which are not that good, or no finite one (an infinite token
// may have a single distance that is not NaN, and it is no less than infinity): the defining fp64 distances
// of all 256, ascending, and the lexicographic minimum of (distance, index), the lowest index among equal distances.
// 30 vector instructions per token and subspace at ds = 2 where the fp64 distances and their minimum over the wavefront
// took 80.
constexpr int FEW_WAVES = 4;  // neighbouring subspaces of a workgroup: they share the lines of the tokens

__device__ __forceinline__ uint32_t few_wave_min(uint32_t x)
{
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, true));   // quad_perm [2,3,0,1]
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, true));  // row_half_mirror
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xf, 0xf, true));  // row_mirror
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return min(min(r0, r1), min(r2, r3));
}

// per_wave: tokens of a wavefront, at most 64; by_n_new: pq_divisor(n_new)
template <int M, int DS, typename T>
__global__ __launch_bounds__(FEW_WAVES * 64) void pq_encode_few_kernel(const pq_encode_args a, const int per_wave, const uint32_t by_n_new)
{
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int which = blockIdx.z & 1;
    const int i = blockIdx.y * FEW_WAVES + wave;
    const int hkv = blockIdx.x;
    const int first = (int)(blockIdx.z >> 1) * per_wave, left = a.B * a.n_new - first;
    const int n_tok = left < per_wave ? left : per_wave;

    // lane u < n_tok fetches token first + u: its sub-vector, sequence and position
    const uint32_t u_mine = (uint32_t)(first + (lane < n_tok ? lane : 0));
    const int b_mine = (int)divided(u_mine, by_n_new);
    const int t_mine = (int)u_mine - b_mine * a.n_new;
    const T *xp = (const T *)a.x[which] + (((int64_t)b_mine * a.Hkv + hkv) * a.n_new + t_mine) * PQ_HEAD_DIM + i * DS;
    float x_mine[DS];
#pragma unroll
    for (int j = 0; j < DS; ++j)
        x_mine[j] = (float)xp[j];
    const int n_old = a.ctx_len[b_mine];

    // centroids 4 lane .. 4 lane + 3
    typedef T quad __attribute__((ext_vector_type(4 * DS)));
    const quad cq = *((const quad *)((const T *)a.codebook[which] + ((int64_t)hkv * M + i) * 256 * DS) + lane);
    float c[4][DS];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < DS; ++j)
            c[r][j] = (float)cq[r * DS + j];

    int code_mine = 0;
    for (int u = 0; u < n_tok; ++u) {
        float x[DS];
#pragma unroll
        for (int j = 0; j < DS; ++j)
            x[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x_mine[j]), u));
        uint32_t d[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float dist = 0.f;
#pragma unroll
            for (int j = 0; j < DS; ++j) {
                const float diff = x[j] - c[r][j];
                dist = j == 0 ? diff * diff : __builtin_fmaf(diff, diff, dist);
            }
            d[r] = __float_as_uint(dist);  // (positive floats order like their bits)
        }
        uint32_t least = few_wave_min(min(min(min(d[0], d[1]), d[2]), d[3]));
        if constexpr (sizeof(T) == 2)  // (no distance of finite fp16 numbers comes near this: none is within 16 steps of it)
            least = min(least, 0x7f000000u);
        uint64_t near[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            near[r] = __builtin_amdgcn_ballot_w64(d[r] <= least + 16u);
        const int n_near = __builtin_popcountll(near[0]) + __builtin_popcountll(near[1]) + __builtin_popcountll(near[2]) +
                           __builtin_popcountll(near[3]);
        int code = 4 * __builtin_ctzll(near[0] | near[1] | near[2] | near[3] | 1ull << 63) +
                   (near[1] != 0 ? 1 : near[2] != 0 ? 2 : near[3] != 0 ? 3 : 0);
        if (n_near != 1 || (sizeof(T) == 4 && least - 0x0d800000u >= 0x7f800000u - 0x0d800000u)) {  // wave-uniform, rare
            double bd = __builtin_huge_val();
            int bc = 4 * lane;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double dist = 0.0;
#pragma unroll
                for (int j = 0; j < DS; ++j) {
                    const double diff = (double)x[j] - (double)c[r][j];
                    dist = __builtin_fma(diff, diff, dist);
                }
                bc = dist < bd ? 4 * lane + r : bc;  // ascending index inside the lane, strict "<"
                bd = __builtin_fmin(bd, dist);
            }
            wave_argmin(bd, bc);
            code = __builtin_amdgcn_readfirstlane(bc);
        }
        code_mine = lane == u ? code : code_mine;
    }
    const int64_t pos = (int64_t)(n_old < 0 ? 0 : n_old) + t_mine;
    if (lane < n_tok && pos < a.max_context) {
        uint8_t *dst = a.codes[which] + ((int64_t)b_mine * a.Hkv + hkv) * a.head_stride;
        const int64_t off = which == 0 ? pq_k_code_offset(pos, i, M, a.k_skew) : pq_v_code_offset(pos, i, M);
        dst[off] = (uint8_t)code_mine;
    }
}

__global__ void pq_bump_len_kernel(int32_t *ctx_len, int B, int n_new, int max_context, unsigned int *dev_err)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B)
        return;
    int n = ctx_len[b];
    n = n < 0 ? 0 : n;
    int64_t m = (int64_t)n + n_new;
    if (m > max_context) {
        m = max_context;
        atomicOr(dev_err, PQ_ERRFLAG_APPEND_OVERFLOW);
    }
    ctx_len[b] = (int32_t)m;
}

}  // namespace

hipError_t pq_launch_bump_len(int32_t *ctx_len, int B, int n_new, int max_context, unsigned int *dev_err, hipStream_t s)
{
    hipLaunchKernelGGL(pq_bump_len_kernel, dim3((B + 255) / 256), dim3(256), 0, s, ctx_len, B, n_new, max_context, dev_err);
    return hipGetLastError();
}

// How many of a head's chunks a wavefront takes in a row; rows: subspaces of all heads, keys and values.  Up to 32, so that
// there are 8192 wavefronts or more, and all about the same number (63 chunks of 32 heads as 31 + 31 + 1: 222 us, as 3 x 21: 198).
// Up to 16384 chunks in all go to about 4096 wavefronts, since setting up a codebook costs about a chunk (2 x 96 tokens x 32
// heads, fp32, M = 64: 23.7 -> 21.3 us; 8 x 16 tokens, fp16: 16.0 -> 14.8), if these get nearly equal shares: workgroups go to the
// XCDs in turn, and where the last of 2 or 4 per head is short, it is short on the same XCDs every time (192 tokens x 32 heads, M =
// 32, fp32: 18.6 us as 2 + 1 chunks, 16.6 as three; 448 tokens as 4 + 3 26.6, as seven 30.1).  Far fewer than 4096 are too few
// (576 tokens x 8 heads, M = 32, fp16: 13.9 us as 4 x 2 + 1, 13.1 as nine).
inline int64_t pq_encode_rounds(int64_t n_chunks, int64_t rows)
{
    const int64_t waves = rows * n_chunks;
    int64_t rounds = waves <= 16384 ? (waves + 4095) / 4096 : waves / 8192 > 32 ? 32 : waves / 8192;
    int64_t jobs = (n_chunks + rounds - 1) / rounds;
    while (waves <= 16384 && rounds > 1 && ((jobs * rounds - n_chunks) * 7 > n_chunks || rows * jobs < 3072)) {
        --rounds;
        jobs = (n_chunks + rounds - 1) / rounds;
    }
    return (n_chunks + jobs - 1) / jobs;
}

template <int M, int DS, typename T>
void launch_fast(const pq_encode_args &a, hipStream_t s)
{
    // whole 64-token chunks of each sequence unless that leaves more than an eighth of the lanes without a token
    const int64_t seq_chunks = ((int64_t)a.n_new + 63) / 64;
    const bool per_seq = seq_chunks * 512 <= (int64_t)a.n_new * 9 || a.B == 1;
    const int64_t n_chunks = per_seq ? a.B * seq_chunks : ((int64_t)a.B * a.n_new + 63) / 64;
    const int64_t rounds = pq_encode_rounds(n_chunks, (int64_t)a.Hkv * M * 2);
    dim3 grid((unsigned)(a.Hkv * ((n_chunks + rounds - 1) / rounds)), M / FAST_WAVES, 2);
    if (per_seq)
        hipLaunchKernelGGL((pq_encode_fast_kernel<M, DS, T, true>), grid, dim3(64 * FAST_WAVES), 0, s, a, (int)rounds);
    else
        hipLaunchKernelGGL((pq_encode_fast_kernel<M, DS, T, false>), grid, dim3(64 * FAST_WAVES), 0, s, a, (int)rounds);
}

// Tokens of a wavefront of the few-token kernel, from a head's tokens and the subspaces of all heads, keys and values; 0: the
// filter does better.  The few-token kernel takes some 2.5 us and 0.11 us for every 1024 (token, subspace) pairs, the filter 5
// to 8 us for any of these sizes, more for more subspaces, whose codebooks it sets up (whole calls with the length reset,
// us, few-token kernel / filter, fp16: M = 64, 32 heads, 8 tokens 8.5 / 11.2, 12 9.7 / 11.2, 16 10.7 / 11.3, 24 13.0 / 11.3; 8
// heads, 8 tokens 6.3 / 8.3, 24 7.7 / 8.2, 32 8.3 / 8.3, 64 10.6 / 8.7; 4 heads, 45 tokens 8.5 / 9.2, 128 11.2 / 8.8; M = 32, 32
// heads, 12 tokens 8.6 / 9.6, 16 9.3 / 9.5, 24 11.4 / 9.4; 8 heads, 32 tokens 7.9 / 8.5, 64 9.7 / 8.7; fp32, where the filter
// has twice the terms: M = 64, 32 heads, 16 tokens 10.4 / 13.1, 24 13.0 / 13.1).
// Some 6000 wavefronts are the best division: 8192 cost 0.1 .. 1 us more, and what a wavefront takes in a row shows from a
// dozen tokens on (8 heads, M = 64, 16 tokens: 1 each 8.1 us, 3 6.9, 8 7.3, 16 8.6).
inline int pq_encode_few_per_wave(int64_t tokens, int64_t rows, int M)
{
    const int64_t pairs = tokens * rows;
    if (pairs > (M == 64 ? 24576 : 16384) + 8 * rows)
        return 0;
    const int64_t per_wave = (pairs + 6143) / 6144, most = per_wave < 64 ? per_wave : 64;
    const int64_t groups = (tokens + most - 1) / most;
    return (int)((tokens + groups - 1) / groups);
}

template <int M, int DS, typename T> void launch_few(const pq_encode_args &a, int per_wave, hipStream_t s)
{
    const int groups = (a.B * a.n_new + per_wave - 1) / per_wave;
    hipLaunchKernelGGL((pq_encode_few_kernel<M, DS, T>), dim3(a.Hkv, M / FEW_WAVES, 2 * groups), dim3(64 * FEW_WAVES), 0, s, a, per_wave,
                       pq_divisor(a.n_new));
}

// Whether a grid workgroup stores the codes of a chunk together, from its chunks of 64 tokens and the number of workgroups: it
// needs a second copy of the loop over the tokens, fetching that costs 1 us, and what is gained shows where the stores of
// several rounds of workgroups queue.  us, single / wide codes: 32 heads x 32K 392 / 366 (normal data), 477 / 458 (Laplace's), 436 /
// 426 (channel scales), over 128 query heads 386 / 350; 16 heads x 33 000 201 / 189, x 20 000 121 / 119; 32 x 9000 135.7 / 134.9 and
// 146.1 / 147.3 (scales), 8 x 32 x 1100, many chunks not full, 143.0 / 145.5; 8 heads, a workgroup per compute unit, 30 000
// tokens 87.7 / 88.1.
inline bool pq_grid_stores_wide(int64_t slice_chunks, int64_t n_new, int64_t workgroups, int n_cu)
{
    return slice_chunks >= 256 && n_new >= 2048 && workgroups >= 2 * (int64_t)n_cu;
}

template <typename T> void launch_grid(const pq_encode_args &a, int seq_chunks, int slices, int n_cu, hipStream_t s)
{
    const int n_chunks = a.B * seq_chunks;
    const int slice_chunks = (n_chunks + slices - 1) / slices;
    const int units = 2 * a.Hkv * slices;
    const dim3 grid((unsigned)((units + 7) / 8 * 128));
    // (fp32: no registers for it)
    if (sizeof(T) == 2 && pq_grid_stores_wide(slice_chunks, a.n_new, (int64_t)units * 16, n_cu))
        hipLaunchKernelGGL((pq_encode_grid_kernel<T, sizeof(T) == 2>), grid, dim3(64 * GRID_WAVES), 0, s, a, seq_chunks, slices, slice_chunks);
    else
        hipLaunchKernelGGL((pq_encode_grid_kernel<T, false>), grid, dim3(64 * GRID_WAVES), 0, s, a, seq_chunks, slices, slice_chunks);
}

// Builds the grids into the context's images when the appends before this one since the codebooks were registered, chunks of 64
// tokens per head, would together have paid for it: the second of two long ones, so that the first takes no longer than by
// building its own (32 heads x 32K tokens 692 us with the images against 672, 9000 tokens 439 against 410), and a context that
// never appends much, or a prompt once, never builds any.  (What is counted decides about time alone: threads that append at
// once may count less, one of them builds.)  Not while a graph is recorded, which would build again with every replay, and not
// for codebooks that were handed to a call, which may be handed to the next one again, nor in a context with a recorded
// registration: every replay of it takes the images away, and appends that count on them then build for themselves, in all four
// rounds of workgroups (32 heads x 2000 tokens 307 us, 123 through the filter).  The first to build allocates (105 MB for
// 32 heads, 35 to 90 us): at creation every context with room for a long append had them, three times the codes of 4096 tokens.
// Without the memory appends go on building for themselves.
static hipError_t keep_grids(pq_attn_ctx *ctx, int64_t filter_chunks, int64_t groups, hipStream_t s)
{
    if (ctx->grid_phase.load(std::memory_order_relaxed) != GRIDS_NONE || ctx->grid_chunks.load(std::memory_order_relaxed) < 0)
        return hipSuccess;
    hipStreamCaptureStatus recording = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(s, &recording) != hipSuccess)
        (void)hipGetLastError();
    if (recording != hipStreamCaptureStatusNone)
        return hipSuccess;
    const int64_t before = ctx->grid_chunks.fetch_add(filter_chunks, std::memory_order_relaxed);
    int none = GRIDS_NONE;
    if (pq_grid_slices(before, before, groups, ctx->n_cu) == 0 || !ctx->grid_phase.compare_exchange_strong(none, GRIDS_CLAIMED))
        return hipSuccess;
    if (ctx->grids == nullptr) {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;  // (another stream may be recording; it is none of its business)
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        const bool ok = hipMalloc(&ctx->grids, (size_t)ctx->grid_bytes) == hipSuccess;
        if (ok && hipHostMalloc((void **)&ctx->grid_found, (size_t)groups * sizeof(uint64_t), 0) == hipSuccess)
            memset(ctx->grid_found, 0, (size_t)groups * sizeof(uint64_t));
        else
            ctx->grid_found = nullptr;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (ctx->grid_found == nullptr)
            (void)hipGetLastError();
        if (!ok) {
            ctx->grids = nullptr;
            ctx->grid_chunks = -1;
            ctx->grid_phase = GRIDS_NONE;
            return hipSuccess;
        }
    }
    const uint32_t generation = ctx->grid_generation.load(std::memory_order_relaxed);
    if (ctx->cfg.dtype == PQ_F16)
        hipLaunchKernelGGL(pq_grid_image_kernel<_Float16>, dim3((unsigned)groups), dim3(GRID_WAVES * 64), 0, s, (const _Float16 *)ctx->kcb_natural,
                           (const _Float16 *)ctx->vcb_natural, (int)groups / 2, ctx->grids, ctx->grid_state, ctx->grid_found, generation);
    else
        hipLaunchKernelGGL(pq_grid_image_kernel<float>, dim3((unsigned)groups), dim3(GRID_WAVES * 64), 0, s, (const float *)ctx->kcb_natural,
                           (const float *)ctx->vcb_natural, (int)groups / 2, ctx->grids, ctx->grid_state, ctx->grid_found, generation);
    const hipError_t e = hipGetLastError();
    ctx->grid_phase = e == hipSuccess ? GRIDS_KEPT : GRIDS_NONE;
    return e;
}

// What a chunk costs with the codebooks in force: the rule's own figures until every image's workgroup has said what it found.  Waits
// for nothing; the appends until then go by codebooks that the grids serve.
static pq_grid_price grid_price(pq_attn_ctx *ctx, int64_t groups)
{
    const uint32_t generation = ctx->grid_generation.load(std::memory_order_relaxed);
    const uint64_t known = ctx->grid_cost.load(std::memory_order_relaxed);
    if ((uint32_t)(known >> 32) == generation)
        return {(uint32_t)known >> 16, (uint32_t)known & 0xffffu};
    uint64_t grid = 0, filter = 0;
    for (int64_t k = 0; k < groups; ++k) {
        const uint64_t found = ctx->grid_found != nullptr ? __atomic_load_n(ctx->grid_found + k, __ATOMIC_RELAXED) : 0u;
        if ((uint32_t)(found >> 32) != generation || (uint32_t)found == 0)
            return {18, 72};
        grid += found >> 16 & 0xffffu;
        filter += found & 0xffffu;
    }
    const uint64_t n = (uint64_t)groups * GRID_SUB;
    const pq_grid_price mean = {(uint32_t)((grid + n / 2) / n), (uint32_t)((filter + n / 2) / n)};
    ctx->grid_cost.store((uint64_t)generation << 32 | mean.grid << 16 | mean.filter, std::memory_order_relaxed);
    return mean;
}

hipError_t pq_launch_encode(pq_attn_ctx *ctx, const pq_encode_args &a, int32_t *ctx_len, unsigned int *dev_err,
                            hipStream_t s)
{
    const bool f16 = ctx->cfg.dtype == PQ_F16;
    const int few = pq_encode_few_per_wave((int64_t)a.B * a.n_new, (int64_t)a.Hkv * ctx->cfg.n_subspaces * 2, ctx->cfg.n_subspaces);
    if (few > 0) {
        if (ctx->cfg.n_subspaces == 64) {
            if (f16) launch_few<64, 2, _Float16>(a, few, s); else launch_few<64, 2, float>(a, few, s);
        } else {
            if (f16) launch_few<32, 4, _Float16>(a, few, s); else launch_few<32, 4, float>(a, few, s);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        return pq_launch_bump_len(ctx_len, a.B, a.n_new, a.max_context, dev_err, s);
    }
    const int seq_chunks = (int)(((int64_t)a.n_new + 126) >> 6);  // blocks of 64 positions that n_new tokens can touch
    // its 16-byte loads ask for rows that start at such an address
    const bool grid_can = ctx->cfg.n_subspaces == 64 && (((uintptr_t)a.x[0] | (uintptr_t)a.x[1]) & 15) == 0 &&
                          (int64_t)a.B * seq_chunks < (1 << 30);
    const int64_t chunks = (int64_t)a.B * seq_chunks, filter_chunks = ((int64_t)a.B * a.n_new + 63) / 64, groups = (int64_t)2 * a.Hkv * 16;
    int slices = grid_can ? pq_grid_slices(chunks, filter_chunks, groups, ctx->n_cu) : 0;
    const int with_kept = grid_can && ctx->grid_state != nullptr ? pq_grid_slices(chunks, filter_chunks, groups, ctx->n_cu, true) : 0;
    if (with_kept > 0) {
        const hipError_t e = keep_grids(ctx, filter_chunks, groups, s);
        if (e != hipSuccess)
            return e;
        if (ctx->grid_phase.load(std::memory_order_acquire) == GRIDS_KEPT)
            slices = pq_grid_slices(chunks, filter_chunks, groups, ctx->n_cu, true, grid_price(ctx, groups));
    }
    if (slices > 0) {
        if (f16) launch_grid<_Float16>(a, seq_chunks, slices, ctx->n_cu, s); else launch_grid<float>(a, seq_chunks, slices, ctx->n_cu, s);
    } else if (ctx->cfg.n_subspaces == 64) {
        if (f16) launch_fast<64, 2, _Float16>(a, s); else launch_fast<64, 2, float>(a, s);
    } else {
        if (f16) launch_fast<32, 4, _Float16>(a, s); else launch_fast<32, 4, float>(a, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    // lengths move only after every encode workgroup has read the old ones (stream order)
    return pq_launch_bump_len(ctx_len, a.B, a.n_new, a.max_context, dev_err, s);
}

int64_t pq_grid_groups(const pq_attn_config *cfg) { return (int64_t)2 * cfg->n_kv_heads * (cfg->n_subspaces / GRID_SUB); }

int64_t pq_grid_images_bytes(const pq_attn_config *cfg, int n_cu)
{
    // (sequences below 1024 tokens are never appended to by thousands)
    if (pq_config_is_12bit(cfg) || cfg->n_subspaces != 64 || cfg->max_context < 1024)
        return 0;
    // the longest append that fits: the launcher's rule for it (which has no upper end that the capacities reach)
    const int64_t seq_chunks = ((int64_t)cfg->max_context + 126) >> 6;
    const int64_t chunks = ((int64_t)cfg->batch * cfg->max_context + 63) / 64;
    if (pq_grid_slices(cfg->batch * seq_chunks, chunks, pq_grid_groups(cfg), n_cu, true) == 0)
        return 0;
    return pq_grid_groups(cfg) * (cfg->dtype == PQ_F16 ? pq_grid_image_bytes<_Float16>() : pq_grid_image_bytes<float>());
}
