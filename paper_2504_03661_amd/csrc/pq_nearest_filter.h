// Nearest centroid of fp16 or fp32 sub-vectors among 256 centroids of the same type: matrix-core filter + fp64
// decision.  Shared by the encode kernel and the k-means assignment; the argument, the error bound and the fall-back
// are described in pq_encode.hip.  Everything here works on ONE wavefront (a 64-token sub-chunk at a time, lane =
// token) and on LDS arrays the caller owns: the A rows of the 256 centroids (pq_filter_row_bytes each) and, where the
// coordinates are not read from the rows, a copy of them.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pq_filter_constants.h"

namespace {

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16e __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2e __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4e __attribute__((ext_vector_type(4)));

// An A row holds the inner indices of one matrix instruction: lanes 0..31 of the wavefront read its first half, lanes
// 32..63 its second.  h + l = |c|^2 / 2, o_0 + 2^15 o_1 = the token's offset.
//   fp16 (v_mfma_f32_32x32x8_f16, 16 bytes), the values of a codebook of small numbers multiplied by a gain: c and
//   |c|^2 / 2 are, which is exact, and so is the offset; x need not be
//     ds = 2   c_0 c_1 h l | 1 2^15 0 0        against the column   -x_0 -x_1 1 1 | o_0 o_1 0 0
//     ds = 4   c_0 c_1 c_2 c_3 | h l 1 2^15    against              -x_0 .. -x_3 | 1 1 o_0 o_1
//   fp32 (v_mfma_f32_32x32x16_f16, 32 bytes), coordinates scaled by a power of two per codebook and split into two
//   fp16, c = c' + c'', x = x' + x''
//     ds = 2   c'_0 c'_1 c''_0 c''_1 c'_0 c'_1 h l | 1 2^15 0 0 0 0 0 0
//                                    against -x'_0 -x'_1 -x'_0 -x'_1 -x''_0 -x''_1 1 1 | o_0 o_1 0 0 0 0 0 0
//     ds = 4   c'_0 .. c'_3 c''_0 .. c''_3 | c'_0 .. c'_3 h l 1 2^15
//                                    against -x'_0 .. -x'_3 -x'_0 .. -x'_3 | -x''_0 .. -x''_3 1 1 o_0 o_1
template <typename T> constexpr int pq_filter_row_bytes() { return sizeof(T) == 2 ? 16 : 32; }

// What a codebook's values are scaled by, from its largest coordinate.
// fp32: the power of two s that brings it into [32, 64); coordinates of centroids and tokens are multiplied by s.
// fp16: with s the power of two that brings it into [2, 4), the gain s^2 of the values, and 1 for larger coordinates.
// Without it the absolute part of tau, there for the roundings of the smallest numbers, is what decides for small ones: at
// a standard deviation of 0.01 every second token marked a second quad, at 0.001 all quads near it (8192 tokens x 32 heads
// 394 us at 1, 804 and 3443 us there; 392 with the gain).  c s^2 stays below 2^15 for the smallest s allowed.
template <typename T> __device__ inline float pq_filter_scale(float c_max)
{
    int e = 0;
    (void)__builtin_frexpf(c_max, &e);
    if constexpr (sizeof(T) == 4) {
        e = e < -100 ? -100 : e;  // (a codebook this small is one cluster of near-ties to the filter)
        return c_max > 0.f ? __builtin_ldexpf(1.0f, 6 - e) : 1.0f;
    } else {
        e = e < -11 ? -11 : e;
        return c_max > 0.f && c_max < 2.0f ? __builtin_ldexpf(1.0f, 4 - 2 * e) : 1.0f;  // (not infinite)
    }
}

// the largest over the wavefront
__device__ inline float pq_filter_wave_max(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        x = fmaxf(x, __shfl_xor(x, o));
    return x;
}

// A row of a centroid (c: its ds coordinates; scale: pq_filter_scale); sets `bad` when |c|^2 / 2 does not split into two fp16
template <int DS, typename T>
__device__ inline void pq_filter_build_row(const T (&c)[DS], const float scale, unsigned char *arow_c, bool &bad)
{
    constexpr int SLOTS = pq_filter_row_bytes<T>() / 2;
    float n = 0.f;
    _Float16 row[SLOTS] = {};
    constexpr int N_AT = sizeof(T) == 2 ? DS : 3 * DS;  // h, l, 1, 2^15 stand behind the coordinates
#pragma unroll
    for (int j = 0; j < DS; ++j) {
        const float f = sizeof(T) == 2 ? (float)c[j] : (float)c[j] * scale;
        n += f * f;  // (the roundings are covered by the bound)
        row[j] = (_Float16)(sizeof(T) == 2 ? f * scale : f);
        if constexpr (sizeof(T) == 4) {
            row[DS + j] = (_Float16)(f - (float)row[j]);
            row[2 * DS + j] = row[j];
        }
    }
    const float h = (sizeof(T) == 2 ? 0.5f * scale : 0.5f) * n;
    const _Float16 hh = (_Float16)h;
    const _Float16 hl = (_Float16)(h - (float)hh);
    row[N_AT] = hh;
    row[N_AT + 1] = hl;
    row[N_AT + 2] = (_Float16)1.f;
    row[N_AT + 3] = (_Float16)32768.f;
    bad |= !(h < 60000.f);
    __builtin_memcpy(arow_c, row, pq_filter_row_bytes<T>());
}

// Takes a centroid out: all its values are infinite, so it is never marked.  For one that repeats an earlier centroid.
template <int DS, typename T> __device__ __forceinline__ void pq_filter_hide_row(unsigned char *arow_c)
{
    constexpr int N_AT = sizeof(T) == 2 ? DS : 3 * DS;  // (h, as above)
    ((_Float16 *)arow_c)[N_AT] = (_Float16)__builtin_inff();
}

// What the matrix instruction and the refinement need of this lane's token
template <int DS, typename T> struct pq_filter_token {
    static constexpr bool F16 = sizeof(T) == 2;
    static constexpr float TAU_NEAR = F16 ? PQ_FILTER_TAU_NEAR : PQ_FILTER_TAU_NEAR_F32;
    typedef typename std::conditional<F16, f16x4, f16x8>::type operand;
    operand col[2];  // the columns of tokens 0..31 and 32..63 of the wavefront
    float x[DS];  // (widened where it is used; fp16: times the gain, as the rows)
    float tau_x;  // the token's share of tau
    bool bad;     // outside the range that the bound covers

    // xin: the token's sub-vector, unscaled
    __device__ __forceinline__ void set(const T (&xin)[DS], const float scale)
    {
#pragma clang fp contract(off)
        float x2 = 0.f, xs[DS];
#pragma unroll
        for (int j = 0; j < DS; ++j) {
            x[j] = F16 ? __builtin_fmaf((float)xin[j], scale, 0.f) : (float)xin[j];  // (fp16: one instruction, exact)
            xs[j] = F16 ? x[j] : x[j] * scale;
            x2 = __builtin_fmaf(xs[j], xs[j], x2);
        }
        // fp16: x2 has the gain twice; 1 / scale of a power of two
        const float x2_to_value = F16 ? __int_as_float(0x7f000000 - __float_as_int(scale)) : 1.f;
        // off: |x|^2/2 with half a per cent on top and a floor, so that every computed value stays above zero, rounded
        // UP to o_0 + 2^15 o_1 (one of the two is zero) by 0.3 % against the half step (2^-11) of the conversion and a
        // subnormal step
        const float off = __builtin_fmaf(PQ_FILTER_X2_FACTOR * x2_to_value, x2, 3.0f * PQ_FILTER_TAU_ABS);
        const float up = __builtin_fmaf(off, 1.003f, 6.0e-8f);
        tau_x = __builtin_fmaf(TAU_NEAR * x2_to_value, x2, PQ_FILTER_TAU_ABS);
        bad = false;
        _Float16 o0 = (_Float16)up, o1 = (_Float16)0.f;
        if (__builtin_amdgcn_ballot_w64(!(off < 60000.f)) != 0) {  // wave-uniform, rare: scaled length beyond 340
            const bool large = !(off < 60000.f);
            o0 = large ? (_Float16)0.f : o0;
            o1 = large ? (_Float16)(up * (1.0f / 32768.f)) : (_Float16)0.f;
            bad = !(off < 2.0e9f);
        }
        const _Float16 one = (_Float16)1.f, zero = (_Float16)0.f;
        operand lo, hi;
        if constexpr (F16 && DS == 2) {
            lo = f16x4{-xin[0], -xin[1], one, one};
            hi = f16x4{o0, o1, zero, zero};
        } else if constexpr (F16) {
            lo = f16x4{-xin[0], -xin[1], -xin[DS - 2], -xin[DS - 1]};
            hi = f16x4{one, one, o0, o1};
        } else {
            _Float16 p[DS], r[DS];
#pragma unroll
            for (int j = 0; j < DS; ++j) {
                p[j] = (_Float16)(-xs[j]);
                r[j] = (_Float16)(-xs[j] - (float)p[j]);
            }
            if constexpr (DS == 2) {
                lo = f16x8{p[0], p[1], p[0], p[1], r[0], r[1], one, one};
                hi = f16x8{o0, o1, zero, zero, zero, zero, zero, zero};
            } else {
                lo = f16x8{p[0], p[1], p[DS - 2], p[DS - 1], p[0], p[1], p[DS - 2], p[DS - 1]};
                hi = f16x8{r[0], r[1], r[DS - 2], r[DS - 1], one, one, o0, o1};
            }
        }
        // lane = token holds both halves of its own column; the instruction wants the upper half of column t in
        // lane t + 32: one exchange of the lane halves gives the operands of both token tiles
        constexpr int WORDS = (int)sizeof(operand) / 4;
        typedef typename std::conditional<F16, u32x2e, u32x4e>::type words;
        const words l = __builtin_bit_cast(words, lo), h = __builtin_bit_cast(words, hi);
        words b0, b1;
#pragma unroll
        for (int k = 0; k < WORDS; ++k) {
            const auto s = __builtin_amdgcn_permlane32_swap(l[k], h[k], false, false);
            b0[k] = s[0];
            b1[k] = s[1];
        }
        col[0] = __builtin_bit_cast(operand, b0);
        col[1] = __builtin_bit_cast(operand, b1);
    }

    // 32 computed values of each of 32 tokens: lane l ends with those of token l mod 32 of the tile whose centroids lie
    // in its half: rows 8 g + 4 (l / 32) + 0..3 of A in registers 4 g .. 4 g + 3 ("quad" g)
    __device__ __forceinline__ f32x16e values(const operand &A, const int tile) const
    {
        const f32x16e none = {};
        if constexpr (F16)
            return __builtin_amdgcn_mfma_f32_32x32x8f16(A, col[tile], none, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(A, col[tile], none, 0, 0, 0);
    }

    // The smallest value of this lane's token from the smallest of either tile in this lane; and what every value
    // within tau of it does not exceed, for both tiles.  (Positive floats order like their bit patterns.)
    __device__ inline int best_of(const int b0, const int b1) const
    {
        const auto s = __builtin_amdgcn_permlane32_swap(b0, b1, false, false);
        return min((int)s[0], (int)s[1]);
    }
    __device__ __forceinline__ void limits(const int best_bits, int (&limit)[2])
    {
        const float best = __int_as_float(best_bits);
        bad |= !(best > 0.f && best < 1.0e30f);  // the offset did not keep the values positive and finite
        // best + tau, tau = TAU_NEAR (|x|^2 + best) + TAU_ABS
        const int lim = __float_as_int(__builtin_fmaf(best, 1.0f + TAU_NEAR, tau_x));
        const auto r = __builtin_amdgcn_permlane32_swap(lim, lim, false, false);
        limit[0] = (int)r[0];
        limit[1] = (int)r[1];
    }
};

// Which minima of a token lie within tau of its best value, as masks over the 64 tokens in scalar registers.  Per tile,
// NR row minima and NC column minima of a grid of value groups stand in every lane; a group can hold such a value only
// if both its row and its column are marked.  One comparison per minimum leaves a mask over the lanes (bits 0..31: the
// tile's tokens against the centroids of lane half 0, bits 32..63: half 1); what follows per mark is scalar work beside
// the other wavefronts' vector instructions: the bits of the marked indices (right where one is marked) and which tokens
// have a second mark.
template <int NR, int NC> struct pq_filter_marks {
    static constexpr int RB = __builtin_ctz(NR), CB = __builtin_ctz(NC);
    uint64_t bit_r[RB], bit_c[CB];             // bit k of the marked row / column
    uint64_t some = 0, in_half1 = 0, several = 0;  // any mark; in lane half 1; more than one group possible

    __device__ inline pq_filter_marks()
    {
#pragma unroll
        for (int k = 0; k < RB; ++k)
            bit_r[k] = 0;
#pragma unroll
        for (int k = 0; k < CB; ++k)
            bit_c[k] = 0;
    }
    __device__ __forceinline__ void add(const int t, const int (&by_r)[NR], const int (&by_c)[NC], const int limit)
    {
        uint64_t ones = 0, ones_c = 0, twos = 0, of_r[RB], of_c[CB];
#pragma unroll
        for (int k = 0; k < RB; ++k)
            of_r[k] = 0;
#pragma unroll
        for (int k = 0; k < CB; ++k)
            of_c[k] = 0;
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            const uint64_t a = __builtin_amdgcn_ballot_w64(by_r[m] <= limit);
            twos |= ones & a;
            ones |= a;
#pragma unroll
            for (int k = 0; k < RB; ++k)
                of_r[k] |= (m >> k) & 1 ? a : 0;
        }
#pragma unroll
        for (int g = 0; g < NC; ++g) {
            const uint64_t a = __builtin_amdgcn_ballot_w64(by_c[g] <= limit);
            twos |= ones_c & a;
            ones_c |= a;
#pragma unroll
            for (int k = 0; k < CB; ++k)
                of_c[k] |= (g >> k) & 1 ? a : 0;
        }
        const auto either = [&](uint64_t a) { return (uint64_t)((uint32_t)a | (uint32_t)(a >> 32)) << (32 * t); };
        ones &= ones_c;
#pragma unroll
        for (int k = 0; k < RB; ++k)
            bit_r[k] |= either(of_r[k]);
#pragma unroll
        for (int k = 0; k < CB; ++k)
            bit_c[k] |= either(of_c[k]);
        some |= either(ones);
        in_half1 |= (uint64_t)(uint32_t)(ones >> 32) << (32 * t);
        several |= (uint64_t)((uint32_t)twos | (uint32_t)(twos >> 32) | ((uint32_t)ones & (uint32_t)(ones >> 32))) << (32 * t);
    }
    // row_step x the token's marked row + col_step x its column + half_step x its half (steps: powers of two)
    __device__ __forceinline__ int index(const int row_step, const int col_step, const int half_step) const
    {
        const auto bit = [](uint64_t mask, int value) { return __builtin_amdgcn_inverse_ballot_w64(mask) ? value : 0; };
        int c = bit(in_half1, half_step);
#pragma unroll
        for (int k = 0; k < RB; ++k)
            c |= bit(bit_r[k], row_step << k);
#pragma unroll
        for (int k = 0; k < CB; ++k)
            c |= bit(bit_c[k], col_step << k);
        return c;
    }
};

// the same marks of one tile as a word per lane, for the rare walk over several groups: bit g a mark of by_c[g], bit
// NC + m one of by_r[m]
template <int NR, int NC>
__device__ inline uint32_t pq_filter_mark_word(const int (&by_r)[NR], const int (&by_c)[NC], int limit)
{
    asm volatile("" : "+v"(limit));  // (keeps these selects inside the branch they are used in)
    uint32_t w = 0;
#pragma unroll
    for (int m = 0; m < NR; ++m)
        w |= by_r[m] <= limit ? 1u << (NC + m) : 0u;
#pragma unroll
    for (int g = 0; g < NC; ++g)
        w |= by_c[g] <= limit ? 1u << g : 0u;
    return w;
}

// code of this lane's token among 256 centroids (xin: its sub-vector; a dead lane passes any finite values and live =
// false).  `coord`: the centroids' coordinates as W (double, float, or _Float16 = inside the fp16 A rows)
template <int DS, typename T, typename W>
__device__ __forceinline__ int pq_filter_code(const unsigned char *arow, const unsigned char *coord, const float scale, const bool cb_bad,
                                     const T (&xin)[DS], const bool live)
{
#pragma clang fp contract(off)
    typedef pq_filter_token<DS, T> token;
    typedef typename token::operand operand;
    constexpr int ROW = pq_filter_row_bytes<T>();
    constexpr int STRIDE = sizeof(W) == 2 ? ROW : DS * (int)sizeof(W);  // of a centroid's coordinates
    const int lane = threadIdx.x & 63;
    token tok;
    tok.set(xin, scale);

    // ---- the 256 computed values of every token, 32 centroids per instruction m.  Kept are the minima over the quads g
    // per m and over m per g: 12 numbers that name every quad with a value near the smallest one without a second pass.
    int by_m[2][8], by_g[2][4];
    const unsigned char *my_row = arow + (lane & 31) * ROW + (lane >> 5) * (ROW / 2);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            by_g[t][g] = 0x7f800000;
#pragma unroll
    for (int m = 0; m < 8; m += 2) {
        const operand A0 = *(const operand *)(my_row + m * (32 * ROW));
        const operand A1 = *(const operand *)(my_row + (m + 1) * (32 * ROW));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const f32x16e d0 = tok.values(A0, t);
            const f32x16e d1 = tok.values(A1, t);
            int q0[4], q1[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                q0[g] = min(min(__float_as_int(d0[4 * g]), __float_as_int(d0[4 * g + 1])), __float_as_int(d0[4 * g + 2]));
                q0[g] = min(q0[g], __float_as_int(d0[4 * g + 3]));
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                q1[g] = min(min(__float_as_int(d1[4 * g]), __float_as_int(d1[4 * g + 1])), __float_as_int(d1[4 * g + 2]));
                q1[g] = min(q1[g], __float_as_int(d1[4 * g + 3]));
                by_g[t][g] = min(min(by_g[t][g], q0[g]), q1[g]);
            }
            by_m[t][m] = min(min(min(q0[0], q0[1]), q0[2]), q0[3]);
            by_m[t][m + 1] = min(min(min(q1[0], q1[1]), q1[2]), q1[3]);
        }
    }
    int b[2], limit[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
        b[t] = min(min(min(by_g[t][0], by_g[t][1]), by_g[t][2]), by_g[t][3]);
    tok.limits(tok.best_of(b[0], b[1]), limit);
    const bool bad = tok.bad || cb_bad;
    pq_filter_marks<8, 4> marks;
#pragma unroll
    for (int t = 0; t < 2; ++t)
        marks.add(t, by_m[t], by_g[t], limit[t]);

    // ---- refine: the defining arithmetic on the marked quads, ascending
    int code = 0;
    double bd = __builtin_huge_val();
    auto coordinates = [&](const unsigned char *at, double (&c)[DS]) {
#pragma unroll
        for (int j = 0; j < DS; ++j) {
            if constexpr (sizeof(W) == 2)
                c[j] = (double)(float)((const W *)at)[j];
            else
                c[j] = (double)((const W *)at)[j];
        }
    };
    auto closer = [&](int c, const double (&y)[DS]) {
        double dist = 0.0;
#pragma unroll
        for (int j = 0; j < DS; ++j) {
            const double diff = (double)tok.x[j] - y[j];
            dist = __builtin_fma(diff, diff, dist);
        }
        code = dist < bd ? c : code;  // strict: the lowest index among equal distances stays
        bd = __builtin_fmin(bd, dist);
    };
    // nearly always one quad is marked, in one of the halves: (m, g) of half s is centroids 32 m + 8 g + 4 s .. + 3
    // (where several are, the sum below is some quad's index all the same)
    {
        const int c0 = marks.index(32, 8, 4);
        const unsigned char *quad = coord + c0 * STRIDE;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double y[DS], dist = 0.0;
            coordinates(quad + k * STRIDE, y);
#pragma unroll
            for (int j = 0; j < DS; ++j) {
                const double diff = (double)tok.x[j] - y[j];
                dist = __builtin_fma(diff, diff, dist);
            }
            code = k > 0 && dist < bd ? k : code;
            bd = k > 0 ? __builtin_fmin(bd, dist) : dist;
        }
        code += c0;
    }
    // several (ties, near-ties, a token far outside the codebook's range): the lane walks every quad whose two bits
    // are set — quad (m, g) of half s is centroids 4 (8 m + 2 g + s) .. + 3
    const uint64_t several = marks.several & __builtin_amdgcn_ballot_w64(live && !bad);
    uint64_t all = 0;  // tokens for which all centroids are the shorter way
    if (several != 0) {  // wave-uniform
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(several);
        const auto halves = __builtin_amdgcn_permlane32_swap(pq_filter_mark_word(by_m[0], by_g[0], limit[0]),
                                                             pq_filter_mark_word(by_m[1], by_g[1], limit[1]), false, false);
        uint64_t left = 0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t h = halves[s];
            const uint32_t of_g = ((h & 1u) | (h & 2u) << 1 | (h & 4u) << 2 | (h & 8u) << 3) << s;  // bits 2 g + s
#pragma unroll
            for (int m = 0; m < 8; ++m)
                left |= (uint64_t)((h >> (4 + m)) & 1u ? of_g : 0u) << (8 * m);
        }
        left = mine ? left : 0;
        all = __builtin_amdgcn_ballot_w64(__builtin_popcountll(left) > 40);
        const int code_one = code;
        code = 0;
        bd = __builtin_huge_val();
        // two quads at a time, the second's coordinates under way with the first's (a lane with nothing left takes its last
        // quad again: no change)
        int quad = 0;
        while (all == 0 && __builtin_amdgcn_ballot_w64(left != 0) != 0) {
            const uint64_t rest = left & (left - 1);
            const int first = left ? __builtin_ctzll(left) : quad;
            quad = rest ? __builtin_ctzll(rest) : first;
            double y[8][DS];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                coordinates(coord + (4 * (k < 4 ? first : quad) + (k & 3)) * STRIDE, y[k]);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                closer(4 * (k < 4 ? first : quad) + (k & 3), y[k]);
            left = rest & (rest - 1);
        }
        if (!mine)
            code = code_one;
    }
    // ... the defining scan for this sub-chunk, also where a token has more than 40 of the 64 quads to walk (4096 tokens x 8
    // heads, a codebook of equal centroids: 436 us walked, 301 scanned; half of them equal: 194 us with one quad at a time
    // and the lanes that are done kept out of it, 168)
    const uint64_t unsure = all | __builtin_amdgcn_ballot_w64(live && bad) | (__builtin_amdgcn_ballot_w64(live) & ~marks.some);
    if (unsure != 0) {  // wave-uniform
        code = 0;
        bd = __builtin_huge_val();
        for (int c = 0; c < 256; ++c) {
            double y[DS];
            coordinates(coord + c * STRIDE, y);
            closer(c, y);
        }
    }
    return code;
}

}  // namespace
