// Nearest centroid of many 2-dim sub-vectors among 256 centroids: a grid over the plane that names, for every cell, the
// centroids that can be the nearest of a point in it.  Shared by the encode of long appends and the k-means assignment;
// the decision is the same fp64 expression as everywhere (pq_encode.hip), so codes are bit-exact.
//
// The filter of pq_nearest_filter.h looks at all 256 values of every token: 355 vector instructions per 64 tokens.  In two
// dimensions the plane can be cut up once per codebook instead, and a token then looks at the 2 or 3 centroids of its cell:
// 68 instructions with codebooks of random vectors, whose cells have long lists more often than trained ones'.  Building a
// grid takes 32 200, as many as 91 chunks of 64 tokens through the filter, so the grid serves appends and trainings of
// thousands of tokens per head (pq_grid_slices below).  Encode (K and V), 32 heads x 32K tokens, kept grids: 392 us, of which 36
// us are workgroups' starts, image loads and ends, 184 the tokens' main path, which vector issue bounds (220 instructions per 64
// tokens and 4 subspaces), and, each left out by itself: 63 the stores of the codes, a byte per token and subspace (stored together 367 us in all: pq_grid_stores_wide), 61 the tokens that
// wait, 34 the rows from memory (1549 us through the filter).  k-means, 32 heads x 64K samples, 2 iterations: 3148 -> 872 us
// (normal data; 940 where the channels' scales go from 1/2 to 2).
//
// Map.  Per axis u = s x + o, chosen from the codebook (mean and mean deviation of its coordinates without outliers):
// |u| <= 28 holds what lies within some 4 standard deviations.  The cell coordinate is five bits of the float |u| + 2 — 8
// cells in each of the four octaves [2, 4) .. [16, 32), fine in the middle and coarse outside, for an addition and a shift —
// and the sign.  64 x 64 cells of 4 bytes.  The last cell on each side takes everything beyond: no list, "outside".
// Lists.  A centroid c can be the nearest of a point of a box only if the bisector of c and some reference centroid r leaves
// part of the box on its side: F_c(g) - F_r(g) <= |da_x| h_x + |da_y| h_y with F_c(p) = |c|^2 / 2 - p . c, g and h the box's
// centre and half sides, da the difference of the gradients.  r is the nearest centroid of the box's centre (any r is safe).
// First for 16 x 16 blocks of 4 x 4 cells, all 256 centroids each; then for every cell, the centroids of its block, which the
// 16 lanes of the block's cells hold and pass to each other (through LDS every candidate cost two 16-byte reads per lane: 860
// us for the encode above, 785 so).
// The test runs in fp32 in u space, where a squared distance is w_x du_x^2 + w_y du_y^2: every F is lowered by 2^-18 of its
// |c|^2 / 2 and the threshold raised by 2^-16 (|r|^2 / 2 + |g|^2 + ..), 16 times what the roundings of u, F and w amount to;
// boxes are 2^-17 wider on each side than the cells (the float |u| + 2 is good to 2^-19).
// A cell's word holds its codes if they are at most 4, filled up with codes that are not in its list; otherwise its halves
// are equal (which those of a list never are): where its words stand in the pool, and how many they are.  Outside, where there is
// no room, or more than 64 candidates in the block: GRID_NONE.
// Tokens.  The four distances in fp32 (relative error below 2^-21), their 8 low bits replaced by the code: one unsigned
// minimum gives the least and its code, one median keeps the second.  More than 2^-16 apart, the order is that of the fp64
// distances.  The others wait in LDS until 64 are there and are then worked on as one: tokens of cells with longer lists (7 % with a
// codebook of random vectors, 1 % with a trained one), whose word gives the least distance twice, in the same way.  What these
// leave undecided ("unsure": near-ties, outside, cells without a list) is put off until 64 of a subspace can go through the filter
// together, and where the codebook gives no useful grid all its tokens go there at once.
// What the data make of it, 32 heads, us, grids built / kept from an earlier append / the filter alone: encode of 9000 tokens,
// normal 358 / 135 / 430, Laplace's distribution 382 / 158 / 429, 2 % of the coordinates times 20 387 / 165 / 429; of 32K 593 / 369
// / 1566, 680 / 462 / 1567, 704 / 485 / 1569.  Centroids that repeat others are taken out: 16 values in all 1430 kept, 2472 by the
// filter (9000 tokens; 2850 when a repeated centroid made its tokens unsure), k-means of 64K samples rounded to quarters 18.5 ->
// 8.1 ms.  A codebook without a useful grid costs the filter four wavefronts per SIMD instead of five: one dead axis in every
// subspace 867 / 750 and 3000 / 2577; with images kept such codebooks are known, and go to the filter's kernel (pq_grid_price_of).
#pragma once

#include <stddef.h>

#include "pq_device_utils.h"
#include "pq_nearest_filter.h"

namespace {

constexpr int GRID_SUB = 4;       // neighbouring subspaces of a workgroup: 16 bytes of every token's fp16 row
constexpr int GRID_WAVES = 16;    // 4 wavefronts build each subspace's grid; then all take tokens, 4 subspaces at a time
constexpr int GRID_SIDE = 64;
// Words of longer lists per subspace.  Random vectors take 400 on average, and up to 1200 where one axis is several times the
// other: its cells then have many candidates.  Tokens of a cell that found no room go to the filter, and a workgroup with such
// subspaces is what the others wait for (k-means of 32 heads x 64K samples, scales 0.5 .. 4 per channel, 5 iterations, when
// these tokens were decided one by one: 0.68 ms each with 1024 words, 0.66 so, and 0.64 with lists of 33 .. 64 by row broadcast).
constexpr int GRID_POOL = 2048;
// Waiting tokens of a wavefront: their number, and where KEEP their fp16 sub-vector as well.  (Read again when its turn came,
// its line had often left the L2: encode, 32K tokens x 32 heads, 696 us, 663 with it.  Beside the k-means' sums, and in
// fp32, there is no room.)  The queue holds fewer than 64 before a chunk, and up to 64 of each subspace more behind it.
template <bool KEEP> using pq_grid_waiting = typename std::conditional<KEEP, uint2, uint32_t>::type;
constexpr int GRID_QUEUE = 64 * (1 + GRID_SUB);
constexpr int GRID_SHIFT = 20;    // 8 cells per octave
constexpr float GRID_BIAS = 2.0f;
constexpr uint32_t GRID_FIRST = 0x40000000u, GRID_LAST = 0x41ffffffu;  // float bits of 2 .. just below 32
constexpr float GRID_COVER = 28.0f;  // where the outermost cell starts, less the bias, ..
constexpr float GRID_DEVIATIONS = 5.0f;  // .. for coordinates this many mean deviations from the mean (normal ones: 3.75 sigma)
constexpr float GRID_LOWERED = 3.814697265625e-06f;   // 2^-18: shares of |c|^2 / 2 that F is lowered by, ..
constexpr float GRID_MARGIN = 1.52587890625e-05f;     // 2^-16: .. that the threshold is raised by,
constexpr float GRID_WIDER = 7.62939453125e-06f;      // 2^-17: and what boxes have more on each side than their cells
constexpr int GRID_LONGEST = 64;  // candidates of a block (a bit each in a 64-bit mask)
constexpr uint32_t GRID_NONE = 0;  // a cell without a list: a list of no words
constexpr uint32_t GRID_SURE = 512;  // keys at least this far apart are in the right order

// The map of a subspace and what is known of its grid.  fp16: a token's cell is found in fp16, both axes at once: 8 instructions
// instead of the 14 of fp32.  Factors, u and |u| + 2 are held there in units of 2^8, whose cells have the same bits: factors then
// reach from deviations of 4e-7 (the smallest fp16 number is 6e-8; in units of 1 they ended at 9e-5, and codebooks of 1e-5 were
// left to the filter: encode of 9000 tokens x 32 heads 585 us) to the largest.  A rounding of 2^-11 of |u| (2^-17 where u is
// subnormal) and one of |u| + 2 move a token by 2^-10 (|u| + 2) at most, which the boxes allow for (GRID_WIDER_F16).
constexpr float GRID_F16_UNIT = 256.0f;
struct pq_grid_map {
    float sx, ox, sy, oy;
    uint32_t s16, o16;     // (fp16: in units of GRID_F16_UNIT, x in the low half)
    float scale;           // of the filter
    uint32_t pool_used, bad;  // bad: 1 no grid, 2 codebook outside the filter's range
    uint32_t lost, unserved;  // how many centroids the grid does not serve: counted before and after its lists
    uint32_t again[8];     // a bit per centroid: equal to one before it
    uint32_t unused;
};
constexpr float GRID_WIDER_F16 = 1.1e-3f;  // of |u| + 2 (2^-10 is 0.98e-3)

// The grids of a workgroup.  Coordinates and cells stand where the 16 bits of an LDS instruction's offset reach those of all
// four (bases apart cost an addition for every look-up); the cells of the four are interleaved, so that the two bytes of a token's
// cell are its address as they are.
template <typename T> struct pq_grids {
    // (what stands in front of arow is the image in memory that a context keeps, the pools as far as they are used)
    T coord[GRID_SUB][256][2];
    uint32_t cell[GRID_SIDE][GRID_SUB][GRID_SIDE];  // [u_x][][u_y]; while building, the 64 bytes of a 4 x 4 block are its list
    pq_grid_map map[GRID_SUB];
    __attribute__((aligned(16))) uint32_t pool[GRID_SUB][GRID_POOL];
    __attribute__((aligned(16))) unsigned char arow[GRID_SUB][256 * pq_filter_row_bytes<T>()];
};
constexpr int GRID_ROW = 4 * GRID_SUB * GRID_SIDE;  // bytes from one u_x to the next
template <typename T> constexpr int pq_grid_image_bytes() { return (int)offsetof(pq_grids<T>, arow); }

// The tokens are taken to lie where the centroids do: where many of the 256 are left to the filter (in cells without a list), it
// does all the work of the subspace.  (For 64 tokens: 68 instructions for the look-ups,
// some 30 for putting tokens off and for 24 of them 135 in the filter; 355 through the filter alone, and building is saved.)
constexpr int GRID_LOST = 96;
__device__ __forceinline__ bool pq_grid_useless(const pq_grid_map &m) { return m.bad != 0 || m.lost > GRID_LOST || m.unserved > GRID_LOST; }

// What a chunk of a subspace's tokens costs a grid workgroup and the filter by itself (10 ns for four such subspaces), for a rule that
// would else take all codebooks to be served by their grids.  A grid that leaves a third of its centroids, so a third of the tokens,
// to the filter takes 233 of its 355 instructions.  A useless one has the filter's work at four wavefronts per SIMD instead of
// five, on codebooks that are the slower ones to the filter as well: 32 heads x 4000 tokens, one dead axis in every subspace 405 us,
// 350 through the filter (200 for normal data); one in four subspaces 176 and 255; centroids beyond the filter's range (bad & 2), all
// distances in fp64, 2494 and 2117 for 9000 tokens with 6 of 10 codebooks so.  Where many centroids repeat others, the filter
// by itself finds all of them and walks over their quads, which these rows do not have (centroids of 16 values 690 and 1118 for
// 4000 tokens, rounded to quarters 566 and 1133).
struct pq_grid_price {
    uint32_t grid, filter;
};
__device__ __forceinline__ pq_grid_price pq_grid_price_of(const pq_grid_map &m)
{
    int repeated = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        repeated += __builtin_popcount(m.again[k]);
    if (m.bad & 2u)
        return {610u, 520u};
    if (repeated >= 64)
        return {240u, 400u};
    if (pq_grid_useless(m))
        return {152u, 130u};
    return {18u + 78u * m.unserved / 256u, 72u};
}

// What building a grid needs of its centroids: a_x, a_y, |c|^2 / 2 lowered, |c|^2 / 2; how many of them lie in each block of
// 4 x 4 cells, 16 bits each (repeated ones not counted); and the first of those whose coordinates have the same hash.  The
// waiting tokens take its place.
typedef float pq_grid_table[256][4];
struct pq_grid_making {
    pq_grid_table table[GRID_SUB];
    uint32_t in_block[GRID_SUB][128];
    uint32_t first_of[GRID_SUB][256];
};
template <bool KEEP> union pq_grid_scratch {
    pq_grid_making making;
    pq_grid_waiting<KEEP> queue[GRID_WAVES][GRID_QUEUE];
};

template <typename T> __device__ __forceinline__ uint32_t pq_grid_hash(const T x, const T y)
{
    uint32_t h;
    if constexpr (sizeof(T) == 2)
        h = (uint32_t)__builtin_bit_cast(uint16_t, x) | (uint32_t)__builtin_bit_cast(uint16_t, y) << 16;
    else
        h = __float_as_uint(x) * 0x85ebca6bu ^ __float_as_uint(y);
    return h * 0x9e3779b1u >> 24;
}

// bits 20 .. 25: the cell coordinate, 0 .. 31 upwards from zero, 63 .. 32 downwards
__device__ __forceinline__ uint32_t pq_grid_axis(const float u)
{
    const uint32_t b = min(__float_as_uint(__builtin_fabsf(u) + GRID_BIAS), GRID_LAST);
    return b ^ (uint32_t)(__float_as_int(u) >> 31);
}

// byte offset of the cell of a point among those of subspace 0, s, o: pq_grid_map's
__device__ __forceinline__ uint32_t pq_grid_cell(const float x, const float y, const float sx, const float ox, const float sy, const float oy)
{
    const uint32_t ex = pq_grid_axis(__builtin_fmaf(x, sx, ox));
    const uint32_t ey = pq_grid_axis(__builtin_fmaf(y, sy, oy));
    static_assert(GRID_SHIFT == 20 && GRID_SIDE == 64 && GRID_ROW == 1024, "the shifts below");
    return ((ex >> 10) & 0xfc00u) | ((ey >> 18) & 0xfcu);
}

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));

// the same in fp16; xy: the point as it stands in memory
__device__ __forceinline__ uint32_t pq_grid_cell_f16(const uint32_t xy, const uint32_t s16, const uint32_t o16)
{
    const f16x2 u = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, xy), __builtin_bit_cast(f16x2, s16), __builtin_bit_cast(f16x2, o16));
    const uint32_t bits = __builtin_bit_cast(uint32_t, u);
    const _Float16 bias = (_Float16)(GRID_BIAS / GRID_F16_UNIT);
    f16x2 w = __builtin_bit_cast(f16x2, bits & 0x7fff7fffu) + (f16x2){bias, bias};
    const _Float16 last = __builtin_bit_cast(_Float16, (uint16_t)0x2fff);  // just below 32 units
    static_assert(GRID_F16_UNIT == 256.0f, "the number above, and three bits of the exponent");
    w = __builtin_elementwise_min(w, (f16x2){last, last});
    // bits 7 .. 12 of each half are its cell coordinate, complemented where u is negative
    const uint32_t five = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, w) >> (u16x2){5, 5});
    const uint32_t sign = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, bits) >> (i16x2){15, 15});
    const uint32_t e = (five ^ sign) & 0x00fc00fcu;
    return __builtin_amdgcn_perm(e, e, 0x0c0c0002u);
}

// the cell of a point of a subspace with a map in memory
template <typename T> __device__ __forceinline__ uint32_t pq_grid_cell_of(const T x, const T y, const pq_grid_map &m)
{
    if constexpr (sizeof(T) == 2)
        return pq_grid_cell_f16((uint32_t)__builtin_bit_cast(uint16_t, x) | (uint32_t)__builtin_bit_cast(uint16_t, y) << 16, m.s16, m.o16);
    else
        return pq_grid_cell(x, y, m.sx, m.ox, m.sy, m.oy);
}

// the block of 4 x 4 cells of a cell's byte offset: [x][y] of 16
__device__ __forceinline__ uint32_t pq_grid_block(const uint32_t cell) { return (cell >> 8 & 0xf0u) | (cell >> 4 & 15u); }

// lower edge of cell coordinate k = -32 .. 32 (31 and -32: the open ones, given an end)
__device__ __forceinline__ float pq_grid_edge(const int k)
{
    const float e = __uint_as_float(GRID_FIRST + ((uint32_t)(k < 0 ? -k : k) << GRID_SHIFT)) - GRID_BIAS;
    return k < 0 ? -e : e;
}

// one of four candidates of a list word: its fp32 distance with the code in the low byte
template <int K, typename T>
__device__ __forceinline__ uint32_t pq_grid_key(const T (&coord)[256][2], const uint32_t word, const T x, const T y, const float minus_one)
{
#pragma clang fp contract(off)
    const uint32_t c = (word >> (8 * K)) & 255u;
    float dx, dy;
    if constexpr (sizeof(T) == 2) {
        const uint32_t both = *(const uint32_t *)&coord[c][0];
        const _Float16 cx = __builtin_bit_cast(_Float16, (uint16_t)both), cy = __builtin_bit_cast(_Float16, (uint16_t)(both >> 16));
        dx = __builtin_fmaf((float)cx, minus_one, (float)x);  // (one instruction takes both halves)
        dy = __builtin_fmaf((float)cy, minus_one, (float)y);
    } else {
        const float2 both = *(const float2 *)&coord[c][0];
        dx = x - both.x;
        dy = y - both.y;
    }
    const float d = __builtin_fmaf(dy, dy, dx * dx);
    return __builtin_amdgcn_perm(__float_as_uint(d), word, 0x07060500u | (uint32_t)K);
}

__device__ __forceinline__ void pq_grid_take(uint32_t &m1, uint32_t &m2, const uint32_t key)
{
    asm("v_med3_u32 %0, %1, %0, %2" : "+v"(m2) : "v"(m1), "v"(key));  // m1 <= m2: the middle one of three
    m1 = min(m1, key);
}

// whether the order of the two least fp32 distances may differ from that of the fp64 ones
template <typename T> __device__ __forceinline__ bool pq_grid_unsure(const uint32_t m1, const uint32_t m2)
{
    // fp32 coordinates: squares below 2^-100 are not good to 2^-21 any more
    return m2 - m1 < GRID_SURE || (sizeof(T) == 4 && m2 < 0x0d800000u);
}

// A wavefront's part of a subspace's tables: the map, which all 4 wavefronts work out alike, and the rows and numbers of
// centroids 64 part .. 64 part + 63.  src: [256][2]; cell, hash: of centroid 64 part + lane
template <typename T>
__device__ __forceinline__ void pq_grid_tables(pq_grids<T> &grids, const int sub, pq_grid_table &table, uint32_t (&first_of)[256], const T *src,
                                               const int part, uint32_t &cell, uint32_t &hash)
{
    pq_grid_map &m = grids.map[sub];
    const int lane = threadIdx.x & 63;
    float x[4], y[4];
    T mine[2] = {};
    float c_max = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const T cx = src[(lane + 64 * r) * 2], cy = src[(lane + 64 * r) * 2 + 1];
        x[r] = (float)cx;
        y[r] = (float)cy;
        c_max = fmaxf(c_max, fmaxf(fabsf(x[r]), fabsf(y[r])));
        if (r == part) {
            mine[0] = cx;
            mine[1] = cy;
        }
    }
    c_max = wave_max(c_max);
    const float scale = pq_filter_scale<T>(c_max);
    // mean and mean deviation, then those of the coordinates within 3 mean deviations
    float mx = 0.f, my = 0.f, ex = 3.0e38f, ey = 3.0e38f, dx = 0.f, dy = 0.f;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        float sx = 0.f, sy = 0.f, nx = 0.f, ny = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool in_x = fabsf(x[r] - mx) <= ex, in_y = fabsf(y[r] - my) <= ey;
            sx += in_x ? x[r] : 0.f;
            sy += in_y ? y[r] : 0.f;
            nx += in_x ? 1.f : 0.f;
            ny += in_y ? 1.f : 0.f;
        }
        nx = 1.0f / wave_sum(nx);
        ny = 1.0f / wave_sum(ny);
        const float new_mx = wave_sum(sx) * nx, new_my = wave_sum(sy) * ny;
        dx = dy = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dx += fabsf(x[r] - mx) <= ex ? fabsf(x[r] - new_mx) : 0.f;
            dy += fabsf(y[r] - my) <= ey ? fabsf(y[r] - new_my) : 0.f;
        }
        dx = wave_sum(dx) * nx;
        dy = wave_sum(dy) * ny;
        mx = new_mx;
        my = new_my;
        ex = 3.0f * dx;
        ey = 3.0f * dy;
    }
    float sx = GRID_COVER / (GRID_DEVIATIONS * dx), sy = GRID_COVER / (GRID_DEVIATIONS * dy);
    float ox = -mx * sx, oy = -my * sy;
    bool usable = dx > 1.0e-30f && dy > 1.0e-30f && c_max < 1.0e30f;
    if constexpr (sizeof(T) == 2) {
        // (an offset of 16384 is rounded to 4 of the 28 on either side of the middle: the mean is then some 3000 mean deviations from
        // zero; 32 heads x 9000 tokens 700 standard deviations from it 2843 us with 4096 for a limit, 644 so)
        const auto rounded = [](float v) { return GRID_F16_UNIT * (float)(_Float16)(v * (1.0f / GRID_F16_UNIT)); };
        sx = rounded(fminf(sx, 60000.f * GRID_F16_UNIT));
        sy = rounded(fminf(sy, 60000.f * GRID_F16_UNIT));
        ox = -mx * sx;
        oy = -my * sy;
        usable = usable && sx > 1.0e-4f && sy > 1.0e-4f && fabsf(ox) < 16384.f && fabsf(oy) < 16384.f;
        ox = rounded(ox);
        oy = rounded(oy);
    }
    // squared distances in units of 1 / s_x^2
    const float ratio = sx / sy, wy = ratio * ratio;
    usable = usable && wy > 1.0e-9f && wy < 1.0e9f;
    bool far_out = false, cb_bad = false;
    const int c = 64 * part + lane;
    pq_filter_build_row<2>(mine, scale, grids.arow[sub] + c * pq_filter_row_bytes<T>(), cb_bad);
    const float ux = __builtin_fmaf((float)mine[0], sx, ox), uy = __builtin_fmaf((float)mine[1], sy, oy);
    far_out = !(fabsf(ux) < 1.0e6f && fabsf(uy) < 1.0e6f);
    const float ay = wy * uy, n = 0.5f * (ux * ux + uy * ay);
    table[c][0] = ux;
    table[c][1] = ay;
    table[c][2] = n * (1.0f - GRID_LOWERED);
    table[c][3] = n;
    grids.coord[sub][c][0] = mine[0];
    grids.coord[sub][c][1] = mine[1];
    const auto both = [](float lo, float hi) {
        return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)(lo * (1.0f / GRID_F16_UNIT))) |
               (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)(hi * (1.0f / GRID_F16_UNIT))) << 16;
    };
    const pq_grid_map here = {sx, ox, sy, oy, both(sx, sy), both(ox, oy)};
    cell = pq_grid_cell_of(mine[0], mine[1], here);
    hash = pq_grid_hash(mine[0], mine[1]);
    atomicMin(&first_of[hash], (uint32_t)c);
    const uint32_t bad = (__builtin_amdgcn_ballot_w64(far_out) != 0 || !usable ? 1u : 0u) |
                         (__builtin_amdgcn_ballot_w64(cb_bad) != 0 ? 3u : 0u);
    if (lane == 0) {
        if (part == 0) {
            m.sx = sx;
            m.ox = ox;
            m.sy = sy;
            m.oy = oy;
            m.s16 = here.s16;
            m.o16 = here.o16;
            m.scale = scale;
        }
        if (bad)
            atomicOr(&m.bad, bad);
    }
}

__device__ __forceinline__ void pq_grid_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// centre and half side of cell coordinates e .. e + n - 1 (e as in pq_grid_axis)
template <typename T> __device__ __forceinline__ void pq_grid_box(const int e, const int n, float &g, float &h)
{
    const int k = e < 32 ? e : e - 64;
    const float lo = pq_grid_edge(k), hi = pq_grid_edge(k + n);
    g = 0.5f * (lo + hi);
    h = 0.5f * (hi - lo) + GRID_WIDER;
    if constexpr (sizeof(T) == 2)
        h = __builtin_fmaf(fmaxf(-lo, hi) + GRID_BIAS, GRID_WIDER_F16, h);
}

// Appending the bit t <= limit to a mask is a comparison and an addition with carry.  What a vector instruction writes to VCC
// or a scalar register may be read by another from two wait states on; the compiler sees to that, but not inside of asm.  So
// several candidates are marked at a time, and every read stands behind two other instructions.  (Left to the compiler, an
// instruction more each: encode of 32K tokens x 32 heads 673 us, 659 so; k-means of 32 heads x 64K samples 1002 and 987.)

// appends the bits t[k] <= limit to a mask, k = 0 .. 3
__device__ __forceinline__ void pq_grid_mark_four(uint32_t &mask, const float (&t)[4], const float limit)
{
    uint64_t of0, of1, of2;
    asm("v_cmp_le_f32_e64 %1, %4, %8\n\t"
        "v_cmp_le_f32_e64 %2, %5, %8\n\t"
        "v_cmp_le_f32_e64 %3, %6, %8\n\t"
        "v_cmp_le_f32_e32 vcc, %7, %8\n\t"
        "v_addc_co_u32_e64 %0, %1, %0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, %0, %0, %3\n\t"
        "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
        : "+&v"(mask), "=&s"(of0), "=&s"(of1), "=&s"(of2)
        : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(limit)
        : "vcc");
}

// the same for two, and shifts the codes of those that are marked into a word
__device__ __forceinline__ void pq_grid_mark_two(uint32_t &mask, uint32_t &word, const uint32_t code0, const uint32_t code1, const float t0,
                                                 const float t1, const float limit)
{
    uint64_t of0;
    uint32_t next;
    asm("v_cmp_le_f32_e64 %2, %6, %8\n\t"
        "v_cmp_le_f32_e32 vcc, %7, %8\n\t"
        "v_lshl_or_b32 %3, %1, 8, %4\n\t"
        "v_cndmask_b32_e64 %1, %1, %3, %2\n\t"
        "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
        "v_lshl_or_b32 %3, %1, 8, %5\n\t"
        "v_cndmask_b32_e32 %1, %1, %3, vcc\n\t"
        "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
        : "+&v"(mask), "+&v"(word), "=&s"(of0), "=&v"(next)
        : "v"(code0), "v"(code1), "v"(t0), "v"(t1), "v"(limit)
        : "vcc");
}

// lane K's value in every row of 16 lanes
template <int K> __device__ __forceinline__ float pq_grid_row(const float x) { return dpp_move<0x150 + K>(x); }

// v += x (lane K's in every row of 16 lanes) ax + y (lane K's) ay; two wait states after a vector write of x or y are due
// before they are read across lanes
template <int K> __device__ __forceinline__ void pq_grid_row_fma(float &v, const float x, const float ax, const float y, const float ay)
{
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+&v"(v) : "v"(x), "v"(ax), "v"(y), "v"(ay), "n"(K));
}

// the word of a cell with a longer list: both halves say where its words stand in the pool and how many they are
__device__ __forceinline__ uint32_t pq_grid_list_word(const uint32_t at, const uint32_t words)
{
    static_assert(GRID_POOL <= 2048 && GRID_LONGEST / 4 < 32, "11 and 5 bits");
    return (at | words << 11) * 0x10001u;
}

// calls f(K, K + 1), integral constants, for the even K < N while K is below `most` (uniform)
template <int K, int N, typename F> __device__ __forceinline__ void pq_grid_twos(const int most, F f)
{
    if constexpr (K < N) {
        if (K < most) {
            f(std::integral_constant<int, K>(), std::integral_constant<int, K + 1>());
            pq_grid_twos<K + 2, N>(most, f);
        }
    }
}

// The lists of one quarter of the grid (cell rows 16 part .. 16 part + 15), by one wavefront.  box: centre and half side of
// the 64 cell coordinates
template <typename T>
__device__ __forceinline__ void pq_grid_lists(pq_grids<T> &grids, const int sub, const pq_grid_table &table, const float2 (&box)[GRID_SIDE],
                                              const int part)
{
    const int lane = threadIdx.x & 63;
    pq_grid_map &m = grids.map[sub];
    unsigned char *bytes = (unsigned char *)grids.cell[0][sub];
    // where candidate k of a block's list stands behind its first byte: 16 in each of the block's rows of cells
    const auto place = [](const uint32_t k) { return k + __umul24(k & 48u, GRID_ROW / 16 - 1); };
    const float sx = m.sx, ox = m.ox, sy = m.sy, oy = m.oy;
    const float ratio = sx / sy, wy = ratio * ratio;

    // ---- lane = block of 4 x 4 cells, all centroids
    int count = 0;
    uint32_t fill = 0;  // a code that is not in the block's list
    {
        const int bx = part * 4 + (lane >> 4), by = lane & 15;
        const uint32_t list = (uint32_t)(bx * 4 * GRID_ROW + by * 16);
        float gx, hx, gy, hy;
        pq_grid_box<T>(4 * bx, 4, gx, hx);
        pq_grid_box<T>(4 * by, 4, gy, hy);
        const float px = (gx - ox) / sx, py = (gy - oy) / sy;
        const float end = sizeof(T) == 2 ? 60000.f : 3.0e37f;
        const T p[2] = {(T)fminf(fmaxf(px, -end), end), (T)fminf(fmaxf(py, -end), end)};
        typedef typename std::conditional<sizeof(T) == 4, float, _Float16>::type W;
        const int r = pq_filter_code<2, T, W>(grids.arow[sub], sizeof(T) == 4 ? (const unsigned char *)grids.coord[sub] : grids.arow[sub],
                                                   m.scale, false, p, true);
        const float4 ref = *(const float4 *)table[r];
        const float far_x = fabsf(gx) + hx, far_y = fabsf(gy) + hy;
        const float limit = __builtin_fmaf(-gy, ref.y, __builtin_fmaf(-gx, ref.x, ref.z)) +
                            GRID_MARGIN * (ref.w + far_x * far_x + wy * far_y * far_y);
        uint32_t used = 0;  // which of codes 0 .. 31 are in the list
#pragma unroll 1
        for (int w = 0; w < 256; w += 32) {
            uint32_t mask = 0;  // candidate w + k in bit 31 - k
#pragma unroll 2
            for (int k = 0; k < 32; k += 4) {
                float t[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float4 c = *(const float4 *)table[w + k + j];
                    t[j] = __builtin_fmaf(-gy, c.y, __builtin_fmaf(-gx, c.x, c.z));
                    t[j] = __builtin_fmaf(-fabsf(c.x - ref.x), hx, t[j]);
                    t[j] = __builtin_fmaf(-fabsf(c.y - ref.y), hy, t[j]);
                }
                pq_grid_mark_four(mask, t, limit);
            }
            used = w == 0 ? __builtin_bitreverse32(mask) : used;
            const int total = count + __builtin_popcount(mask);
            mask = total <= GRID_LONGEST ? mask : 0;
            while (__builtin_amdgcn_ballot_w64(mask != 0) != 0) {
                if (mask != 0) {
                    const int k = __builtin_clz(mask);
                    bytes[list + place((uint32_t)count)] = (unsigned char)(w + k);
                    ++count;
                    mask ^= 0x80000000u >> k;
                }
            }
            count = total;  // (beyond GRID_LONGEST nothing is written any more)
        }
        // Lists are filled up to whole words with a code that is not in them: it is never the least, and being there more
        // than once it hides no second least.
        const uint32_t others = used | m.again[0];  // (a repetition of a listed one would be as near as that)
        fill = (uint32_t)__builtin_ctz(~others | 0x80000000u);
        for (int k = count; (k & 3) != 0 && k < GRID_LONGEST; ++k)
            bytes[list + place((uint32_t)k)] = (unsigned char)fill;
        count = others == 0xffffffffu ? GRID_LONGEST + 1 : count;  // (none to fill up with: no list)
    }
    pq_grid_fence();

    // The blocks in the order of their lists' lengths: the 4 that a step takes are then about equally long.
    int order = 0;  // lane n: the n-th block
    {
        const int key = count * 64 + lane;
        int rank = 0;
#pragma unroll 8
        for (int l = 0; l < 64; ++l)
            rank += __builtin_amdgcn_readlane(key, l) < key ? 1 : 0;
        order = __builtin_amdgcn_ds_permute(rank * 4, lane);
    }

    // ---- 16 lanes = the cells of a block, 4 blocks at a time, the centroids of its list: lane k of the 16 holds the k-th
#pragma unroll 1
    for (int it = 0; it < 16; ++it) {
        const int in_row = lane & 15;
        const int block = __shfl(order, it * 4 + (lane >> 4));
        const int n = __shfl(count, block);
        const int cell_x = 4 * (part * 4 + (block >> 4)) + (in_row >> 2);
        const int cell_y = 4 * (block & 15) + (in_row & 3);
        const uint32_t list = (uint32_t)((part * 4 + (block >> 4)) * (4 * GRID_ROW) + (block & 15) * 16);
        const int longest = __builtin_amdgcn_readlane(n, 63);  // of the 4 blocks: the last
        uint32_t word = 0;
        const bool inside = cell_x != 31 && cell_x != 32 && cell_y != 31 && cell_y != 32;
        const float2 x = box[cell_x], y = box[cell_y];
        const float far_x = fabsf(x.x) + x.y, far_y = fabsf(y.x) + y.y;
        const float half = 0.5f * (x.x * x.x + wy * y.x * y.x);
        const float minus_gx = -x.x, minus_gy = -y.x;
        const float far = far_x * far_x + wy * far_y * far_y;
        const uint32_t fill_cell = (uint32_t)__shfl((int)fill, block) * 0x01010101u;
        // more than four candidates: written to the pool from a mask of the block's list (candidate k in the k-th bit from
        // the top)
        auto write_list = [&](auto mask, const bool listed) {
            constexpr bool LONG = sizeof(mask) == 8;
            const int total = LONG ? __builtin_popcountll(mask) : __builtin_popcount((uint32_t)mask);
            const uint32_t words = (uint32_t)(total + 3) >> 2;
            uint32_t at = GRID_POOL;
            if (listed)
                at = atomicAdd(&m.pool_used, words);
            const bool fits = listed && at + words <= GRID_POOL;
            mask = fits ? mask : 0;
            for (uint32_t w = 0; __builtin_amdgcn_ballot_w64(mask != 0) != 0; ++w) {
                uint32_t four = fill_cell;
                const bool any = mask != 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = LONG ? __builtin_clzll(mask | 1u) : __builtin_clz((uint32_t)mask | 1u);
                    const uint32_t c = bytes[list + place((uint32_t)k)];
                    four = mask != 0 ? __builtin_amdgcn_perm(c, four, 0x03020100u + ((4u - (uint32_t)j) << (8 * j))) : four;
                    mask &= ~((decltype(mask))1 << (LONG ? 63 - k : 31 - k));
                }
                if (any)
                    grids.pool[sub][at + w] = four;
            }
            if (listed)
                word = fits ? pq_grid_list_word(at, words) : GRID_NONE;
        };
        if (__builtin_amdgcn_readlane(n, 0) <= 32) {
            const int most = longest < 32 ? longest : 32;
            const uint32_t code1 = bytes[list + (uint32_t)in_row];
            float4 first = *(const float4 *)table[code1];
            first.z = in_row < n ? first.z : 1.0e30f;  // behind the block's own list: far away
            uint32_t code2 = code1;
            float4 second = first;
            if (most > 16) {
                code2 = bytes[list + GRID_ROW + (uint32_t)in_row];
                second = *(const float4 *)table[code2];
                second.z = in_row + 16 < n ? second.z : 1.0e30f;
            }
            // half the squared distances of its centre; the least, with its place in the list in the low bits
            float v[32];
            int least = 0x7f7fffff;
            const auto distance = [&](auto K) {
                const float4 &e = K < 16 ? first : second;
                constexpr int k = K & 15;
                v[K] = pq_grid_row<k>(e.z) + half;
                pq_grid_row_fma<k>(v[K], e.x, minus_gx, e.y, minus_gy);
                least = min(least, (__float_as_int(v[K]) & ~31) | (int)K);
            };
            pq_grid_twos<0, 32>(most, [&](auto K0, auto K1) {
                distance(K0);
                distance(K1);
            });
            const float4 ref = *(const float4 *)table[bytes[list + place((uint32_t)least & 31u)]];
            const float nearest = __int_as_float(least & ~31);
            const float limit = nearest + GRID_MARGIN * (2.f * fabsf(nearest) + ref.w + far);
            uint32_t mask = 0, marked = fill_cell;
            pq_grid_twos<0, 32>(most, [&](auto K0, auto K1) {
                const auto test = [&](auto K, uint32_t &code) {
                    const float4 &e = K < 16 ? first : second;
                    constexpr int k = K & 15;
                    code = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(K < 16 ? code1 : code2), 0x150 + k, 0xf, 0xf, true);
                    const float t = __builtin_fmaf(-fabsf(pq_grid_row<k>(e.x) - ref.x), x.y, v[K]);
                    return __builtin_fmaf(-fabsf(pq_grid_row<k>(e.y) - ref.y), y.y, t);
                };
                uint32_t code[2];
                const float t0 = test(K0, code[0]), t1 = test(K1, code[1]);
                pq_grid_mark_two(mask, marked, code[0], code[1], t0, t1, limit);
            });
            mask <<= 32 - ((most + 1) & ~1);
            word = n <= 32 ? marked : word;
            const bool listed = n <= 32 && inside && __builtin_popcount(mask) > 4;
            if (__builtin_amdgcn_ballot_w64(listed) != 0)  // wave-uniform
                write_list(mask, listed);
        }
        // longer lists (many where one axis is several times the other), the same 16 candidates at a time
        if (longest > 32 && __builtin_amdgcn_ballot_w64(n > 32 && n <= GRID_LONGEST) != 0) {
            const int most = longest < GRID_LONGEST ? longest : GRID_LONGEST;
            auto sixteen = [&](const int q) {
                float4 e = *(const float4 *)table[bytes[list + (uint32_t)(q * GRID_ROW + in_row)]];
                e.z = 16 * q + in_row < n ? e.z : 1.0e30f;
                return e;
            };
            int least = 0x7f7fffff;
#pragma unroll 1
            for (int q = 0; 16 * q < most; ++q) {
                const float4 e = sixteen(q);
                const auto distance = [&](auto K) {
                    float v = pq_grid_row<K>(e.z) + half;
                    pq_grid_row_fma<K>(v, e.x, minus_gx, e.y, minus_gy);
                    least = min(least, (__float_as_int(v) & ~63) | (16 * q + (int)K));
                };
                pq_grid_twos<0, 16>(most - 16 * q, [&](auto K0, auto K1) {
                    distance(K0);
                    distance(K1);
                });
            }
            const float4 ref = *(const float4 *)table[bytes[list + place((uint32_t)least & 63u)]];
            const float nearest = __int_as_float(least & ~63);
            const float limit = nearest + GRID_MARGIN * (2.f * fabsf(nearest) + ref.w + far);
            uint64_t mask = 0;  // candidate k in bit 63 - k
#pragma unroll 1
            for (int q = 0; 16 * q < most; ++q) {
                const float4 e = sixteen(q);
                uint32_t some = 0;
                const auto test = [&](auto K) {
                    float t = pq_grid_row<K>(e.z) + half;
                    pq_grid_row_fma<K>(t, e.x, minus_gx, e.y, minus_gy);
                    t = __builtin_fmaf(-fabsf(pq_grid_row<K>(e.x) - ref.x), x.y, t);
                    return __builtin_fmaf(-fabsf(pq_grid_row<K>(e.y) - ref.y), y.y, t);
                };
                pq_grid_twos<0, 16>(most - 16 * q, [&](auto K0, auto K1) {
                    const float t0 = test(K0), t1 = test(K1);
                    some = some * 4 + (t0 <= limit ? 2u : 0u) + (t1 <= limit ? 1u : 0u);
                });
                const int n_marked = most - 16 * q < 16 ? (most - 16 * q + 1) & ~1 : 16;
                mask |= (uint64_t)(some << (16 - n_marked)) << (48 - 16 * q);
            }
            const bool own = n > 32 && n <= GRID_LONGEST && inside;
            if (own && __builtin_popcountll(mask) <= 4) {
                word = fill_cell;
                for (uint64_t left = mask; left != 0;) {
                    const int k = __builtin_clzll(left);
                    word = word << 8 | bytes[list + place((uint32_t)k)];
                    left &= ~(1ull << (63 - k));
                }
            }
            const bool listed = own && __builtin_popcountll(mask) > 4;
            if (__builtin_amdgcn_ballot_w64(listed) != 0)
                write_list(mask, listed);
        }
        grids.cell[cell_x][sub][cell_y] = inside && n <= GRID_LONGEST ? word : GRID_NONE;
    }
}

// A centroid that repeats an earlier one is never a code: it is taken out of the filter's rows and of all lists, so that its
// tokens have one nearest centroid (left in, a token there was unsure, and a codebook of some 100 values no case for a
// grid).  A repetition behind a clash of hashes is not seen, and costs time only.
template <typename T>
__device__ __forceinline__ bool pq_grid_take_out(pq_grids<T> &grids, const int sub, pq_grid_table &table, uint32_t (&in_block)[128],
                                                 const uint32_t (&first_of)[256], const int part, const uint32_t cell, const uint32_t hash)
{
    const int lane = threadIdx.x & 63, c = 64 * part + lane;
    const int other = (int)first_of[hash];
    const T(&coord)[256][2] = grids.coord[sub];
    const bool again = other < c && coord[other][0] == coord[c][0] && coord[other][1] == coord[c][1];
    const uint64_t of = __builtin_amdgcn_ballot_w64(again);
    if (lane < 2)
        grids.map[sub].again[2 * part + lane] = (uint32_t)(of >> (32 * lane));
    const uint32_t block = pq_grid_block(cell);
    if (again) {
        pq_filter_hide_row<2, T>(grids.arow[sub] + c * pq_filter_row_bytes<T>());
        table[c][2] = 1.0e30f;  // far from everywhere
    } else {
        atomicAdd(&in_block[block >> 1], 1u << (16 * (block & 1u)));
    }
    return again;
}

// How many of the wavefront's 64 centroids the grid will not serve, known before the lists are, which take most of the
// building: those outside the map or in a block with more than GRID_LONGEST of them, all of which would be in its list (tight
// clusters).
__device__ __forceinline__ int pq_grid_lost(const uint32_t (&in_block)[128], const uint32_t cell, const bool again)
{
    const uint32_t ex = cell >> 10, ey = cell >> 2 & 63u, block = pq_grid_block(cell);
    const bool outside = ex - 31u < 2u || ey - 31u < 2u;
    const uint32_t n = in_block[block >> 1] >> (16 * (block & 1u)) & 0xffffu;
    return __builtin_popcountll(__builtin_amdgcn_ballot_w64(!again && (outside || n > GRID_LONGEST)));
}

// Builds the grids of a workgroup's 4 subspaces.  src: the codebook of the first of them, [4][256][2]
template <typename T> __device__ __forceinline__ void pq_grid_build(pq_grids<T> &grids, pq_grid_making &making, float2 (&box)[GRID_SIDE], const T *src)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = wave >> 2, part = wave & 3;
    pq_grid_map &m = grids.map[sub];
    if (threadIdx.x < GRID_SUB) {
        grids.map[threadIdx.x].pool_used = 0;
        grids.map[threadIdx.x].bad = 0;
        grids.map[threadIdx.x].lost = 0;
        grids.map[threadIdx.x].unserved = 0;
    }
    if (threadIdx.x < GRID_SIDE)
        pq_grid_box<T>((int)threadIdx.x, 1, box[threadIdx.x].x, box[threadIdx.x].y);
    if (threadIdx.x < GRID_SUB * 128)
        ((uint32_t *)making.in_block)[threadIdx.x] = 0;
    ((uint32_t *)making.first_of)[threadIdx.x] = 255;
    __syncthreads();
    uint32_t cell, hash;
    pq_grid_tables(grids, sub, making.table[sub], making.first_of[sub], src + sub * 512, part, cell, hash);
    __syncthreads();
    const bool again = pq_grid_take_out(grids, sub, making.table[sub], making.in_block[sub], making.first_of[sub], part, cell, hash);
    __syncthreads();
    const int n_lost = pq_grid_lost(making.in_block[sub], cell, again);
    if (lane == 0)
        atomicAdd(&m.lost, (uint32_t)n_lost);
    __syncthreads();
    const bool lists = m.bad == 0 && m.lost <= GRID_LOST;  // (the same for the 4 wavefronts)
    if (lists)
        pq_grid_lists(grids, sub, making.table[sub], box, part);
    __syncthreads();
    if (lists) {
        const uint32_t word = *(const uint32_t *)((const char *)grids.cell[0][sub] + cell);
        const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(word == GRID_NONE));
        if (lane == 0 && n != 0)
            atomicAdd(&m.unserved, (uint32_t)n);
    }
    __syncthreads();
    if (pq_grid_useless(m)) {
        for (int k = part; k < GRID_SIDE; k += 4)
            grids.cell[k][sub][lane] = GRID_NONE;
        if constexpr (sizeof(T) == 2) {  // what the filter refines with, in place of the lists
            const int c = 64 * part + lane;
            double *wide = (double *)grids.pool[sub] + 2 * c;
            wide[0] = (double)((float)grids.coord[sub][c][0] * m.scale);
            wide[1] = (double)((float)grids.coord[sub][c][1] * m.scale);
        }
    }
    __syncthreads();
}

// the value of subspace j of the group (as values: a choice among array elements would put the array into memory)
template <typename V> __device__ __forceinline__ V pq_grid_pick(const int j, const V a, const V b, const V c, const V d)
{
    return j == 0 ? a : j == 1 ? b : j == 2 ? c : d;
}

// The coordinates that the filter refines with in a subspace without a grid: fp64, which then stand in place of the lists, as
// in the encode's own filter kernel; fp32 as they are.
template <typename T> using pq_grid_wide = typename std::conditional<sizeof(T) == 4, float, double>::type;

// The chunks of a workgroup through the filter, for the subspaces in the mask `useless`
template <typename T, typename TOKEN, typename FETCH, typename STORE>
__device__ __forceinline__ void pq_grid_filter_scan(const pq_grids<T> &grids, const uint32_t useless, const int first, const int last,
                                                    FETCH fetch, STORE store)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    TOKEN next;
    fetch(first + wave, next);
#pragma unroll 1
    for (int chunk = first + wave; chunk < last; chunk += GRID_WAVES) {
        const TOKEN k = next;
        fetch(chunk + GRID_WAVES, next);
#pragma unroll 1
        for (int j = 0; j < GRID_SUB; ++j) {
            if (((useless >> j) & 1u) == 0)
                continue;
            const T x[2] = {pq_grid_pick(j, k.x[0][0], k.x[1][0], k.x[2][0], k.x[3][0]),
                            pq_grid_pick(j, k.x[0][1], k.x[1][1], k.x[2][1], k.x[3][1])};
            const int code = pq_filter_code<2, T, pq_grid_wide<T>>(
                grids.arow[j], sizeof(T) == 4 ? (const unsigned char *)grids.coord[j] : (const unsigned char *)grids.pool[j], grids.map[j].scale,
                (grids.map[j].bad & 2u) != 0, x, k.live);
            store(k, j, code, k.live);
        }
    }
}

// The values are here, in registers of their own, from here on: without it the copy from the registers that the next chunk's rows
// are loaded into stands at the end of the loop, and waits for them there.
template <typename T> __device__ __forceinline__ void pq_grid_hold(T (&x)[GRID_SUB][2])
{
    uint32_t w[sizeof(x) / 4];
    __builtin_memcpy(w, x, sizeof(x));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(x) / 4); ++i)
        asm volatile("" : "+v"(w[i]));
    __builtin_memcpy(x, w, sizeof(x));
}

// the subspaces that are the filter's alone, a bit each
template <typename T> __device__ __forceinline__ uint32_t pq_grid_useless_of(const pq_grids<T> &grids)
{
    uint32_t useless = 0;
#pragma unroll
    for (int j = 0; j < GRID_SUB; ++j)
        useless |= (uint32_t)__builtin_amdgcn_readfirstlane(pq_grid_useless(grids.map[j]) ? 1 << j : 0);
    return useless;
}

// All tokens of a workgroup, 64 at a time, chunks first + wave, first + wave + 16, .. below last.
//   fetch(chunk, token &)    the chunk's tokens, lane = token: x[4][2] and live; called for one chunk more than there are,
//                            in ascending order; copied for another walk over the chunks
//   store(token, j, code, decided)  the code of this lane's token for subspace j of the group, if it is decided
//   store_four(token, codes)  FOUR, the number of its stores, is not 0: the codes of this lane's token, one a byte, for chunks with a
//                            token in every lane.  Those not decided are stored with the others, and again by store_late: by the
//                            same wavefront, whose stores stay in order, or behind a wait.  No subspace is the filter's alone
//   again(id, x, y)          the sub-vector of a token that was put off, id = (chunk - first) << 8 | lane << 2 | j
//   store_late(id, x, y, code)
// Two kinds of tokens are put off until 64 of them can be worked on as one:
//   waiting  not decided by the distances of a cell's word: in LDS, all four subspaces together
//   unsure   nor by those of its list: per subspace, in a register that holds their ids lane by lane (fp16: another their sub-vectors); the filter takes
//            64 for 355 instructions.  (All lanes on one token's fp64 distances take 80, and 3 to 4 % of the tokens lie outside
//            where the coordinates have heavy tails: encode of 32 heads x 9000 tokens, Laplace's distribution, 682 us one at a
//            time, 411 so.)  What the 16 wavefronts have left over in the end is decided together: 457 us by each for itself.
template <typename T, bool KEEP, int FOUR, typename TOKEN, typename FETCH, typename STORE, typename STORE_FOUR, typename AGAIN, typename STORE_LATE>
__device__ __forceinline__ void pq_grid_scan(pq_grids<T> &grids, pq_grid_waiting<KEEP> (&queue)[GRID_WAVES][GRID_QUEUE], const int first,
                                             const int last, FETCH fetch, STORE store, STORE_FOUR store_four, AGAIN again, STORE_LATE store_late)
{
    typedef typename std::conditional<sizeof(T) == 4, float, _Float16>::type W;
    constexpr bool WITH = sizeof(T) == 2;  // unsure tokens keep their sub-vectors
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t useless = FOUR != 0 ? 0u : pq_grid_useless_of(grids);
    if (useless != 0) {
        pq_grid_filter_scan<T, TOKEN>(grids, useless, first, last, fetch, store);
        if (useless == (1u << GRID_SUB) - 1u)
            return;
    }
    pq_grid_map map[GRID_SUB];  // (in registers, as far as it is used)
#pragma unroll
    for (int j = 0; j < GRID_SUB; ++j) {
        const auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
        map[j].s16 = (uint32_t)__builtin_amdgcn_readfirstlane((int)grids.map[j].s16);
        map[j].o16 = grids.map[j].o16;
        map[j].sx = uniform(grids.map[j].sx);
        map[j].sy = uniform(grids.map[j].sy);
        map[j].ox = grids.map[j].ox;
        map[j].oy = grids.map[j].oy;
    }
    float minus_one = -1.0f;
    asm volatile("" : "+s"(minus_one));  // (a difference of two halves in one instruction, not two conversions more)

    const auto word_of = [](const T x, const T y) {
        return WITH ? (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x) | (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)y) << 16 : 0u;
    };
    const auto of_word = [](const uint32_t xy, T &x, T &y) {
        x = (T)__builtin_bit_cast(_Float16, (uint16_t)xy);
        y = (T)__builtin_bit_cast(_Float16, (uint16_t)(xy >> 16));
    };
    // the codes of 64 unsure tokens of subspace j; a lane that is not live passes the id of a token too
    const auto decide = [&](const int j, const uint32_t id, const uint32_t xy, const bool live) {
        T x[2];
        if constexpr (WITH)
            of_word(xy, x[0], x[1]);
        else
            again(id, x[0], x[1]);
        const int code = pq_filter_code<2, T, W>(grids.arow[j], sizeof(T) == 4 ? (const unsigned char *)grids.coord[j] : grids.arow[j],
                                                 grids.map[j].scale, (grids.map[j].bad & 2u) != 0, x, live);
        if (live)
            store_late(id, x[0], x[1], code);
    };
    int n_waiting = 0;
    uint32_t n_unsure = 0;  // of subspace j in byte j; below 64
    uint32_t unsure_id[GRID_SUB] = {}, unsure_xy[GRID_SUB] = {};

    TOKEN next;
    int chunk = first + wave;
    fetch(chunk, next);
    // (as many stores behind the rows as in the loop, so that there is one number to wait for; nothing is stored)
    if constexpr (WITH) {
#pragma unroll
        for (int s = 0; s < (FOUR != 0 ? FOUR : GRID_SUB); ++s)
            store(next, s, s, false);
    }
    for (;;) {
        uint64_t unsure;  // the lanes whose tokens this step leaves unsure, of subspace `j`
        uint32_t id, xy;
        int j;
        if (n_waiting < 64 && chunk < last) {
            TOKEN k = next;
            if constexpr (sizeof(T) == 2)
                pq_grid_hold(k.x);
            fetch(chunk + GRID_WAVES, next);  // in flight while this chunk is worked on
            const uint32_t at = (uint32_t)(chunk - first) << 8 | (uint32_t)lane << 2;
            uint32_t word[GRID_SUB], m1[GRID_SUB], m2[GRID_SUB];
#pragma unroll
            for (int s = 0; s < GRID_SUB; ++s)
                word[s] = *(const uint32_t *)((const char *)grids.cell[0][s] + pq_grid_cell_of(k.x[s][0], k.x[s][1], map[s]));
#pragma unroll
            for (int s = 0; s < GRID_SUB; ++s) {
                const uint32_t k0 = pq_grid_key<0>(grids.coord[s], word[s], k.x[s][0], k.x[s][1], minus_one);
                const uint32_t k1 = pq_grid_key<1>(grids.coord[s], word[s], k.x[s][0], k.x[s][1], minus_one);
                m1[s] = min(k0, k1);
                m2[s] = max(k0, k1);
                pq_grid_take(m1[s], m2[s], pq_grid_key<2>(grids.coord[s], word[s], k.x[s][0], k.x[s][1], minus_one));
                pq_grid_take(m1[s], m2[s], pq_grid_key<3>(grids.coord[s], word[s], k.x[s][0], k.x[s][1], minus_one));
            }
            const uint64_t live = __builtin_amdgcn_ballot_w64(k.live);
            const bool whole = FOUR != 0 && ~live == 0;
            if (whole)
                store_four(k, __builtin_amdgcn_perm(m1[1], m1[0], 0x0c0c0400u) | __builtin_amdgcn_perm(m1[3], m1[2], 0x04000c0cu));
#pragma unroll
            for (int s = 0; s < GRID_SUB; ++s) {
                const uint64_t mine = (useless >> s) & 1u ? 0 : live;
                const uint64_t waits = __builtin_amdgcn_ballot_w64(pq_grid_unsure<T>(m1[s], m2[s])) & mine;
                if (!whole)
                    store(k, s, (int)(m1[s] & 255u), __builtin_amdgcn_inverse_ballot_w64(mine & ~waits));
                if (__builtin_amdgcn_inverse_ballot_w64(waits)) {
                    const int to = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(waits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)waits, (uint32_t)n_waiting));
                    if constexpr (KEEP)
                        queue[wave][to] = make_uint2(at | (uint32_t)s, word_of(k.x[s][0], k.x[s][1]));
                    else
                        queue[wave][to] = at | (uint32_t)s;
                }
                n_waiting += __builtin_popcountll(waits);
            }
            chunk += GRID_WAVES;
            continue;
        } else if (n_waiting > 0) {  // the last 64 of those that wait
            const int n = n_waiting < 64 ? n_waiting : 64;
            n_waiting -= n;
            const bool live = lane < n;
            pq_grid_fence();
            const pq_grid_waiting<KEEP> entry = queue[wave][n_waiting + (live ? lane : 0)];
            T x, y;
            if constexpr (KEEP) {
                id = entry.x;
                of_word(entry.y, x, y);
            } else {
                id = entry;
                again(id, x, y);
            }
            pq_grid_fence();
            j = (int)(id & 3u);
            id &= ~3u;
            const uint32_t word = *(const uint32_t *)((const char *)grids.cell[0][j] + pq_grid_cell_of(x, y, grids.map[j]));
            // (a token whose cell has no list keeps two equal distances)
            const uint32_t words = word >> 16 == (word & 0xffffu) ? word >> 27 : 0u, at = word & 2047u;
            uint32_t m1 = 0xffffffffu, m2 = 0xffffffffu;
            for (uint32_t k = 0; __builtin_amdgcn_ballot_w64(k < words) != 0; ++k) {
                if (k < words) {
                    const uint32_t four = grids.pool[j][at + k];
                    pq_grid_take(m1, m2, pq_grid_key<0>(grids.coord[j], four, x, y, minus_one));
                    pq_grid_take(m1, m2, pq_grid_key<1>(grids.coord[j], four, x, y, minus_one));
                    pq_grid_take(m1, m2, pq_grid_key<2>(grids.coord[j], four, x, y, minus_one));
                    pq_grid_take(m1, m2, pq_grid_key<3>(grids.coord[j], four, x, y, minus_one));
                }
            }
            unsure = __builtin_amdgcn_ballot_w64(live && pq_grid_unsure<T>(m1, m2));
            if (live && !__builtin_amdgcn_inverse_ballot_w64(unsure))
                store_late(id | (uint32_t)j, x, y, (int)(m1 & 255u));
            if (unsure == 0)  // wave-uniform
                continue;
            xy = word_of(x, y);
        } else {
            break;
        }
#pragma unroll 1
        for (int s = 0; s < GRID_SUB; ++s) {
            const uint64_t lanes = unsure & __builtin_amdgcn_ballot_w64(j == s);
            if (lanes == 0)
                continue;
            const int n = (int)((n_unsure >> (8 * s)) & 255u), total = n + __builtin_popcountll(lanes);
            // The new ones move to the lanes from n on, cyclically, and the other lanes' values to the rest.
            const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
            const int to = 4 * (63 & (__builtin_amdgcn_inverse_ballot_w64(lanes) ? n + below : total + lane - below));
            const uint32_t old_id = pq_grid_pick(s, unsure_id[0], unsure_id[1], unsure_id[2], unsure_id[3]);
            const uint32_t new_id = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)id);
            uint32_t old_xy = 0, new_xy = 0;
            if constexpr (WITH) {
                old_xy = pq_grid_pick(s, unsure_xy[0], unsure_xy[1], unsure_xy[2], unsure_xy[3]);
                new_xy = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)xy);
            }
            // together; 64 are decided, and the rest of the new ones then stands in lanes 0 .. total - 65
            const uint32_t now_id = lane < n ? old_id : new_id, now_xy = lane < n ? old_xy : new_xy;
            const bool full = total >= 64;
            const uint32_t kept_id = full ? new_id : now_id, kept_xy = full ? new_xy : now_xy;
            n_unsure = (n_unsure & ~(255u << (8 * s))) | (uint32_t)(full ? total - 64 : total) << (8 * s);
#pragma unroll
            for (int r = 0; r < GRID_SUB; ++r) {
                unsure_id[r] = s == r ? kept_id : unsure_id[r];
                if constexpr (WITH)
                    unsure_xy[r] = s == r ? kept_xy : unsure_xy[r];
            }
            if (full)
                decide(s, now_id | (uint32_t)s, now_xy, true);
        }
    }

    // What is left of the unsure tokens, the 16 wavefronts' together, in the place of the lists: every wavefront has 64 entries
    // of each subspace's pool, which nothing reads any more.
    static_assert(GRID_POOL * 4 >= GRID_WAVES * 64 * 8, "the place of the lists");
    typedef typename std::conditional<WITH, uint2, uint32_t>::type left_over;
    uint32_t *const counts = (uint32_t *)&queue[0];
    if constexpr (FOUR != 0)  // other wavefronts store some of this one's codes again
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int j = 0; j < GRID_SUB; ++j) {
        left_over &entry = ((left_over *)grids.pool[j])[64 * wave + lane];
        if constexpr (WITH)
            entry = make_uint2(unsure_id[j], unsure_xy[j]);
        else
            entry = unsure_id[j];
    }
    if (lane == 0)
        counts[wave] = n_unsure;
    __syncthreads();
    // lane 16 j + w: how many of subspace j wavefronts 0 .. w have
    int end = (int)(counts[lane & (GRID_WAVES - 1)] >> (8 * (lane >> 4)) & 255u);
    static_assert(GRID_WAVES == 16 && GRID_SUB == 4, "a row of 16 lanes per subspace");
    end += __builtin_amdgcn_update_dpp(0, end, 0x111, 0xf, 0xf, true);  // (row_shr: 0 from outside of the row)
    end += __builtin_amdgcn_update_dpp(0, end, 0x112, 0xf, 0xf, true);
    end += __builtin_amdgcn_update_dpp(0, end, 0x114, 0xf, 0xf, true);
    end += __builtin_amdgcn_update_dpp(0, end, 0x118, 0xf, 0xf, true);
    int batch = wave;  // of 64, over the subspaces in turn
#pragma unroll 1
    for (int j = 0; j < GRID_SUB; ++j) {
        const int total = __builtin_amdgcn_readlane(end, 16 * j + GRID_WAVES - 1);
        for (; 64 * batch < total; batch += GRID_WAVES) {
            const int t = 64 * batch + lane;
            const bool live = t < total;
            const int k = live ? t : 64 * batch;
            int of = 0, start = 0;
#pragma unroll
            for (int w = 0; w < GRID_WAVES - 1; ++w) {
                const int e = __builtin_amdgcn_readlane(end, 16 * j + w);
                of += k >= e ? 1 : 0;
                start = k >= e ? e : start;
            }
            const left_over entry = ((const left_over *)grids.pool[j])[64 * of + k - start];
            if constexpr (WITH)
                decide(j, entry.x | (uint32_t)j, entry.y, live);
            else
                decide(j, entry | (uint32_t)j, 0u, live);
        }
        batch -= (total + 63) >> 6;
    }
}

// In how many slices the tokens of a head (groups: workgroups per slice; chunks: 64-token chunks that all slices together
// walk) go through grid workgroups; 0: the filter, which walks filter_chunks, does better.  Modelled: a workgroup, which fills
// a compute unit, takes 74 us to build and 0.18 us per chunk; through the filter a chunk of 4 subspaces takes 0.72 us of a
// compute unit.  Measured on normal data, 256 compute units: fp16 encode 66 and 0.18, filter 0.78; fp32 encode 65 and 0.27,
// 0.94; k-means 78 and 0.14, 0.85.  So the model is on the filter's side for all three, and data that the grids serve less well
// still gain at the line (32 heads x 9000 tokens or samples, us, grids / filter, the three in turn: normal 364 / 440, 410 /
// 530, 198 / 267; Laplace's distribution 411 / 441, 437 / 526, 219 / 266; channel scales 0.5 .. 4 444 / 458 and 248 / 275).
// kept: the grids are there (pq_encode_grid_kernel), a workgroup takes some 9 us to start, fetch them and end.  Grids / filter,
// fp16, whole appends with the length reset: 32 heads, 500 tokens 45 / 37 us, 1000 52 / 61, 2000 63 / 109, 8000 127 / 383; 8
// heads, 500 tokens 14.8 / 15.3, 1000 15.6 / 22.7, 4000 24 / 60; 4 heads in two slices, 1000 tokens 14.3 / 15.2, 4000 18.8 / 36.5;
// fp32, 32 heads, 500 tokens 48 / 45, 1000 55 / 70, 4000 93 / 230.  price: the mean
// pq_grid_price_of of the codebooks, once it is known.
inline int pq_grid_slices(const int64_t chunks, const int64_t filter_chunks, const int64_t groups, const int n_cu, const bool kept = false,
                          const pq_grid_price price = {18, 72})
{
    int64_t best = filter_chunks * groups * price.filter / n_cu;  // 10 ns
    const int64_t fixed = kept ? 900 : 7400;
    int slices = 0;
    // (no number of slices takes less than this: appends of some tens of tokens are spared the walk below, 0.1 us)
    if (best <= (groups + n_cu - 1) / n_cu * (fixed + price.grid))
        return 0;
    for (int s = 1; s <= 32; ++s) {
        const int64_t rounds = (groups * s + n_cu - 1) / n_cu;
        const int64_t time = rounds * (fixed + (chunks + s - 1) / s * price.grid);
        // (chunk numbers of a slice and workgroup numbers have their limits)
        if (time < best && chunks / s < (1 << 20) && groups * s < (1 << 24)) {
            best = time;
            slices = s;
        }
    }
    return slices;
}

}  // namespace
