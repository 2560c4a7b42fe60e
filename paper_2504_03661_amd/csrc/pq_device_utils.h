// Device-side helpers shared by the decode kernels (gfx950): LDS pointer types, wave-wide
// reductions by DPP, the LDS work counter, the code-block loader.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pq_internal.h"

namespace {

typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

constexpr float NEG_BIG = -1.0e30f;  // "no score yet": finite so that differences stay finite

template <typename T> struct elem;
template <> struct elem<__half> {
    static __device__ float ld(const void *p, int64_t i) { return __half2float(((const __half *)p)[i]); }
};
template <> struct elem<float> {
    static __device__ float ld(const void *p, int64_t i) { return ((const float *)p)[i]; }
};

template <int CTRL> __device__ inline float dpp_move(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

// maximum over the 64 lanes, same value returned to every lane (wave-uniform)
__device__ inline float wave_max(float x)
{
    x = fmaxf(x, dpp_move<0xB1>(x));   // quad_perm [1,0,3,2]
    x = fmaxf(x, dpp_move<0x4E>(x));   // quad_perm [2,3,0,1]
    x = fmaxf(x, dpp_move<0x141>(x));  // row_half_mirror
    x = fmaxf(x, dpp_move<0x140>(x));  // row_mirror
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

// sum over the 64 lanes in a fixed order, wave-uniform result
__device__ inline float wave_sum(float x)
{
    x += dpp_move<0xB1>(x);
    x += dpp_move<0x4E>(x);
    x += dpp_move<0x141>(x);
    x += dpp_move<0x140>(x);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
    return (r0 + r1) + (r2 + r3);
}

// Zero in a vector register, opaque to the compiler: added to a wave-uniform index it keeps a
// load a vector load that can stay in flight, where the compiler would otherwise issue a scalar
// read and wait for it at once.
__device__ inline int lane_zero()
{
    int z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}

// ---------------------------------------------------------------------------------------------------
// Exchange of split partials between the workgroups of one output row.  Every workgroup of the row
//   1. publishes its partial with relaxed atomic stores at agent scope: on gfx942 / gfx950 the compiler emits
//      these as write-through stores (sc1) that are performed in the memory all XCDs share, not left dirty in
//      the XCD's own L2;
//   2. waits until those stores have completed (s_waitcnt vmcnt(0): the counter falls only when the memory
//      system has acknowledged the store at the scope it was issued with);
//   3. takes a ticket: a relaxed atomic add at agent scope on the row's counter — all of a row's tickets are
//      totally ordered on that one location;
// and the workgroup that draws the last ticket
//   4. loads all partials with relaxed atomic loads at agent scope (sc1: not served from a line its own L2
//      might hold), issued after its ticket has returned, merges them and puts the counter back to zero.
// Steps 2 and 4 stand where a release fence and an acquire fence would stand.  The code sequences the AMDGPU
// backend documents for those fences at agent scope are "write back the L2, then s_waitcnt vmcnt(0)" and
// "invalidate the caches"; the write-back and the invalidate exist for earlier plain stores and later plain
// loads, which may live in the non-coherent L2 — every store and load of this exchange is itself an
// agent-scope atomic access and bypasses that cache, so only the wait remains.  (The fences were measured:
// about 1.8 us per workgroup for the release, 3 us with the acquire, on a 33 us kernel.)  The counter is put
// back by the one workgroup that has seen every other ticket of the launch; nobody touches it again before
// the next launch, which the kernel boundary orders after this one: calls on a context must be
// stream-ordered.
// ---------------------------------------------------------------------------------------------------
__device__ inline void publish(float *p, float x, float y)
{
    const uint64_t bits = (uint64_t)__float_as_uint(x) | ((uint64_t)__float_as_uint(y) << 32);
    __hip_atomic_store((uint64_t *)p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// all stores this wavefront has issued are complete
__device__ inline void publish_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ inline float2 fetch(const float *p)
{
    const uint64_t bits = __hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)bits), __uint_as_float((uint32_t)(bits >> 32)));
}

__device__ inline void ticket_reset(unsigned int *ticket)
{
    __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline uint32_t comp(const uint4 &v, int r)
{
    return r == 0 ? v.x : r == 1 ? v.y : r == 2 ? v.z : v.w;
}

// Takes the next unowned block of the workgroup's split from a counter in LDS.  One lane adds
// 1; the execution mask is narrowed to that lane inside the assembly block, so no branch
// appears in the scan loop (the compiler's wait-count analysis turns conservative at
// control-flow joins) and the atomic unit serves one lane, not sixty-four on one address.
__device__ inline int lds_grab(uint32_t lds_addr)
{
    uint32_t r;
    uint64_t saved_exec;
    const uint32_t one = 1;
    asm volatile("s_mov_b64 %1, exec\n\t"
                 "s_mov_b64 exec, 1\n\t"
                 "ds_add_rtn_u32 %0, %2, %3\n\t"
                 "s_mov_b64 exec, %1\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r), "=&s"(saved_exec)
                 : "v"(lds_addr), "v"(one)
                 : "memory");
    return __builtin_amdgcn_readfirstlane((int)r);
}


// Which (unit, split) a workgroup owns; unit = a (sequence, head or head group).  Workgroups are dealt round-robin
// to the 8 XCDs; they are un-dealt so that all splits of a unit — and neighbouring units: the heads of a KV group,
// the same KV head of other sequences — sit on one XCD and share its L2.  Where every XCD gets whole units, its
// workgroups are numbered SPLIT-major: the first splits of all its units come first.  With unit-major numbering the
// live workgroups of an oversubscribed grid whose surplus splits leave at once (8 launched splits, 1 live) sit 8
// apart, and the dispatcher, which deals consecutive workgroups to the shader engines in turn, put them all on one
// engine's compute units: 8 x 32 heads x 32K with 8 launched splits took 483 us instead of 165.
//   BY: divides by n_units / 8 where 8 divides n_units, else by S
template <typename BY>
__device__ inline void unit_and_split(uint32_t bid, uint32_t n_units, uint32_t S, const BY &by, uint32_t &unit, uint32_t &split)
{
    const uint32_t xcd = bid & 7u;
    if ((n_units & 7u) == 0) {
        const uint32_t per_xcd = n_units >> 3, local = bid >> 3;
        split = by(local, per_xcd);
        uint32_t j = local - split * per_xcd;
        // ... and where the XCD's unit count is a power of two, the units are visited in a scrambled order (low 3
        // bits XOR the next 3): the long sequences of a ragged batch sit at a fixed stride in the unit numbering
        // (unit = head x batch + sequence), which met the same engine every time
        if (per_xcd >= 16u && (per_xcd & (per_xcd - 1u)) == 0u)
            j ^= (j >> 3) & 7u;
        unit = xcd * per_xcd + j;
    } else {
        // XCD x runs workgroups x, x + 8, ..: grid / 8 of them, one more on the first grid % 8.  Any grid can be un-dealt:
        // left as dealt where 8 does not divide it, each of a head's workgroups fetched the codebooks from memory for
        // itself (28 heads: 9 workgroups each over 16 sequences of 1000 tokens 22.3 us, now 19.0; 9 splits of one
        // sequence of 10000 tokens 15.8 us, now 12.6).  Only workgroups with a sequence each stay as dealt: they share
        // less, and neighbouring sequences of a ragged batch are better spread (5 heads, 65 sequences of 500 .. 30000
        // tokens: 149 us, un-dealt 162).
        const uint32_t grid = n_units * S, extra = grid & 7u;
        const uint32_t logical = S == 1u ? bid : xcd * (grid >> 3) + (xcd < extra ? xcd : extra) + (bid >> 3);
        unit = by(logical, S);
        split = logical - unit * S;
    }
}

__device__ inline void unit_and_split(uint32_t bid, uint32_t n_units, uint32_t S, uint32_t &unit, uint32_t &split)
{
    unit_and_split(bid, n_units, S, [](uint32_t x, uint32_t d) { return x / d; }, unit, split);
}

// The numberings of a batch divide by multiplying (pq_batch_divisors, set by the host): the compiler divides uniform
// numbers on the vector ALU, some 25 instructions of every wavefront before its first load — two or three such divisions
// cost a workgroup of 16 wavefronts 0.4 us.
__device__ inline uint32_t divided(uint32_t x, uint32_t by) { return by != 0u ? __umulhi(x, by) : x; }

// BATCH_WALK: unit = query head (one per KV head), split = workgroup of it
__device__ inline void unit_and_walker(uint32_t bid, uint32_t n_units, uint32_t S, const pq_batch_divisors &d, uint32_t &unit,
                                       uint32_t &walker)
{
    unit_and_split(bid, n_units, S, [&](uint32_t x, uint32_t) { return divided(x, d.unit); }, unit, walker);
}

// BATCH_DEAL: job `job` of query head (or group of them) `sub` of the n per KV head.
// The n workgroups that read the same codes — the same job of each query head — are neighbours and share an XCD's L2, as
// the query heads of a sequence are in the other numbering.  (With a head's jobs in a row they were S workgroups apart:
// 8 query heads of one KV head, 31 sequences of 4K tokens, fp32, 1.37 times the time of splits per sequence, 1.01 so;
// 12 of 30K, fp16, 1.06 and 0.98 times.)
__device__ inline void unit_and_job(uint32_t bid, uint32_t Hkv, uint32_t S, uint32_t n, const pq_batch_divisors &d, uint32_t &hkv,
                                    uint32_t &sub, uint32_t &job)
{
    uint32_t both;
    unit_and_split(bid, Hkv, S * n, [&](uint32_t x, uint32_t) { return divided(x, d.unit); }, hkv, both);
    job = divided(both, d.sub);
    sub = both - job * n;
}

// BATCH_ORDER: one workgroup per sequence and query head (or group of them, n per KV head).  The (place, KV head) pairs,
// place-major — the longest sequences of all heads first — are dealt to the XCDs one by one, and an XCD runs the n
// workgroups of a pair, which read the same codes, in a row: 8 / gcd(8, Hkv) XCDs share a head, each has long and short
// sequences.  (Head-major, a stretch of the units per XCD: one XCD had all the long sequences of a head that several
// shared — 8 query heads of one KV head, fp32, 40 sequences of 1000 .. 10000 tokens 94 us, unranked 68, now 50 — and the
// last heads' longest sequences began in the second round: 28 heads of 32 subspaces, 16 sequences 46 -> 39.)
__device__ inline void unit_and_place(uint32_t bid, uint32_t B, uint32_t Hkv, uint32_t n, const pq_batch_divisors &d, uint32_t &hkv,
                                      uint32_t &sub, uint32_t &place)
{
    const uint32_t pairs = B * Hkv, whole = (pairs & ~7u) * n;  // the last pairs % 8 as dealt
    const bool row = bid < whole;
    const uint32_t at = row ? bid >> 3 : bid - whole, step = divided(at, d.sub);
    sub = at - step * n;
    const uint32_t pair = row ? step * 8u + (bid & 7u) : (pairs & ~7u) + step;
    place = divided(pair, d.unit);
    hkv = pair - place * Hkv;
}

// Sum over the batch of (cached tokens + recent rows), each clamped like the sequence's own lengths: lane l adds
// sequences l, l + 64, ...; the loads go out with the workgroup's own lengths.  Only batches need it (the live
// split count of a sequence follows its share of the batch's work).
// (a float: 64 sequences of 2^24 tokens already exceed an int, and every workgroup adds in the same order)
template <typename A> __device__ inline float batch_work_lane(const A &a, bool has_recent, int lane)
{
    float w = 0.f;
    for (int b2 = lane; b2 < a.B; b2 += 64) {
        int n2 = a.ctx_len[b2];
        n2 = n2 < 0 ? 0 : (n2 > a.max_context ? a.max_context : n2);
        int r2 = has_recent ? a.recent_len[b2] : 0;
        r2 = r2 < 0 ? 0 : (r2 > a.max_recent ? a.max_recent : r2);
        w += (float)(n2 + r2);
    }
    return w;
}

// The live splits of a sequence in a batch: no more than its share of the compute units — n_cu x (its work) /
// (workgroups per split x the batch's work) — so that in an oversubscribed grid (explicit n_splits on a large
// batch: a cache that must serve ragged batches) the splits go to the long sequences and a batch of equal lengths
// runs one split per sequence, as if none had been asked for.  Every workgroup of the row computes the same number
// from the same lengths.
template <typename A> __device__ inline uint32_t live_split_cap(const A &a, int units, int own_work, float w_lane)
{
    float total = w_lane;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        total += __shfl_xor(total, o);
    total = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(total)));
    const float share = (float)a.n_cu * (float)own_work / ((float)units * (total > 0.f ? total : 1.f));
    return share >= 1.f ? (share < 64.f ? (uint32_t)share : 64u) : 1u;
}

// ---------------------------------------------------------------------------------------------------
// Which workgroups a batch's sequences get ("0 = choose" splits, 2..64 sequences); every workgroup reads all lengths and
// works it out in the same way.  Work is counted in 64-token blocks and 16 recent rows.
//   BATCH_DEAL   (the head's share of the compute units is larger than the batch: that many workgroups per head)
//       sequence b gets ceil(work / T) of them, no more than pay, T the smallest trial size whose sum fits, so that
//       no workgroup has much more than its share, whatever the lengths (a fixed number of splits per sequence leaves the longest sequence's
//       workgroups the last ones by far: 32 heads, three sequences of 30000, 15256 and 512 tokens 59.6 -> 39.1 us; 32
//       query / 8 KV heads, eight sequences of 2.5K .. 20K: 33 -> 28 us).
//   BATCH_ORDER  (other kernels: one workgroup per sequence and head, more than one round of them but at most two) the
//       longest sequences come first: a long one that starts in the second round would run alone (32 query / 8 KV heads,
//       40 sequences of 200 .. 8000: 61 -> 49 us).  Ranking 64 lengths and fetching the query behind them costs a workgroup
//       1.5 us, so lengths within a quarter of the first one's stay in their order, and so does a batch without a sequence
//       of 20 blocks (63 sequences, 32 query / 8 KV heads, of 30 .. 200 tokens 20.0 us, 16.5 unranked; of 300 .. 1000 27.2
//       and 25.5; of 200 .. 1500 29.5 and 28.3, but 7 of 56 heads 16.9 and 18.3); with more rounds, where the last one
//       matters less, nothing is ranked (32 heads, 64 sequences of 3000 .. 4096: 181 us, ranked 190; of 97 .. 4001: 133 us,
//       ranked 134).
//   BATCH_WALK   (the per-head kernel, more sequences than the head's share of the compute units) as many workgroups per
//       head as the chip holds at once; workgroup w walks whole sequences, those of rank w, 2 S - 1 - w, 2 S + w, ... by
//       length.  What a workgroup pays before its first block — 4 us: launch, lengths, 128 KiB of codebook images through
//       the compute unit's address pipeline — it pays once; the next sequence needs its query, the key codebook again
//       (L2) and a new table, requested before the wavefronts' merge of the previous one (32 heads, 64 sequences of 97
//       .. 4001 tokens: 131.5 -> 118.5 us; 20 of 700 .. 8000: 84 -> 69; 16 of them 63 -> 53.5; 64 of 4096: 201 -> 193).
//   BATCH_NONE   splits per sequence as launched (one sequence, splits asked for, more than 64 sequences)
// ---------------------------------------------------------------------------------------------------
enum { BATCH_NONE = 0, BATCH_DEAL = 1, BATCH_ORDER = 2, BATCH_WALK = 3 };

struct batch_job {
    int b, split, S;  // sequence, split, splits of it (split >= S: nothing to do)
};

template <int CTRL, int ROWS> __device__ inline uint32_t dpp_add(uint32_t x)
{
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}

// running sum over the lanes (lane l: lanes 0 .. l)
__device__ inline uint32_t wave_scan(uint32_t x)
{
    x = dpp_add<0x111, 0xf>(x);  // row_shr:1
    x = dpp_add<0x112, 0xf>(x);  // row_shr:2
    x = dpp_add<0x114, 0xf>(x);  // row_shr:4
    x = dpp_add<0x118, 0xf>(x);  // row_shr:8
    x = dpp_add<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    x = dpp_add<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
    return x;
}

// BATCH_DEAL: the sequence that job j has if all lengths are equal (its q is requested before the lengths are there)
__device__ inline int batch_guess(int B, const pq_batch_divisors &d, int j)
{
    const int b = (int)divided((uint32_t)j, d.even);
    return b < B ? b : B - 1;
}

__device__ inline uint32_t batch_work(uint32_t n, uint32_t r) { return ((n + 63u) >> 6) + ((r + 15u) >> 4); }

// BATCH_DEAL: job j of `jobs` (n, r: clamped lengths of sequence `lane`; lanes beyond the batch: anything).  WHOLE: blocks
// below which a sequence has one workgroup; AT_ONCE: partials that the kernel's merge loads in one round trip; ROOT,
// ROWS: see below.
template <int WHOLE, int AT_ONCE, int ROOT, int ROWS>
__device__ inline batch_job batch_deal(int B, int jobs, const pq_batch_divisors &d, int j, uint32_t n, uint32_t r, int lane)
{
    const bool in = lane < B;
    const uint32_t work = in ? batch_work(n, r) : 0u;
    // The splits that pay.  Exchanging partials costs 1 .. 3 us and the merge another round trip for every AT_ONCE of them,
    // a block of the scan 0.15 us.  Measured on one sequence: 16 heads of 64 subspaces, 12 blocks 7.5 us, split in two 7.8,
    // 16 blocks 8.6 and 8.0 (32 subspaces, 16 wavefronts: 8.9 and 9.4, 24 blocks 9.6 and 9.3; 32 query / 8 KV heads, 12
    // blocks 10.7 and 12.0, 16 blocks in four 11.8 and 11.3); the best number from there about ROOT / 4 times the square root of
    // the blocks, ROOT = 6 (4 heads: 8 splits of 2K tokens 7.4 us; 16 of 8K 8.5, 32 10.1; 24 of 16K 10.2, 64 13.7; 48 of 64K
    // 15.4, 64 16.1), 3 for the per-head kernels of 16 wavefronts (32 subspaces: 6 of 8K 10.6, 16 11.9; 12 of 16K 12.2).
    const uint32_t root = (uint32_t)(0.25f * (float)ROOT * __builtin_amdgcn_sqrtf((float)work));
    const uint32_t paying = root < (uint32_t)AT_ONCE ? (uint32_t)AT_ONCE : root < PQ_MAX_SPLITS ? root : PQ_MAX_SPLITS;
    // 16 recent rows count as a block, and from the ROWS-th on as three: 3 sequences of 300 tokens and up to 128 rows, 32 query
    // / 8 KV heads, whole 14.9 us, in four 11.9; per head 5 of 200 and up to 128 whole 8.1, cut 9.4, up to 200 whole 10.9, cut 9.8
    const uint32_t rows = in ? (r + 15u) >> 4 : 0u;
    const uint32_t long_rows = rows > (uint32_t)ROWS ? 2u * (rows - (uint32_t)ROWS) : 0u;
    const uint32_t most = work + long_rows < (uint32_t)WHOLE ? 1u : paying;
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)work);
    if (__builtin_amdgcn_ballot_w64(most > 1u) == 0 ||
        __builtin_amdgcn_ballot_w64(in && (work > w0 + w0 / 8u || work < w0 - w0 / 8u)) == 0) {
        // nothing to cut, or lengths within an eighth: the same number of jobs for all, at least 4 blocks each
        const int b = batch_guess(B, d, j);
        const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane((int)work, b), by_4 = (mine + 3u) >> 2;
        uint32_t splits = (uint32_t)__builtin_amdgcn_readlane((int)most, b);
        splits = splits < d.even_jobs ? splits : d.even_jobs;
        splits = splits > 1u && splits > by_4 ? by_4 : splits;
        return {b, j - b * (int)d.even_jobs, (int)splits};
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(work), 63);
    // T is 2^(i / 10.5) x the even share (at least 4 blocks), i the first of 0 .. 63 whose sum fits: steps of 7 %, the last
    // one 64 shares, which fits (jobs / 64 workgroups beyond one per sequence at most).  In floats, the same in every
    // workgroup.
    const float share = (float)total / (float)jobs;
    const float least = share > 4.f ? share : 4.f;
    const float beyond = (float)(work > 0u ? work - 1u : 0u);
    const auto size_inv = [&](int i) { return __builtin_amdgcn_rcpf(least * __builtin_amdgcn_exp2f((float)i * (6.0f / 63.0f))); };
    const auto splits_of = [](float more, uint32_t limit, float inv) {
        const uint32_t splits = 1u + (uint32_t)(more * inv);
        return splits < limit ? splits : limit;
    };
    int trial = 0;
    if (B <= 24) {  // a lane per trial, all sequences in turn
        const float inv = size_inv(lane);
        uint32_t sum = 0;
#pragma unroll 4
        for (int b = 0; b < B; ++b)
            sum += splits_of(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(beyond), b)),
                             (uint32_t)__builtin_amdgcn_readlane((int)most, b), inv);
        const uint64_t fits = __builtin_amdgcn_ballot_w64(sum <= (uint32_t)jobs) | 1ull << 63;
        trial = __builtin_ctzll(fits);
    } else {
        // a lane per sequence, three rounds of three trials whose latencies overlap, two sums (each at most 64 x 64) in one
        // scan (4 heads x 1000 tokens, against fixed splits: 63 sequences 1.19 with the loop, 1.08 so; 10 sequences 1.03, 1.09)
#pragma unroll
        for (int step = 16; step > 0; step >>= 2) {
            const auto at = [&](int i) { return in ? splits_of(beyond, most, size_inv(trial + i * step - 1)) : 0u; };
            const uint32_t sums = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(at(1) | at(2) << 16), 63);
            const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(at(3)), 63);
            const uint32_t fit = (uint32_t)jobs;
            trial += ((sums & 0xffffu) > fit ? step : 0) + ((sums >> 16) > fit ? step : 0) + (last > fit ? step : 0);
        }
    }
    const uint32_t mine = in ? splits_of(beyond, most, size_inv(trial)) : 0u;
    const uint32_t upto = wave_scan(mine);
    const uint32_t first = in ? upto - mine : ~0u;
    const int b = __builtin_popcountll(__builtin_amdgcn_ballot_w64(first <= (uint32_t)j)) - 1;
    return {b, j - __builtin_amdgcn_readlane((int)first, b), __builtin_amdgcn_readlane((int)mine, b)};
}

// Rank of sequence `lane` by length, the longest first, equal ones by their number; lengths within a quarter of the
// first one's are ranked by number alone, and so are those of a batch without a sequence of SHORT blocks.  Lanes beyond the
// batch: 64.
template <uint32_t SHORT>
__device__ inline int batch_rank(int B, uint32_t n, uint32_t r, int lane)
{
    const bool in = lane < B;
    const uint32_t work = in ? batch_work(n, r) : 0u;  // below 2^21
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)work);
    if (__builtin_amdgcn_ballot_w64(in && (work > w0 + w0 / 4u || work < w0 - w0 / 4u)) == 0 ||
        (SHORT > 0 && __builtin_amdgcn_ballot_w64(work >= SHORT) == 0))
        return in ? lane : 64;
    const uint32_t key = in ? (work << 6) | (uint32_t)(63 - lane) : 0u;
    int rank = 0;
    for (int b = 0; b < B; ++b)
        rank += (uint32_t)__builtin_amdgcn_readlane((int)key, b) > key ? 1 : 0;
    return in ? rank : 64;
}

__device__ inline int batch_of_rank(int rank, int j) { return (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(rank == j)); }

// 16 code bytes of one lane.  Codes that are read once per launch are loaded with the
// non-temporal hint: the stream then does not displace the tables and each other's lines in L2
// and the memory-side cache, and HBM delivers markedly more (measured on the 8 x 32 heads x 32K
// workload: 192 us with plain loads, 164 us with the hint; a kernel that only reads shows the same).
template <bool READ_ONCE> __device__ inline uint4 load_codes(const u32x4 *p)
{
    const u32x4 t = READ_ONCE ? __builtin_nontemporal_load(p) : *p;
    return make_uint4(t.x, t.y, t.z, t.w);
}

// (d, c) <- the smaller of (d, c) and (od, oc) in the order (distance, index)
__device__ inline void argmin_take(double &d, int &c, const double od, const int oc)
{
    const bool take = od < d || (od == d && oc < c);
    d = take ? od : d;
    c = take ? oc : c;
}

template <int CTRL> __device__ inline void argmin_dpp(double &d, int &c)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(d), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(d), CTRL, 0xf, 0xf, true);
    const int oc = __builtin_amdgcn_update_dpp(0, c, CTRL, 0xf, 0xf, true);
    argmin_take(d, c, __hiloint2double(hi, lo), oc);
}

// minimum over the 64 lanes, the same in every lane: lane exchanges inside a row of 16 by DPP (vector-ALU
// speed; a shuffle goes through the LDS crossbar), then the 4 rows' results
__device__ inline void wave_argmin(double &d, int &c)
{
    argmin_dpp<0xB1>(d, c);   // quad_perm [1,0,3,2]
    argmin_dpp<0x4E>(d, c);   // quad_perm [2,3,0,1]
    argmin_dpp<0x141>(d, c);  // row_half_mirror
    argmin_dpp<0x140>(d, c);  // row_mirror
    double rd[4];
    int rc[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        rd[r] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(d), 16 * r),
                                 __builtin_amdgcn_readlane(__double2loint(d), 16 * r));
        rc[r] = __builtin_amdgcn_readlane(c, 16 * r);
    }
    d = rd[0];
    c = rc[0];
#pragma unroll
    for (int r = 1; r < 4; ++r)
        argmin_take(d, c, rd[r], rc[r]);
}


}  // namespace
