// Scan for batches whose queries hardly share filters (levels with thresholds in force).
//
// The wavefront dot-product scan gathers one item row per passing pair: at 10 M items x 256 bytes and 256
// filters that pass 5 % each, 2 G 16-byte gathers, 64 cache lines to an instruction.  Here a wavefront holds
// the rows of 64 items in registers and multiplies them with all queries by MFMA, whether a filter
// passes them or not; the filters decide which scores count.  That costs the same for every selectivity, so a
// wavefront whose filters pass few pairs gathers after all.
//
// Eight wavefronts share the queries and the tables in LDS and nothing else between set-up and report: each draws
// units of 64 items from a counter, so that one forms masks or waits for rows while another multiplies.  A unit's
// words of the index (the rows that some filter names, m <= kOwnRows) come to LDS with loads requested a unit
// ahead, and the mask words of all filters are formed there (a filter's rows fetched one by one from memory took
// longer than the products).  A mask word is what the unit needs for one query: lane l of a product's result holds query l % 32,
// and 16 items of each of the two halves of 32.  The bound is part of the product (the slices of st_bound.h), so that the
// signs of the results are the tests: one instruction to a pair takes them to the bits of its item, where the
// mask word is.  (Where bounds are larger than digits can say, the accumulators start at a part of them: one branch to a block.  3 M x
// 256, 256 queries, rows with a mean cosine of 0.5: 599 -> 345 us a call; 472 with a multiply-add for every pair.)  Pairs left are queued with their results; dot product, exact score, key and
// threshold test follow where the queue is emptied, 64 pairs at a time.  A block's operands are read while the results of the one
// before are tested, and an operand serves both halves.
// The queries lie in LDS with 16 bytes of padding a row (an odd number of 16-byte pieces: no bank conflicts).
//
// 10 M x 256 bytes, 256 queries, 161 filters (5 % each), K = 500: the level after the first takes 0.82 ms in a long series of
// calls (0.81 to 1.17 in a run's first sixty, 0.87 on average).  With 213 of the queries, a call took 1.31 ms with a multiply-add for every pair, operands read for
// each half, queued lanes of 16 results and segments of 512 items tied to a workgroup, and 1.01 so; gathering took 4.5 in this kernel's place.
// A unit of seven blocks takes a wavefront 21,500 cycles: 13,500 in products
// and tests (4,200 is what the products alone need, and two wavefronts share the matrix unit), 4,000
// in masks, 1,200 and 2,000 around the first and the last block.
//
// A unit whose filters pass few pairs hands them to a list that goes from unit to unit until 64 are there, and
// whose rows come several lanes to a row (a lane to a row touches 64 lines with every load: 10,000 cycles to a round at
// d = 256).  Calls on 3 M x 256, 64 queries that pass 0.5 %: 125 -> 99 us.  It takes the place of the gathering scan whatever
// the filters pass, which the host cannot know.
#pragma once
#include "st_search_kernels.h"

namespace st {

constexpr int kOwnThreads = 512;
constexpr int kOwnSeg = 512;            // items of a segment
constexpr int kOwnWords = kOwnSeg / 64; // one mask word per wavefront
constexpr int kOwnCols = 256;           // queries resident at a time (one row of the grid), at most
constexpr int kOwnRows = 512;           // signature rows of the index, at most
// Items of a level, at least: two segments to each of the workgroups that are resident.  (Whether the candidate
// regions have room for segments of this size is the plan's to say: level_takes_segments.)
constexpr int64_t kOwnMinItems = 512 * kOwnSeg;
constexpr int kOwnAllRows = 64;         // an index of no more rows is staged whole
constexpr int kOwnQueue = 64;           // pairs of a wavefront that wait for the exact test
constexpr int kOwnSlots = 4;            // regions of a workgroup, at most (the host launches that many workgroups)
constexpr int kOwnRowRefs = 6144;       // rows all filters name together, at most
static_assert(kOwnWords == kOwnThreads / 64, "a word per wavefront");

constexpr int own_row_bytes(int d) { return d + kSliceBytes + 16; }  // of a query in LDS
constexpr int own_grid_rows(int n_q) { return (n_q + kOwnCols - 1) / kOwnCols; }
constexpr int own_cols(int n_q) { return ((n_q + own_grid_rows(n_q) - 1) / own_grid_rows(n_q) + 31) / 32 * 32; }  // of each row
// A wavefront whose filters pass no more pairs than own_few of its 64 items gathers the pairs' rows instead of multiplying all;
// one that multiplies has the next rows already, and goes on down to own_stay.
// Up to 64 queries the line is 64:
//   entering at 16 or 32: 3 M x 256, 64 queries at 0.5 %: 100 -> 200 us
//   leaving at 64 too: 2 M x 64, 17 at 10 %: 82 -> 86, where units lie below the line now and then; but 2.3 M x 192, 41 at 2 %,
//   units on either side of it: 129 -> 121
// With more queries all products take longer, and it is 112, as many as the list has room for. 64 -> 112:
//   3.4 M x 256, 117 at 1 %: 257 -> 198;  3.5 M x 256, 259 at 1 %: 377 -> 327;  2 M x 128, 250 at 0.5 %: 180 -> 139
constexpr int own_few(int cols) { return cols <= 64 ? 64 : 112; }
constexpr int own_stay(int cols) { return own_few(cols) / 2; }
constexpr int kOwnPairs = 64 + own_few(kOwnCols);  // of a list: what is left of a round, and a unit's
// (a filter's rows take whole multiples of four entries: three more to a filter of the resident queries, at most)
constexpr size_t own_lds_bytes(int n_q, int d, int m_bits)
{
    const size_t c = own_cols(n_q);
    return c * own_row_bytes(d) + c * kOwnWords * 8 + (size_t)m_bits * kOwnWords * 8 + kOwnWords * kOwnPairs * 8 + c * 8 +
           (kOwnRowRefs + c * 3 + 10) / 8 * 16 + 64 + c * (4 * (2 + kOwnSlots) + 2 * 3) + kOwnRows * 2 + kOwnRows / 8;
}
static_assert(own_lds_bytes(kOwnCols, 256, kOwnRows) <= 160 * 1024, "LDS of a compute unit");

typedef int own_i4 __attribute__((ext_vector_type(4)));
typedef int own_i16 __attribute__((ext_vector_type(16)));

// LDS exchange of the workgroup's set-up.
__device__ inline void own_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The words of a corpus that the first level's sample left: their numbers and back.
struct SampleWords {
    uint32_t stride, taken, rest, segs, per;  // words from one segment of the sample to the next, in it, between them; segments; 2^32 / rest, less up to 2
    __device__ explicit SampleWords(const ScanParams& p)
        : stride((uint32_t)(p.samp_stride_items >> 6)), taken((uint32_t)p.samp_seg_items >> 6), rest(max(stride - taken, 1u)), segs((uint32_t)p.samp_segs),
          per(0xFFFFFFFFu / rest)
    {
    }
    __device__ uint32_t others_before(uint32_t word) const
    {
        const uint32_t i = word / stride, in = word - i * stride;
        return word - (i < segs ? i * taken + min(in, taken) : segs * taken);
    }
    __device__ uint32_t other(uint32_t no) const
    {
        uint32_t i = __umulhi(no, per);  // (the quotient or one less: below 2^25)
        if (no - i * rest >= rest) ++i;
        return no + min(i + 1u, segs) * taken;
    }
};

// A value that the compiler takes for a new one: what is formed from it is formed here, and no register holds it from
// outside a loop on.  (A condition of the lanes is two scalar registers, and some twenty that a unit needs, held over the loop, went to
// lanes of vector registers and back: without them 2 M x 64, 16 queries: 82.0 -> 79.5 us, 4 M x 128, 16: 149.9 -> 148.2.)
template <class V>
__device__ inline V fresh(V v)
{
    asm volatile("" : "+v"(v));
    return v;
}
// ... the same of a value in a scalar register: lanes are compared with it, and no vector register is taken.  (With a fresh
// lane number there was none left at 256 bytes a row, and that form kept its 84 spills: with fresh limits 51; 10 M x 256, 256
// queries: 892 -> 887 us, 2 M x 64, 16: 107.3 -> 105.6, 0.75 M x 96, 211: 136.5 -> 134.9, 4 M x 128, 200: 278 -> 272.)
__device__ inline int fresh_scalar(int v)
{
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
}

// d = 32 * KS.  Grid (workgroups, own_grid_rows(queries)).  One
// workgroup to a compute unit is resident (registers), so that many are launched and each takes several
// regions in turn: the queries and tables are brought to LDS once.
// SAMP: the first level took a sample of the corpus; the other words are numbered, and segments are of these numbers.  (A form of its
// own: what it keeps in scalar registers cost calls with 16 queries 1 to 3.6 %, whose first level is the seed pass and none of a
// sample.  Leaving the sample's words out of segments of the corpus gave some workgroups a segment more: 2 M x 128, 250 queries at
// 0.5 %: 146 -> 156 us.)
template <int KS, bool SAMP>
__global__ __launch_bounds__(kOwnThreads) void scan_own_kernel(ScanParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char own_lds[];
    constexpr int D = 32 * KS, DP = own_row_bytes(D);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    const int n_q = p.grp_q_off[p.n_groups];
    const int cols = own_cols(n_q), c0 = (int)blockIdx.y * cols, n_c = min(n_q - c0, cols);
    const int n_blk = (n_c + 31) & ~31;  // (of these columns the last row of the grid may have fewer)
    unsigned char* at = own_lds;
    int8_t* s_q = reinterpret_cast<int8_t*>(at);                  at += (size_t)cols * DP;          // [cols][DP] rows and their slices
    uint64_t* s_mask = reinterpret_cast<uint64_t*>(at) + (size_t)wv * cols;      at += (size_t)cols * kOwnWords * 8;
    uint64_t* s_idx = reinterpret_cast<uint64_t*>(at) + (size_t)wv * p.m_bits;   at += (size_t)p.m_bits * kOwnWords * 8;
    uint2* s_pairs = reinterpret_cast<uint2*>(at) + (size_t)wv * kOwnPairs;  at += (size_t)kOwnWords * kOwnPairs * 8;  // of a wavefront that gathers
    int4* queue = reinterpret_cast<int4*>(s_pairs);               // ... that multiplies
    static_assert(kOwnQueue * sizeof(int4) <= kOwnPairs * sizeof(uint2) && kOwnPairs * sizeof(uint2) % 16 == 0, "the queue lies where the pairs do");
    uint64_t* s_tau = reinterpret_cast<uint64_t*>(at);            at += (size_t)cols * 8;
    uint16_t* s_refs = reinterpret_cast<uint16_t*>(at);           at += (size_t)(kOwnRowRefs + cols * 3 + 10) / 8 * 16;
    uint32_t* s_max = reinterpret_cast<uint32_t*>(at);            at += 64;  // [8] largest 1 / scale of a wavefront's sample; largest tau / s_q; first filter, last; no bound for some query; next unit
    float* s_sq = reinterpret_cast<float*>(at);                   at += (size_t)cols * 4;
    int32_t* s_query = reinterpret_cast<int32_t*>(at);            at += (size_t)cols * 4;
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(at);            at += (size_t)cols * 4 * kOwnSlots;  // [slots][cols]
    uint16_t* s_r0 = reinterpret_cast<uint16_t*>(at);             at += (size_t)cols * 2;
    uint16_t* s_rn = reinterpret_cast<uint16_t*>(at);             at += (size_t)cols * 2;
    uint16_t* s_u = reinterpret_cast<uint16_t*>(at);              at += (size_t)cols * 2;   // bounds as slices' numbers (kNoBound: none)
    uint16_t* s_named = reinterpret_cast<uint16_t*>(at);          at += (size_t)kOwnRows * 2;
    uint32_t* s_bits = reinterpret_cast<uint32_t*>(at);           // [kOwnRows / 32]
    constexpr int kNoBound = 0xFFFF;
    static_assert(kSliceTop < kNoBound, "a query's number in 16 bits");

    // ---- set-up: the queries, their thresholds, the filters' rows; and a sample of the scales, spread over the level.
    // All chains of loads are begun before the first one is waited for (0.36 M x 96, 16 queries: the call 41.2 -> 40.3 us).
    if (tid < kOwnRows / 32) s_bits[tid] = 0;
    if (tid < 4) s_refs[tid] = 0;  // (columns without rows read these)
    if (tid == 0) {
        s_max[8] = 0;
        s_max[9] = (uint32_t)p.n_groups;
        s_max[10] = s_max[11] = 0;
        s_max[12] = kOwnWords;
    }
    own_barrier();  // (s_max, s_bits)
    // Units of 64 items, drawn by the wavefronts from a counter in LDS (tied to a segment, or to a region at a time, they waited a
    // sixth to a half of the time for the slowest of them).  The words of the level go to the workgroups in rounds, a visit of
    // seg_per_visit segments to each, whose candidates go to its regions in turn; the words behind the last whole round are dealt
    // evenly (as visits they made some workgroups wait for others: 1.65 M x 96, 200 queries: 168.7 -> 151.2 us, 2 M x 64, 16: 79.5 -> 73.7,
    // 10 M x 256, 256: 944 -> 914).
    const int spv = p.seg_per_visit, visit = spv * kOwnWords, wgs = (int)gridDim.x;
    const SampleWords samp(p);
    const int first_word = (int)(SAMP ? samp.others_before((uint32_t)(p.item_begin >> 6)) : (uint32_t)(p.item_begin >> 6));
    const int end_word = (int)(SAMP ? samp.others_before((uint32_t)((p.item_end + 63) >> 6)) : (uint32_t)((p.item_end + 63) >> 6));
    const int slots = (p.groups - (int)blockIdx.x + wgs - 1) / wgs;
    const int n_rounds = (end_word - first_word) / (wgs * visit), last_word = first_word + n_rounds * wgs * visit, dealt = (end_word - last_word + wgs - 1) / wgs;
    const int n_units = n_rounds * visit + dealt;
    const int64_t item_lim = p.item_end < p.n_items ? p.item_end : p.n_items;
    // (first item and region slot of a unit; negative: the workgroups at the end may have fewer)
    const uint32_t per_spv = 0xFFFFFFFFu / (uint32_t)spv + 1u, per_slots = 0xFFFFFFFFu / (uint32_t)slots + 1u;  // (0 for 1)
    auto unit_at = [&](int unit, int& slot) -> int64_t {
        const int t = unit / kOwnWords, round = spv == 1 ? t : (int)__umulhi((uint32_t)t, per_spv);  // (divisors up to four, below 2^29)
        slot = slots == 1 ? 0 : round - (int)__umulhi((uint32_t)round, per_slots) * slots;
        const int in = unit - round * visit;
        const int word = round < n_rounds ? first_word + (round * wgs + (int)blockIdx.x) * visit + in : last_word + (int)blockIdx.x * dealt + in;
        if (word >= end_word) return -1;
        return (int64_t)(SAMP ? samp.other((uint32_t)word) : (uint32_t)word) << 6;
    };
    const bool short_unit = cols <= 64;  // (a unit takes hardly longer than its index words: they are requested as early as can be)
    int unit = wv, slot = 0, next_slot = 0;
    int64_t my0 = -1, next0 = -1;
    auto draw = [&]() __attribute__((always_inline)) {
        uint32_t drawn = 0;
        if (lane == 0) drawn = atomicAdd(&s_max[12], 1u);
        unit = __builtin_amdgcn_readfirstlane((int)drawn);
    };
    auto settle = [&]() __attribute__((always_inline)) {  // the next unit that has items
        next0 = -1;
        while (unit < n_units) {
            next0 = unit_at(unit, next_slot);
            if (next0 >= 0) break;
            draw();
        }
    };
    // This wavefront's item rows, 32 items to a half (past the end the last row is repeated: no mask names it), and the
    // scale of item `lane`.  If the wavefront multiplied its last items, the next ones are requested behind the
    // products of the last block of queries, into the same registers, before the masks are known.  Otherwise they are requested behind
    // the masks: where the filters pass little they are never read.
    own_i4 a[2][KS];
    float si = 0.0f;
    auto rows = [&](int64_t my0) __attribute__((always_inline)) {
        si = p.iscale[my0 + (uint32_t)min(lane, (int)min(p.n_items - 1 - my0, (int64_t)63))];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            // (offsets within the 64 rows: the base is the same for all lanes)
            const int it = min(s * 32 + (lane & 31), (int)min(p.n_items - 1 - my0, (int64_t)63));
            const own_i4* row = reinterpret_cast<const own_i4*>(p.items + my0 * D + (uint32_t)(it * D + half * 16));
#pragma unroll
            for (int k = 0; k < KS; ++k) a[s][k] = row[2 * k];
        }
    };
    settle();
    my0 = next0;
    slot = next_slot;
    const int64_t span = min(p.item_end, p.n_items) - p.item_begin;
    const float sample = p.iscale[p.item_begin + span * tid / kOwnThreads];
    constexpr int kPieces = kOwnCols * (D / 16) / kOwnThreads;  // of 16 bytes to a thread
    static_assert(kOwnCols * (D / 16) % kOwnThreads == 0, "the same number to every thread");
    int4 piece[kPieces];
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
        const int i = tid + u * kOwnThreads, c = i / (D / 16), x = i - c * (D / 16);
        piece[u] = make_int4(0, 0, 0, 0);
        if (c < n_c) piece[u] = reinterpret_cast<const int4*>(p.queries + (int64_t)p.grp_q[c0 + c] * D)[x];
    }
    float tq = -__builtin_inff();  // tau / s_q of column tid (kOwnCols columns, at most)
    int own_q = -1;
    static_assert(kOwnCols <= kOwnThreads, "a column per thread");
    if (tid < cols) {
        own_q = tid < n_c ? p.grp_q[c0 + tid] : -1;
        uint64_t t = ~0ULL;
        if (own_q >= 0)
            for (int pp = 0; pp < p.tau_parts; ++pp) t = min(t, p.tau[(int64_t)own_q * kTauParts + pp]);
        s_query[tid] = own_q;
        s_tau[tid] = t;
        const float sq = own_q >= 0 ? p.qscale[own_q] : 0.0f;
        s_sq[tid] = sq;
#pragma unroll
        for (int k = 0; k < kOwnSlots; ++k) s_cnt[k * cols + tid] = 0;
        if (own_q >= 0 && t) tq = bound_quotient(key_score(t), sq);
        if (tq > 0.0f) atomicMax(&s_max[8], __float_as_uint(tq));
    }
    // The filters of these queries: their rows lie one filter behind the other, each from a multiple of four on and
    // filled up to one with its last row.  (A filter to a thread, from the last thread on: the first ones have the columns.)
    int g0 = 0, g1 = p.n_groups;
    if (n_q > kOwnCols) {  // (filters in front and behind have no query here)
        for (int g = tid; g < p.n_groups; g += kOwnThreads)
            if (p.grp_q_off[g + 1] > c0 && p.grp_q_off[g] < c0 + n_c) {
                atomicMin(&s_max[9], (uint32_t)g);
                atomicMax(&s_max[10], (uint32_t)g + 1u);
            }
        own_barrier();
        g0 = (int)s_max[9];
        g1 = (int)s_max[10];
    }
    const int ref0 = p.grp_row_off[g0];
    auto refs_at = [&](int g) { return (p.grp_row_off[g] - ref0 + 3 * (g - g0) + 3) & ~3; };
    const bool all_rows = p.m_bits <= kOwnAllRows;
    for (int g = g0 + kOwnThreads - 1 - tid; g < g1; g += kOwnThreads) {
        const int r0 = p.grp_row_off[g], rn = p.grp_row_off[g + 1] - r0, to = refs_at(g);
        for (int r = 0; r < rn; r += 8) {
            int row[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) row[u] = p.grp_rows[r0 + min(r + u, rn - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (r + u < ((rn + 3) & ~3)) {
                    s_refs[to + r + u] = (uint16_t)row[u];
                    if (!all_rows) atomicOr(&s_bits[row[u] >> 5], 1u << (row[u] & 31));
                }
        }
        for (int i = p.grp_q_off[g]; i < p.grp_q_off[g + 1]; ++i)
            if (i >= c0 && i < c0 + n_c) {
                s_r0[i - c0] = (uint16_t)to;
                s_rn[i - c0] = (uint16_t)rn;
            }
    }
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
        const int i = tid + u * kOwnThreads, c = i / (D / 16), x = i - c * (D / 16);
        if (c < cols) *reinterpret_cast<int4*>(s_q + (size_t)c * DP + x * 16) = piece[u];
    }
    // (1 / scale of what is positive and of ordinary size, as a bit pattern: these order as the numbers do)
    const float inv_sample = sample > 0x1p-90f && sample < 0x1p90f ? __builtin_amdgcn_rcpf(sample) : 0.0f;
    const uint32_t top = wave_max_u32(__float_as_uint(inv_sample));
    if (lane == 63) s_max[wv] = top;
    // The bounds, and the slices behind the queries' rows.
    own_barrier();
    uint32_t inv_top = 0xFFFFFFFFu;  // the smallest of the wavefronts' largest ones: a few odd scales do not count
#pragma unroll
    for (int w = 0; w < 8; ++w) inv_top = min(inv_top, s_max[w] ? s_max[w] : 0xFFFFFFFFu);
    const float h_max = inv_top != 0xFFFFFFFFu ? __uint_as_float(inv_top) : 0.0f, tq_max = __uint_as_float(s_max[8]);
    const float ref = slice_ref(h_max, tq_max), factor = slice_factor(ref);
    const float shared_below = slice_wide(h_max, tq_max) ? slice_shared_below(tq_max) : 0.0f;
    const bool wide = __builtin_amdgcn_readfirstlane(__float_as_int(shared_below)) != 0;
    if (tid < cols) {
        const int u = tq > 0.0f ? slice_query(tq, ref) : 0;
        const bool none = own_q >= 0 && !(tq > 0.0f);
        s_u[tid] = (uint16_t)(none ? kNoBound : u);
        if (none) s_max[11] = 1;
#pragma unroll
        for (int w = 0; w < kSliceBytes / 16; ++w)
            *reinterpret_cast<int4*>(s_q + (size_t)tid * DP + D + 16 * w) =
                make_int4(slice_query_word(u, 4 * w), slice_query_word(u, 4 * w + 1), slice_query_word(u, 4 * w + 2), slice_query_word(u, 4 * w + 3));
    }
    // The signature rows that some filter names, numbered in order: only these are staged.  (A small index is staged
    // whole: reading the names first holds up the first segment, 2.5 us of 39 with 8 rows.)
    static_assert(kOwnRows == kOwnThreads, "a row per thread");
    int n_named = p.m_bits;
    if (!all_rows) {
        // (lane w: named rows in front of the 32 of word w)
        const uint32_t of_word = lane < kOwnRows / 32 ? (uint32_t)__popc(s_bits[lane]) : 0u, upto = wave_scan_add(of_word), front = upto - of_word;
        auto named_before = [&](int r) { return (int)__shfl(front, r >> 5) + __popc(s_bits[r >> 5] & ((1u << (r & 31)) - 1u)); };
        const int of_mine = named_before(tid);
        if (s_bits[tid >> 5] >> (tid & 31) & 1) s_named[of_mine] = (uint16_t)tid;
        const int refs = g1 > g0 ? refs_at(g1 - 1) + ((p.grp_row_off[g1] - p.grp_row_off[g1 - 1] + 3) & ~3) : 0;
        for (int i0 = 0; i0 < refs; i0 += kOwnThreads) {  // (all lanes take part in the exchange)
            const int i = min(i0 + tid, refs - 1), no = named_before(s_refs[i] & (kOwnRows - 1));
            if (i0 + tid < refs) s_refs[i] = (uint16_t)no;
        }
        n_named = (int)lane_value(upto, 63);
    }
    own_barrier();  // the last one: from here on every wavefront works by itself, up to the report
    const bool open = __builtin_amdgcn_readfirstlane((int)s_max[11]) != 0;

    // index words of the wavefront's 64 items: one to a named row
    constexpr int kIdx = KS < 8 ? kOwnRows / 64 : 4;  // (those of rows beyond are read when they are needed: registers)
    uint64_t idx[kIdx];
    uint32_t idx_at[kIdx];  // bytes
#pragma unroll
    for (int u = 0; u < kIdx; ++u) {
        const int x = max(min(lane + u * 64, n_named - 1), 0);  // (the last row again: an unconditional load)
        idx_at[u] = (uint32_t)(all_rows ? min(x, p.m_bits - 1) : n_named > 0 ? (int)s_named[x] : 0) * (kTileWords * 8);
    }
    auto fetch = [&](int64_t first) __attribute__((always_inline)) {
        const int64_t w0 = first >> 6;
        const char* src = reinterpret_cast<const char*>(p.bloom + (w0 >> 4) * (int64_t)p.m_bits * kTileWords + (w0 & 15));
#pragma unroll
        for (int u = 0; u < kIdx; ++u) idx[u] = u * 64 < n_named ? *reinterpret_cast<const uint64_t*>(src + idx_at[u]) : 0;
    };
    // the rows of this lane's columns: place of the first one, and of the last four from there
    constexpr uint32_t kNoRows = 0x80000000u;  // an empty filter: all items pass
    uint32_t my_refs[kOwnCols / 64];
    int rn_max = 0;
#pragma unroll
    for (int u = 0; u < kOwnCols / 64; ++u) {
        const int c = lane + u * 64, rn = c < n_c ? (s_rn[c] + 3) & ~3 : 0;
        my_refs[u] = rn ? (uint32_t)s_r0[c] | (uint32_t)(rn - 4) << 16 : c < n_c ? kNoRows : 0u;
        rn_max = max(rn_max, rn);
    }
    rn_max = (int)lane_value(wave_max_u32((uint32_t)rn_max), 63);
    if (my0 >= 0) fetch(my0);
    // Pairs that may be admissible, for the exact test.  LIST: items, and columns with region slots, in one list for a wavefront that
    // multiplies and one that gathers, and their rows are read again.  Otherwise a wavefront that multiplies has a queue of dot products
    // less their bounds, items and columns: to pick the result takes some 45 instructions to a pair of each lane, which a product
    // of rows of 192 or 256 bytes covers (with the list there, 1 M x 192, 100 queries, scales of many sizes: 144 -> 157 us; 10 M x 256,
    // 256: 918 -> 930) and one of shorter rows does not (1.26 M x 96, 238 queries: 133.5 -> 129.6; 1.65 M x 96, 200: 151.6 -> 146.7; 2 M x 64, 256: 196 -> 185).
    constexpr bool LIST = KS <= 4;
    int qn = 0;
    auto admit = [&](uint64_t key, int c, int sl_no) __attribute__((always_inline)) {
        const uint32_t n = atomicAdd(&s_cnt[sl_no * cols + c], 1u);
        if (n < (uint32_t)p.cap)
            p.cand[((int64_t)s_query[c] * p.groups + (int)blockIdx.x + sl_no * (int)gridDim.x) * p.cap + n] = key;
    };
    // (of a unit's largest scale, as a bit pattern; 0: none)
    auto shared = [](uint32_t top_scale) { return top_scale ? slice_shared(__builtin_amdgcn_rcpf(__uint_as_float(top_scale))) : 0.0f; };
    auto drain = [&]() __attribute__((always_inline)) {
        if (lane < qn) {
            const int4 e = queue[lane];
            const int c = e.z & 255, u = s_u[c] == kNoBound ? 0 : s_u[c];
            const float s_i = p.iscale[(uint32_t)e.y], h = shared((uint32_t)e.w);
            const int dot = e.x + slice_base(u, slice_base_factor(h, factor)) + slice_bound(u, slice_item(__builtin_amdgcn_rcpf(s_i) - h, factor));
            const uint64_t key = make_key(rescale(dot, s_sq[c], s_i), (uint32_t)e.y);
            if (key >= s_tau[c]) admit(key, c, e.z >> 8);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");  // (what is written here next may be of the list, another type)
        qn = 0;
    };
    // The list goes from one unit to the next until there are 64 pairs.  Their rows come kGl lanes to a row, so that a load takes whole
    // lines (a lane to a row takes four times as many).
    int pn = 0;
    constexpr int kPer = D % 96 == 0 ? 3 : 1, kGl = D / 16 / kPer, kGp = 64 / kGl;  // (pieces of a row to a lane, lanes to a row, rows to a load)
    auto gather = [&](int k0, int n) __attribute__((always_inline)) {
        const int piece = lane & (kGl - 1), in_load = lane / kGl;
        // (the pair whose result this lane keeps)
        const int my_pair = piece * kGp + in_load;
        const uint2 mine = s_pairs[k0 + min(my_pair, n - 1)];
        const float my_si = p.iscale[mine.x];
        int4 v[kGl][kPer];
#pragma unroll
        for (int j = 0; j < kGl; ++j) {
            const int4* row = reinterpret_cast<const int4*>(p.items + (int64_t)s_pairs[k0 + min(j * kGp + in_load, n - 1)].x * D) + piece;
#pragma unroll
            for (int t = 0; t < kPer; ++t) v[j][t] = row[t * kGl];
        }
        int my_dot = 0;
#pragma unroll
        for (int j = 0; j < kGl; ++j) {
            const int c = (int)(s_pairs[k0 + min(j * kGp + in_load, n - 1)].y & 255u);
            const int4* qr = reinterpret_cast<const int4*>(s_q + c * DP) + piece;
            int dot = 0;
#pragma unroll
            for (int t = 0; t < kPer; ++t) dot = dot16(v[j][t], qr[t * kGl], dot);
            dot += __builtin_amdgcn_update_dpp(0, dot, 0xB1, 0xF, 0xF, false);                // lanes 1, 0, 3, 2 of four
            if (kGl > 2) dot += __builtin_amdgcn_update_dpp(0, dot, 0x4E, 0xF, 0xF, false);   // lanes 2, 3, 0, 1
            if (kGl > 4) dot += __builtin_amdgcn_update_dpp(0, dot, 0x141, 0xF, 0xF, false);  // eight lanes mirrored
            if (kGl > 8) dot += __builtin_amdgcn_update_dpp(0, dot, 0x140, 0xF, 0xF, false);  // sixteen
            if (piece == j) my_dot = dot;
        }
        if (my_pair < n) {
            const int c = (int)(mine.y & 255u);
            const uint64_t key = make_key(rescale(my_dot, s_sq[c], my_si), mine.x);
            if (key >= s_tau[c]) admit(key, c, (int)(mine.y >> 8));
        }
    };
    // ... all whole rounds of the list, what is left goes to its front
    auto rounds = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        if (pn < 64) return;
        const int whole = pn & ~63;
        for (int k0 = 0; k0 < whole; k0 += 64) gather(k0, 64);
        const uint2 rest = s_pairs[min(whole + lane, kOwnPairs - 1)];
        pn -= whole;
        if (lane < pn) s_pairs[fresh(lane)] = rest;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    };
    // A unit's masks, of all filters: the words of four columns to a lane, so that a step's reads do not wait for each other.
    // Also draws the next unit, and brings this one's index words to LDS.
    uint64_t m[kOwnCols / 64];
    uint32_t n_pass = 0, before = 0, total = 0;  // pairs that pass: this lane's, the lower lanes', all
    auto masks = [&]() __attribute__((always_inline)) {
        draw();
        const int named = fresh_scalar(n_named), cl = fresh_scalar(n_c);
        const uint32_t no_rows = (uint32_t)fresh_scalar((int)kNoRows);
#pragma unroll
        for (int u = 0; u < kIdx; ++u)
            if (lane < named - u * 64) s_idx[lane + u * 64] = idx[u];
        if (kIdx * 64 < kOwnRows && n_named > kIdx * 64) {
            const uint64_t* src = p.bloom + (my0 >> 10) * (int64_t)p.m_bits * kTileWords + ((my0 >> 6) & 15);
            for (int x = lane + kIdx * 64; x < n_named; x += 64) s_idx[x] = src[(int)s_named[x] * kTileWords];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        settle();
        if (next0 >= 0 && short_unit) fetch(next0);
        const int64_t left = item_lim - my0;
        const uint64_t all = left >= 64 ? ~0ULL : left > 0 ? ((1ULL << left) - 1ULL) : 0ULL;
#pragma unroll
        for (int u = 0; u < kOwnCols / 64; ++u) m[u] = lane < cl - u * 64 ? all : 0;
        for (int r = 0; r < rn_max; r += 4) {
            ushort4 f[kOwnCols / 64];
#pragma unroll
            for (int u = 0; u < kOwnCols / 64; ++u)
                if (u * 64 < cols) f[u] = *reinterpret_cast<const ushort4*>(s_refs + (my_refs[u] & 0xFFFFu) + min(r, (int)(my_refs[u] >> 16 & 0x7FFFu)));
#pragma unroll
            for (int u = 0; u < kOwnCols / 64; ++u)
                if (u * 64 < cols) m[u] &= (s_idx[f[u].x] & s_idx[f[u].y]) & (s_idx[f[u].z] & s_idx[f[u].w]);
        }
        n_pass = 0;
#pragma unroll
        for (int u = 0; u < kOwnCols / 64; ++u)
            if (u * 64 < cols) {
                if (my_refs[u] & no_rows) m[u] = all;
                n_pass += (uint32_t)__popcll(m[u]);
            }
        const uint32_t incl = wave_scan_add(n_pass);
        before = incl - n_pass;
        total = lane_value(incl, 63);
    };
    // The loop has two parts, so that the rows in registers are none while a wavefront gathers.
    if (my0 >= 0) masks();
    while (my0 >= 0) {
        if (total <= (uint32_t)own_few(cols)) {
            if (next0 >= 0 && !short_unit) fetch(next0);
            if (!LIST && qn > 0) drain();
            uint32_t pos = (uint32_t)pn + before;
#pragma unroll
            for (int u = 0; u < kOwnCols / 64; ++u)
                while (m[u]) {
                    const int bit = __ffsll((long long)m[u]) - 1;
                    m[u] &= m[u] - 1;
                    s_pairs[pos++] = make_uint2((uint32_t)my0 + (uint32_t)bit, (uint32_t)(lane + u * 64) | (uint32_t)slot << 8);
                }
            pn = __builtin_amdgcn_readfirstlane(pn + (int)total);
            rounds();
            my0 = next0;
            slot = next_slot;
            if (my0 >= 0) masks();
            continue;
        }
        if (!LIST && pn > 0) {  // (the queue lies where the list does)
            gather(0, pn);
            pn = 0;
        }
        rows(my0);
        for (;;) {
            const int cl = fresh_scalar(cols);
#pragma unroll
            for (int u = 0; u < kOwnCols / 64; ++u)
                if (lane < cl - u * 64) s_mask[lane + u * 64] = m[u];
            // The scales, and the items' slices: half a slice to a lane, as the operand has it.
            const bool odd = ballot(!(si >= 0.0f && si < 0x1p90f)) != 0;  // (outside the range that has bounds: all pairs of these items are tested exactly)
            uint32_t top_scale = 0;  // the largest one as a bit pattern, where a part of the bounds is shared
            if (wide && !odd) {
                const uint32_t top = lane_value(wave_max_u32(__float_as_uint(si) & 0x7FFFFFFFu), 63);
                if (__uint_as_float(top) < shared_below) top_scale = top;
            }
            const int g = slice_item(__builtin_amdgcn_rcpf(si) - shared(top_scale), factor);
            own_i4 sl[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int gs = __shfl(g, 32 * s + (lane & 31));
                const int same = slice_item_word(gs, 0);
                sl[s] = own_i4{same, same, same, half ? slice_item_word(gs, 7) : same};
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            own_i4 q[KS + 1];  // a block's operands: the rows and slices of 32 queries
            auto operands = [&](int b) __attribute__((always_inline)) {
                const own_i4* qr = reinterpret_cast<const own_i4*>(s_q + (size_t)(b + (lane & 31)) * DP) + half;
#pragma unroll
                for (int k = 0; k <= KS; ++k) q[k] = qr[2 * k];
            };
            own_i16 acc[2];
            auto products = [&](int b) __attribute__((always_inline)) {
                own_i16 from;
                auto first = [&](int start) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) from[i] = start;
#pragma unroll
                    for (int s = 0; s < 2; ++s) acc[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s][0], q[0], from, 0, 0, 0);
                };
                if (top_scale) {  // (otherwise the instructions start at a constant 0)
                    const int u = s_u[fresh(b + (lane & 31))];
                    first(u == kNoBound ? 0 : -slice_base(u, slice_base_factor(shared(top_scale), factor)));
                } else {
                    first(0);
                }
#pragma unroll
                for (int k = 1; k <= KS; ++k)
#pragma unroll
                    for (int s = 0; s < 2; ++s) acc[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(k < KS ? a[s][k < KS ? k : 0] : sl[s], q[k], acc[s], 0, 0, 0);
            };
            auto test = [&](int b, uint64_t word) __attribute__((always_inline)) {
                const int c = b + (lane & 31);
                uint32_t keep = ~0u;
                if (open || odd) keep = odd || s_u[c] == kNoBound ? 0u : ~0u;
                // result i is item 32 s + 8 (i / 4) + 4 half + i % 4; the signs go to the bits of the mask word
                uint32_t below[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    uint32_t part[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        part[j] = (uint32_t)acc[s][4 * j + 3] >> 31;
#pragma unroll
                        for (int i = 2; i >= 0; --i) part[j] = __builtin_amdgcn_alignbit(part[j], (uint32_t)acc[s][4 * j + i], 31);
                    }
                    below[s] = (part[3] << 24 | part[2] << 16) | (part[1] << 8 | part[0]);
                }
                // (the second half's bits in the gaps of the first one's)
                const uint32_t pass = ((uint32_t)word >> (4 * half) & 0x0F0F0F0Fu) | ((uint32_t)(word >> 32) >> (4 * half) & 0x0F0F0F0Fu) << 4;
                uint32_t over = pass & ~((below[0] | below[1] << 4) & keep);
                uint64_t hits;
                while ((hits = ballot(over != 0)) != 0) {  // (as a rule one pair to a lane)
                    const int n = __popcll(hits), rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
                    if (!LIST && qn + n > kOwnQueue) drain();
                    if (over != 0) {
                        const int bit = __ffs((int)over) - 1, at_item = (bit & 27) + 8 * (bit & 4) + 4 * half;
                        over &= over - 1;
                        if constexpr (LIST) {
                            s_pairs[pn + rank] = make_uint2((uint32_t)my0 + (uint32_t)at_item, (uint32_t)(c | slot << 8));
                        } else {
                            // (by masks: choices by a condition become an access indexed by the lane, in private memory)
                            const int b0 = -(bit & 1), b1 = -(bit >> 1 & 1), b2 = -(bit >> 2 & 1), b3 = -(bit >> 3 & 1), b4 = -(bit >> 4 & 1);
                            auto pick = [](int m, int x, int y) { return (x & m) | (y & ~m); };
                            int v[16];
#pragma unroll
                            for (int i = 0; i < 16; ++i) v[i] = pick(b2, acc[1][i], acc[0][i]);
#pragma unroll
                            for (int i = 0; i < 8; ++i) v[i] = pick(b0, v[2 * i + 1], v[2 * i]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] = pick(b1, v[2 * i + 1], v[2 * i]);
#pragma unroll
                            for (int i = 0; i < 2; ++i) v[i] = pick(b3, v[2 * i + 1], v[2 * i]);
                            queue[qn + rank] = make_int4(pick(b4, v[1], v[0]), (int)((uint32_t)my0 + (uint32_t)at_item), c | slot << 8, (int)top_scale);
                        }
                    }
                    if constexpr (LIST) {
                        pn = __builtin_amdgcn_readfirstlane(pn + n);
                        if (pn >= 64) rounds();
                    } else {
                        qn = __builtin_amdgcn_readfirstlane(qn + n);
                    }
                }
            };
            // A block's operands are read behind the products of the one before, and tested while they come.  The next segment's
            // index words are requested once the rows are there, and its rows behind the last block's products: a wait for
            // what is older is none for them.
            operands(0);
            uint64_t word = s_mask[lane & 31];
            products(0);
            if (next0 >= 0 && !short_unit) fetch(next0);
            for (int b = 32; b < n_blk; b += 32) {
                operands(b);
                const uint64_t next_word = s_mask[b + (lane & 31)];
                test(b - 32, word);
                word = next_word;
                products(b);
            }
            rows(next0 >= 0 ? next0 : my0);  // (without a condition: one would turn the wait for the index words into one for the rows)
            test(n_blk - 32, word);
            my0 = next0;
            slot = next_slot;
            if (my0 < 0) break;
            masks();
            if (total <= (uint32_t)own_stay(cols)) break;
        }
    }
    if (!LIST && qn > 0) drain();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    if (pn > 0) gather(0, pn);
    __syncthreads();
    // fill counts of the workgroup's regions
    for (int i = tid; i < n_c * slots; i += kOwnThreads) {
        const int k = i / n_c, c = i - k * n_c, q = s_query[c];
        const uint32_t n = s_cnt[k * cols + c];
        p.cnt[(int64_t)q * p.groups + (int)blockIdx.x + k * (int)gridDim.x] = n < (uint32_t)p.cap ? n : (uint32_t)p.cap;
        if (n > (uint32_t)p.cap) p.ovf[q] = 1u;
    }
}

// The first level of such a search, which admits every passing pair: the same products, 64 items (a region) to a
// wavefront.  An item's place among a filter's passing ones is its place in the region, so there are no counters; the
// number of bits of the mask word is the region's count.  In sample mode region r takes segment r of the sample, elsewhere the
// r-th 64 items of the level.  Masks are formed from the index in memory (a wavefront has one
// segment: staging would not pay).  Grid (regions / 8, ceil(queries / kOwnFirstCols)): half the queries to a workgroup, so that 256 of
// them fill the chip.  Bound by its round trips and the scattered stores of the keys: 65,536 items, 213 queries with filters
// of their own (5 %), d = 256: 190 us by gathering a row per pair, now 27 (the call 1.48 -> 1.31 ms; 800,000 x 64, 256 queries: 320 -> 175).
constexpr int kOwnFirstCols = 128;
constexpr size_t own_first_lds_bytes(int d) { return (size_t)kOwnFirstCols * (d + 16 + 8 * 8 + 2 * 4); }

template <int KS>
__global__ __launch_bounds__(kOwnThreads) void scan_own_first_kernel(ScanParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char own_lds[];
    constexpr int D = 32 * KS, DP = D + 16;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    const int n_q = p.grp_q_off[p.n_groups], c0 = (int)blockIdx.y * kOwnFirstCols, n_c = min(n_q - c0, kOwnFirstCols);
    int8_t* s_q = reinterpret_cast<int8_t*>(own_lds);                                              // [cols][DP]
    uint64_t* s_mask = reinterpret_cast<uint64_t*>(s_q + (size_t)kOwnFirstCols * DP) + (size_t)wv * kOwnFirstCols;
    float* s_sq = reinterpret_cast<float*>(s_q + (size_t)kOwnFirstCols * (DP + 64));               // [cols]
    int32_t* s_query = reinterpret_cast<int32_t*>(s_sq + kOwnFirstCols);                           // [cols]
    const int region = (int)blockIdx.x * (kOwnThreads / 64) + wv;
    const int64_t my0 = p.samp_role == 1 ? region * p.samp_stride_items : p.item_begin + (int64_t)region * 64;
    const int64_t lim = p.item_end < p.n_items ? p.item_end : p.n_items, left = p.samp_role == 1 ? (region < p.samp_segs ? 64 : 0) : lim - my0;
    const uint64_t all = left >= 64 ? ~0ULL : left > 0 ? ((1ULL << left) - 1ULL) : 0ULL;

    // item rows and scales (past the end the last item is repeated: no mask names it)
    own_i4 a[2][KS];
    float si[2][16];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int64_t it = min(my0 + s * 32 + (lane & 31), p.n_items - 1);
        const own_i4* row = reinterpret_cast<const own_i4*>(p.items + it * D) + half;
#pragma unroll
        for (int k = 0; k < KS; ++k) a[s][k] = row[2 * k];
#pragma unroll
        for (int i = 0; i < 16; ++i) si[s][i] = p.iscale[min(my0 + s * 32 + 8 * (i >> 2) + 4 * half + (i & 3), p.n_items - 1)];
    }
    for (int i = tid; i < kOwnFirstCols * (D / 16); i += kOwnThreads) {
        const int c = i / (D / 16), x = i - c * (D / 16);
        int4 v = make_int4(0, 0, 0, 0);
        if (c < n_c) v = reinterpret_cast<const int4*>(p.queries + (int64_t)p.grp_q[c0 + c] * D)[x];
        *reinterpret_cast<int4*>(s_q + (size_t)c * DP + x * 16) = v;
    }
    if (tid < kOwnFirstCols) {
        const int q = tid < n_c ? p.grp_q[c0 + tid] : -1;
        s_query[tid] = q;
        s_sq[tid] = q >= 0 ? p.qscale[q] : 0.0f;
    }
    // mask words: a filter of mine at a time, for its queries among these columns
    const int64_t w0 = my0 >> 6;
    const uint64_t* base = p.bloom + (w0 >> 4) * (int64_t)p.m_bits * kTileWords + (w0 & 15);
    for (int c = lane; c < kOwnFirstCols; c += 64) s_mask[c] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    for (int g = lane; g < p.n_groups; g += 64) {
        const int q0 = max(p.grp_q_off[g] - c0, 0), q1 = min(p.grp_q_off[g + 1] - c0, n_c);
        if (q0 >= q1) continue;
        uint64_t m = all;
        const int r1 = p.grp_row_off[g + 1];
        if (m)
            for (int r = p.grp_row_off[g]; r < r1; r += 8) {  // eight rows are requested together (the last one again)
                uint64_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = base[(int64_t)p.grp_rows[min(r + u, r1 - 1)] * kTileWords];
#pragma unroll
                for (int u = 0; u < 8; ++u) m &= v[u];
            }
        for (int c = q0; c < q1; ++c) {
            s_mask[c] = m;
            p.cnt[(int64_t)p.grp_q[c0 + c] * p.groups + region] = (uint32_t)__popcll(m);
        }
    }
    __syncthreads();
    for (int b = 0; b < n_c; b += 32) {
        const int c = b + (lane & 31);
        const uint64_t word = s_mask[c];
        if (ballot(word != 0) == 0) continue;
        const float sq = s_sq[c];
        uint64_t* dst = p.cand + ((int64_t)max(s_query[c], 0) * p.groups + region) * p.cap;
        const own_i4* qr = reinterpret_cast<const own_i4*>(s_q + (size_t)c * DP) + half;
        own_i16 acc[2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[s][i] = 0;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const own_i4 bq = qr[2 * k];
            acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0][k], bq, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[1][k], bq, acc[1], 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // results 4 j .. 4 j + 3 are the items from bit0 on
                const int bit0 = 32 * s + 8 * j + 4 * half;
                const uint32_t four = (uint32_t)(word >> bit0) & 15u;
                if (ballot(four != 0) == 0) continue;
                const int at = __popcll(word & ((1ULL << bit0) - 1ULL));
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (four >> i & 1u)
                        dst[at + __popc(four & ((1u << i) - 1u))] =
                            make_key(rescale(acc[s][4 * j + i], sq, si[s][4 * j + i]), (uint32_t)my0 + (uint32_t)(bit0 + i));
            }
    }
}

// The kernel for rows of d bytes, or null.  (One copy of the kernel to a length: the lengths the MFMA scan has, as far as
// a workgroup's registers hold the rows of 64 items, and 96 and 192 between them; others go to the gathering scan.)
template <bool SAMP>
inline auto own_kernel(int d) -> decltype(&scan_own_kernel<8, SAMP>)
{
    switch (d) {
    case 64: return &scan_own_kernel<2, SAMP>;
    case 96: return &scan_own_kernel<3, SAMP>;
    case 128: return &scan_own_kernel<4, SAMP>;
    case 192: return &scan_own_kernel<6, SAMP>;
    case 256: return &scan_own_kernel<8, SAMP>;
    default: return nullptr;
    }
}
inline auto own_kernel(int d, bool sample = false) -> decltype(&scan_own_kernel<8, true>) { return sample ? own_kernel<true>(d) : own_kernel<false>(d); }
inline auto own_first_kernel(int d) -> decltype(&scan_own_first_kernel<8>)
{
    switch (d) {
    case 64: return &scan_own_first_kernel<2>;
    case 96: return &scan_own_first_kernel<3>;
    case 128: return &scan_own_first_kernel<4>;
    case 192: return &scan_own_first_kernel<6>;
    case 256: return &scan_own_first_kernel<8>;
    default: return nullptr;
    }
}

}  // namespace st
