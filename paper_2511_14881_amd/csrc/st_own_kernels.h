// Scan for batches whose queries hardly share filters (levels with thresholds in force).
//
// The wavefront dot-product scan gathers one item row per passing pair: at 10 M items x 256 bytes and 256
// filters that pass 5 % each, 2 G 16-byte gathers, 64 cache lines to an instruction.  Here a wavefront holds
// the rows of 64 items in registers and multiplies them with all queries by MFMA, whether a filter
// passes them or not; the filters decide which scores count.  That costs the same for every selectivity, so a
// wavefront whose filters pass few pairs (own_pairs) gathers after all, and one that did so requests the next
// items' rows only when their masks are known.
//
// Eight wavefronts take a segment of 512 items, 64 items each; up to the reports of a region they share the queries
// and the tables in LDS and nothing else, so that one forms masks or waits for rows while another multiplies.  A wavefront's
// words of the index (the rows that some filter names, m <= kOwnRows) come to LDS with loads requested a segment
// ahead, and its mask words of all filters are formed there (a filter's rows fetched one by one from memory took
// longer than the products).  A mask word is what it needs for one query: lane l of the product's result holds query l % 32,
// and 16 of its items.  The items go in two halves of 32; the first half of the next ones is requested behind the
// products of the first half, into the same registers.  A pair is tested by one multiply-add (the item's scale in fixed point,
// the query's bound) whose sign goes to the bit of the pair's item; lanes with a bit left under the mask are
// queued with their 16 dot products, and the exact score, key and threshold test run where the queue is emptied.
// The queries stay in LDS, padded by 16 bytes a row (an odd number of 16-byte pieces: no bank conflicts).
// 10 M x 256 bytes, 256 queries with filters of their own (5 % each), K = 500: the level after the first takes
// 1.09 ms in a long series of calls (1.15 to 1.4 in a run's first twelve), where gathering took 4.5 (1.26 with exact
// tests of all scores and two barriers to a segment); 778 k x 96 with 37 filter programs: 36 us (38).  Bound by round
// trips to LDS (operands, masks, queue: 55 % of a wavefront's
// time) with two wavefronts to a SIMD; the products alone keep the matrix units busy a fifth of the time, the
// rows of all items once are 0.5 ms of memory.
//
// It takes the place of the gathering scan whatever the filters pass, which the host cannot know.  Calls on 3 M
// items, m = 512, K = 100, every query with a filter of its own, gathering -> this scan, in us (d = 256 unless
// said; with rows requested and all index rows staged before the masks were known, 16 queries took 280 to 300 throughout):
//   queries   0.05 % pass   0.2 %        1 %          5 %          the broadest (3 to 16 %)
//     16      112 -> 107    155 -> 122   161 -> 124   216 -> 186   410 -> 225
//     64      244 -> 124    353 -> 129   464 -> 182   527 -> 253   734 -> 269
//    256      909 -> 341   1458 -> 401  1909 -> 620  2127 -> 733  2222 -> 747
//     16, 64 bytes  99 -> 88   129 -> 95   128 -> 88   131 -> 103   200 -> 130
// (with two barriers to a segment and the first level gathered; without them and with scan_own_first_kernel, 256 queries,
// same card: 349 -> 272, 396 -> 300, 621 -> 427, 711 -> 496, 700 -> 485)
// one filter for 64 queries, 10 M x 192: 447 -> 176 at 0.02 %, 807 -> 339 at 0.5 %, 825 -> 543 at 5 %; behind cluster probing
// (600 of 4096 clusters, 3 M x 128, 32 queries) 326 -> 243.
#pragma once
#include "st_search_kernels.h"

namespace st {

constexpr int kOwnThreads = 512;
constexpr int kOwnSeg = 512;            // items of a segment
constexpr int kOwnWords = kOwnSeg / 64; // one mask word per wavefront
constexpr int kOwnBlock = 32;           // queries of one product
constexpr int kOwnCols = 256;           // queries resident at a time (one row of the grid)
constexpr int kOwnRows = 512;           // signature rows of the index, at most
// Items of a level, at least: two segments to each of the workgroups that are resident.  (Whether the candidate
// regions have room for segments of this size is the plan's to say: level_takes_segments.)
constexpr int64_t kOwnMinItems = 512 * kOwnSeg;
constexpr int kOwnAllRows = 64;         // an index of no more rows is staged whole
constexpr int kOwnQueue = 16;           // lanes of a wavefront that wait for the exact test
constexpr int kOwnRowRefs = 6144;       // rows all filters name together, at most
static_assert(kOwnWords == kOwnThreads / 64, "a word per wavefront");

constexpr int own_cols(int n_q) { return n_q < kOwnCols ? (n_q + 31) / 32 * 32 : kOwnCols; }
// A wavefront whose filters pass no more pairs than this of its 64 items gathers the pairs' rows instead of
// multiplying all: 64 gathered rows of d bytes keep the load path busy for 64 * d / 16 cycles, the product with its
// tests for 64 items x 256 queries about 12,000 cycles of one of four matrix units (d = 256); and 64 pairs or fewer
// name no more rows than the product would read.
constexpr int own_pairs(int cols) { return cols < 64 ? 64 : cols; }
constexpr size_t own_lds_bytes(int n_q, int d, int m_bits)
{
    const size_t c = own_cols(n_q);
    return c * (d + 16) + c * kOwnWords * 8 + (size_t)m_bits * kOwnWords * 8 + kOwnRowRefs * 2 + c * (8 + 4 * 7) +
           own_pairs((int)c) * (kOwnThreads / 64) * 2 + kOwnRows * 2 + kOwnRows / 8 +
           (size_t)kOwnWords * (64 * 4 + kOwnQueue * (16 * 4 + 8));
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

// d = 32 * KS.  Grid (workgroups, ceil(queries / kOwnCols)); segments start at multiples of 512 items.  One
// workgroup to a compute unit is resident (registers), so that many are launched and each takes several
// regions in turn: the queries and tables are brought to LDS once.
// ONE: at most kOwnBlock queries.
template <int KS, bool ONE>
__global__ __launch_bounds__(kOwnThreads) void scan_own_kernel(ScanParams p, int n_refs)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char own_lds[];
    constexpr int D = 32 * KS, DP = D + 16;
    constexpr int P = KS <= 2 ? 10 : (KS <= 4 ? 9 : 8);   // bits of a scale in fixed point: |dot| <= 2^14 d, the product at most 2^30
    constexpr int kPass = (1 << 30) - 1, kNever = -(1 << 30) - 1;  // bounds that every pair reaches, and none
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    const int n_q = p.grp_q_off[p.n_groups];
    const int cols = own_cols(n_q), c0 = (int)blockIdx.y * kOwnCols, n_c = min(n_q - c0, cols);
    unsigned char* at = own_lds;
    int8_t* s_q = reinterpret_cast<int8_t*>(at);                  at += (size_t)cols * DP;          // [cols][DP]
    uint64_t* s_mask = reinterpret_cast<uint64_t*>(at) + (size_t)wv * cols;      at += (size_t)cols * kOwnWords * 8;
    uint64_t* s_idx = reinterpret_cast<uint64_t*>(at) + (size_t)wv * p.m_bits;   at += (size_t)p.m_bits * kOwnWords * 8;
    uint64_t* s_tau = reinterpret_cast<uint64_t*>(at);            at += (size_t)cols * 8;
    float* s_sq = reinterpret_cast<float*>(at);                   at += (size_t)cols * 4;
    int32_t* s_query = reinterpret_cast<int32_t*>(at);            at += (size_t)cols * 4;
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(at);            at += (size_t)cols * 4;
    int32_t* s_r0 = reinterpret_cast<int32_t*>(at);               at += (size_t)cols * 4;
    int32_t* s_rn = reinterpret_cast<int32_t*>(at);               at += (size_t)cols * 4;
    const int few = own_pairs(cols);
    uint16_t* s_pairs = reinterpret_cast<uint16_t*>(at) + (size_t)wv * few;  at += (size_t)few * (kOwnThreads / 64) * 2;
    uint16_t* s_refs = reinterpret_cast<uint16_t*>(at);           at += (size_t)kOwnRowRefs * 2;
    uint16_t* s_named = reinterpret_cast<uint16_t*>(at);          at += (size_t)kOwnRows * 2;
    uint32_t* s_bits = reinterpret_cast<uint32_t*>(at);           at += kOwnRows / 8;               // [kOwnRows / 32]
    uint32_t* q_val = reinterpret_cast<uint32_t*>(at) + (size_t)wv * kOwnQueue * 16;  at += (size_t)kOwnWords * kOwnQueue * 64;
    uint2* q_code = reinterpret_cast<uint2*>(at) + (size_t)wv * kOwnQueue;  at += (size_t)kOwnWords * kOwnQueue * 8;
    float* s_si = reinterpret_cast<float*>(at) + (size_t)wv * 64; at += (size_t)kOwnWords * 64 * 4;  // scales of the wavefront's items
    int32_t* s_neg = reinterpret_cast<int32_t*>(at);              at += (size_t)cols * 4;  // bounds, for the largest exponent so far
    float* s_tq = reinterpret_cast<float*>(at);                   // [cols] tau / s_q (see bound_quotient)

    if (tid < kOwnRows / 32) s_bits[tid] = 0;
    for (int c = tid; c < cols; c += kOwnThreads) {
        const int q = c < n_c ? p.grp_q[c0 + c] : -1;
        uint64_t t = ~0ULL;
        if (q >= 0)
            for (int pp = 0; pp < p.tau_parts; ++pp) t = min(t, p.tau[(int64_t)q * kTauParts + pp]);
        s_query[c] = q;
        s_tau[c] = t;
        const float sq = q >= 0 ? p.qscale[q] : 0.0f;
        s_sq[c] = sq;
        s_tq[c] = t ? bound_quotient(key_score(t), sq) : -__builtin_inff();
        s_cnt[c] = 0;
        s_neg[c] = kNever;
    }
    for (int g = tid; g < p.n_groups; g += kOwnThreads) {
        const int r0 = p.grp_row_off[g], rn = p.grp_row_off[g + 1] - r0;
        for (int i = p.grp_q_off[g]; i < p.grp_q_off[g + 1]; ++i)
            if (i >= c0 && i < c0 + n_c) {
                s_r0[i - c0] = r0;
                s_rn[i - c0] = rn;
            }
    }
    for (int i = tid; i < cols * (D / 16); i += kOwnThreads) {
        const int c = i / (D / 16), x = i - c * (D / 16);
        int4 v = make_int4(0, 0, 0, 0);
        if (c < n_c) v = reinterpret_cast<const int4*>(p.queries + (int64_t)p.grp_q[c0 + c] * D)[x];
        *reinterpret_cast<int4*>(s_q + (size_t)c * DP + x * 16) = v;
    }

    // The signature rows that some filter names, numbered in order: only these are staged.  (A small index is staged
    // whole: reading the names first holds up the first segment, 2.5 us of 39 with 8 rows.)
    static_assert(kOwnRows == kOwnThreads, "a row per thread");
    int n_named = p.m_bits;
    if (p.m_bits <= kOwnAllRows) {
        for (int i = tid; i < n_refs; i += kOwnThreads) s_refs[i] = (uint16_t)p.grp_rows[i];
    } else {
        own_barrier();
        for (int i = tid; i < n_refs; i += kOwnThreads) {
            const int r = p.grp_rows[i];
            s_refs[i] = (uint16_t)r;
            atomicOr(&s_bits[r >> 5], 1u << (r & 31));
        }
        own_barrier();
        uint32_t bits[kOwnRows / 32];
#pragma unroll
        for (int w = 0; w < kOwnRows / 32; ++w) bits[w] = s_bits[w];
        auto named_before = [&](int r) {
            int n = 0;
#pragma unroll
            for (int w = 0; w < kOwnRows / 32; ++w) {
                const int below = min(max(r - 32 * w, 0), 32);
                n += __popc(bits[w] & (uint32_t)((1ull << below) - 1ull));
            }
            return n;
        };
        if (s_bits[tid >> 5] >> (tid & 31) & 1) s_named[named_before(tid)] = (uint16_t)tid;
        for (int i = tid; i < n_refs; i += kOwnThreads) s_refs[i] = (uint16_t)named_before(s_refs[i]);
        n_named = named_before(kOwnRows);
    }
    own_barrier();  // the last one: from here on every wavefront works by itself, up to the reports

    const int64_t n_seg = (p.item_end - p.item_begin + kOwnSeg - 1) / kOwnSeg;
    const int64_t n_visit = (n_seg + p.seg_per_visit - 1) / p.seg_per_visit;
    const int64_t item_lim = p.item_end < p.n_items ? p.item_end : p.n_items;
    // the segments of this workgroup: the visits of its regions, one region after the other
    int region = blockIdx.x;
    int64_t vs = region, seg = vs * p.seg_per_visit;
    auto settle = [&]() __attribute__((always_inline)) {  // past the region's last visit: on to the next one that has some
        while (vs >= n_visit && region < p.groups) {
            region += gridDim.x;
            vs = region;
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
        ++seg;
        if (seg >= (vs + 1) * p.seg_per_visit || seg >= n_seg) {
            vs += p.groups;
            settle();
            seg = vs * p.seg_per_visit;
        }
    };
    // fill counts of a finished region (and of the ones without a visit behind it)
    auto report = [&](int from, int to) {
        __syncthreads();
        for (int c = tid; c < n_c; c += kOwnThreads) {
            const int q = s_query[c];
            const uint32_t n = s_cnt[c];
            p.cnt[(int64_t)q * p.groups + from] = n < (uint32_t)p.cap ? n : (uint32_t)p.cap;
            if (n > (uint32_t)p.cap) p.ovf[q] = 1u;
            s_cnt[c] = 0;
            for (int r = from + (int)gridDim.x; r < to && r < p.groups; r += (int)gridDim.x) p.cnt[(int64_t)q * p.groups + r] = 0;
        }
        __syncthreads();
    };
    // index words of the wavefront's 64 items: one to a named row
    constexpr int kIdx = kOwnRows / 64;
    uint64_t idx[kIdx];
    int idx_at[kIdx];
#pragma unroll
    for (int u = 0; u < kIdx; ++u) {
        const int x = max(min(lane + u * 64, n_named - 1), 0);  // (the last row again: an unconditional load)
        idx_at[u] = (p.m_bits <= kOwnAllRows ? min(x, p.m_bits - 1) : n_named > 0 ? (int)s_named[x] : 0) * kTileWords;
    }
    auto fetch = [&](int64_t sg) __attribute__((always_inline)) {
        const int64_t w0 = ((p.item_begin + sg * kOwnSeg) >> 6) + wv;
        const uint64_t* src = p.bloom + (w0 >> 4) * (int64_t)p.m_bits * kTileWords + (w0 & 15);
#pragma unroll
        for (int u = 0; u < kIdx; ++u)
            if (u * 64 < n_named) idx[u] = src[idx_at[u]];
    };
    // This wavefront's item rows (past the end the last row is repeated: no mask names it), 32 items to a half, and the
    // scales of the items this lane holds results of.  If the wavefront multiplied its last items, the first half of the
    // next ones is requested behind the products of the first half, into the same registers, and the second half
    // at the top of the segment; both before the masks are known.  Otherwise they are requested behind the masks: where
    // the filters pass little they are never read.
    own_i4 a[2][KS];
    float4 si[2][4];
    bool have0 = false;
    // (In two forms: whole words of items with vector loads of the scales, and any, for the words that are late.)
    auto rows = [&](auto whole, int s, int64_t my0) __attribute__((always_inline)) {
        constexpr bool kWhole = decltype(whole)::value;
        int64_t it = my0 + s * 32 + (lane & 31);
        if (!kWhole) it = min(it, p.n_items - 1);
        const own_i4* row = reinterpret_cast<const own_i4*>(p.items + it * D) + half;
#pragma unroll
        for (int k = 0; k < KS; ++k) a[s][k] = row[2 * k];
        int64_t it0 = my0 + 4 * half + s * 32;
        if (!kWhole) asm volatile("" : "+v"(it0));  // (16 offsets, kept in registers all the time otherwise)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (kWhole) {
                si[s][j] = *reinterpret_cast<const float4*>(p.iscale + it0 + j * 8);
            } else {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = p.iscale[min(it0 + j * 8 + i, p.n_items - 1)];
                si[s][j] = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    };
    int cur_E = -1000;        // every scale that this wavefront's factors cover is below 2^cur_E (none yet)
    float fix_scale = 0.0f;   // 2^(P - cur_E)
    const int first_region = region;
    settle();
    seg = vs * p.seg_per_visit;
    if (region < p.groups) {
        fetch(seg);
        const int64_t my0 = p.item_begin + seg * kOwnSeg + wv * 64;
        have0 = my0 + 64 <= p.n_items;
        if (have0) rows(std::true_type{}, 0, my0);
    }
    int filling = first_region;  // the region that the counters belong to
    while (region < p.groups) {
        if (region != filling) {
            report(filling, region);
            filling = region;
        }
        const int at_region = region;
        const int64_t item0 = p.item_begin + seg * kOwnSeg, my0 = item0 + wv * 64;
        auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kIdx; ++u)
                if (lane + u * 64 < n_named) s_idx[lane + u * 64] = idx[u];
        };
        // (the index block is stored in either branch: behind one where the rows may or may not have been
        // requested, the wait for the block is one for the rows as well)
        const bool early = have0;  // this wavefront multiplied its last items, and the first half of these rows is requested
        if (early) {
            stage();
            rows(std::true_type{}, 1, my0);
        } else {
            stage();
        }
        have0 = false;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        advance();
        if (region < p.groups) fetch(seg);
        const int64_t left = item_lim - my0;
        const uint64_t all = left >= 64 ? ~0ULL : left > 0 ? ((1ULL << left) - 1ULL) : 0ULL;
        uint32_t n_pass = 0;  // pairs that pass, over all queries
        for (int c = lane; c < cols; c += 64) {
            uint64_t m = 0;
            if (c < n_c) {
                m = all;
                const uint16_t* refs = s_refs + s_r0[c];
                const int rn = s_rn[c];
                int r = 0;
                for (; r + 4 <= rn; r += 4) {
                    const uint64_t m0 = s_idx[refs[r]], m1 = s_idx[refs[r + 1]], m2 = s_idx[refs[r + 2]], m3 = s_idx[refs[r + 3]];
                    m &= (m0 & m1) & (m2 & m3);
                }
                for (; r < rn; ++r) m &= s_idx[refs[r]];
            }
            s_mask[c] = m;
            n_pass += (uint32_t)__popcll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        const uint32_t incl = wave_scan_add(n_pass);
        const uint32_t total = lane_value(incl, 63);
        if (total <= (uint32_t)few) {
            uint32_t pos = incl - n_pass;
            for (int c = lane; c < cols; c += 64) {
                uint64_t m = s_mask[c];
                while (m) {
                    const int bit = __ffsll((long long)m) - 1;
                    m &= m - 1;
                    s_pairs[pos++] = (uint16_t)((c << 6) | bit);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            for (uint32_t k = lane; k < total; k += 64) {
                const int pr = s_pairs[k], c = pr >> 6;
                const int64_t item = my0 + (pr & 63);
                const int4* row = reinterpret_cast<const int4*>(p.items + item * D);
                int4 v[D / 16];
#pragma unroll
                for (int x = 0; x < D / 16; ++x) v[x] = row[x];
                const float s_i = p.iscale[item];
                int acc = 0;
#pragma unroll
                for (int x = 0; x < D / 16; ++x) acc = dot16(v[x], *reinterpret_cast<const int4*>(s_q + (size_t)c * DP + x * 16), acc);
                const uint64_t key = make_key(rescale(acc, s_sq[c], s_i), (uint32_t)item);
                if (key >= s_tau[c]) {
                    const uint32_t slot = atomicAdd(&s_cnt[c], 1u);
                    if (slot < (uint32_t)p.cap) p.cand[((int64_t)s_query[c] * p.groups + at_region) * p.cap + slot] = key;
                }
            }
            continue;
        }
        if (!early) {
            rows(std::false_type{}, 0, my0);
            rows(std::false_type{}, 1, my0);
        }
        // Lanes in which an admission is possible, emptied four lanes to an entry: the exact test of their pairs.
        int qn = 0;
        auto drain = [&]() __attribute__((always_inline)) {
            const int e = lane >> 2, h = lane & 3;
            if (e < qn) {
                const uint2 code = q_code[e];  // (admissible results, where the lane was: column, half, set)
                const int4 v4 = reinterpret_cast<const int4*>(q_val + e * 16)[h];
                const int c = (int)(code.y & 255u), bit0 = (int)(code.y >> 9) * 32 + 8 * h + 4 * (int)((code.y >> 8) & 1u);
                const float4 si4 = *reinterpret_cast<const float4*>(s_si + bit0);
                const float sq = s_sq[c];
                const uint64_t tau = s_tau[c];
                const int v[4] = {v4.x, v4.y, v4.z, v4.w};
                const float sv[4] = {si4.x, si4.y, si4.z, si4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint64_t key = make_key(rescale(v[i], sq, sv[i]), (uint32_t)my0 + (uint32_t)(bit0 + i));
                    if ((code.x >> (8 * h + i) & 1u) && key >= tau) {
                        const uint32_t slot = atomicAdd(&s_cnt[c], 1u);
                        if (slot < (uint32_t)p.cap) p.cand[((int64_t)s_query[c] * p.groups + at_region) * p.cap + slot] = key;
                    }
                }
            }
            qn = 0;
        };
        auto next_rows = [&]() __attribute__((always_inline)) {
            const int64_t next0 = p.item_begin + seg * kOwnSeg + wv * 64;  // (the segment advanced above)
            have0 = region < p.groups && next0 + 64 <= p.n_items;
            if (have0) rows(std::true_type{}, 0, next0);
        };
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            // The scales: exact ones for the tests, and fixed-point factors against a power of two above the scales met
            // so far.  A pair can only be admitted if dot * factor reaches its query's bound (rounded down by more than all
            // roundings involved).
            const float sv[16] = {si[s][0].x, si[s][0].y, si[s][0].z, si[s][0].w, si[s][1].x, si[s][1].y, si[s][1].z, si[s][1].w,
                                  si[s][2].x, si[s][2].y, si[s][2].z, si[s][2].w, si[s][3].x, si[s][3].y, si[s][3].z, si[s][3].w};
            if constexpr (ONE) {
                // A single block: factors for 16 items cost more than the exact scores of its 16 pairs, and few lanes pass.
                const int c = lane & 31;
                own_i16 acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0;
                const own_i4* qr = reinterpret_cast<const own_i4*>(s_q + (size_t)c * DP) + half;
#pragma unroll
                for (int k = 0; k < KS; ++k) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s][k], qr[2 * k], acc, 0, 0, 0);
                const float sq = s_sq[c];
                const uint64_t tau = s_tau[c];
                const float bound = tau ? key_score(tau) : -__builtin_inff();
                uint32_t over = 0;  // (scores not below the threshold's, also where a NaN is involved: compared as keys)
#pragma unroll
                for (int i = 0; i < 16; ++i) over |= !(rescale(acc[i], sq, sv[i]) < bound) ? 1u << (8 * (i >> 2) + (i & 3)) : 0u;
                over &= (uint32_t)(s_mask[c] >> (32 * s)) >> (4 * half);
                if (ballot(over != 0) != 0) {
                    uint32_t it0 = (uint32_t)my0 + 32u * s + 4u * half;
                    asm volatile("" : "+v"(it0));  // (16 ids to a half, kept in registers all the time otherwise)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int bit = 8 * (i >> 2) + (i & 3);
                        if (over >> bit & 1u) {
                            const uint64_t key = make_key(rescale(acc[i], sq, sv[i]), it0 + bit);
                            if (key >= tau) {
                                const uint32_t slot = atomicAdd(&s_cnt[c], 1u);
                                if (slot < (uint32_t)p.cap) p.cand[((int64_t)s_query[c] * p.groups + at_region) * p.cap + slot] = key;
                            }
                        }
                    }
                }
                if (s == 0) next_rows();
                continue;
            }
            if ((lane & 31) == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) *reinterpret_cast<float4*>(s_si + 32 * s + 8 * j + 4 * half) = si[s][j];
            }
            uint32_t top = 0;  // (scales are positive, so their bit patterns order as they do; others switch the bound off)
#pragma unroll
            for (int i = 0; i < 16; ++i) top = max(top, __float_as_uint(sv[i]));
            const float smax = __uint_as_float(max(lane_value(top, 0), lane_value(top, 32)));
            const bool cull = smax > 0x1p-90f && smax < 0x1p90f;
            const int E = (int)(__float_as_uint(smax) >> 23) - 126;  // 2^E > smax
            if (cull && E > cur_E) {  // (a handful of times to a launch; a bound for a larger exponent lets more pairs through)
                cur_E = E;
                fix_scale = __uint_as_float((uint32_t)(P - E + 127) << 23);
                for (int c = lane; c < cols; c += 64) {
                    const float tq = s_tq[c];
                    int neg = kPass;
                    if (tq > 0.0f)
                        neg = -min(__float2int_rd(fminf(tq * (fix_scale * 0.99999618530273f), 1.2e9f)), (1 << 30) + 1);  // (1 - 2^-18)
                    atomicMax(&s_neg[c], neg);
                }
            }
            int fix[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) fix[i] = cull ? max(__float2int_ru(sv[i] * fix_scale), 1) : 0;
            for (int b = 0; b < cols; b += 32) {
                const int c = b + (lane & 31);
                const uint32_t word = (uint32_t)(s_mask[c] >> (32 * s)) >> (4 * half);
                own_i16 acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0;
                const own_i4* qr = reinterpret_cast<const own_i4*>(s_q + (size_t)c * DP) + half;
#pragma unroll
                for (int k = 0; k < KS; ++k) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s][k], qr[2 * k], acc, 0, 0, 0);
                const int neg = cull ? s_neg[c] : kPass;
                // result i is item 32 s + 8 (i / 4) + 4 half + i % 4; the signs of the tests go to the bits of the mask word
                uint32_t below = 0;
#pragma unroll
                for (int j = 3; j >= 0; --j) {
                    if (j < 3) below <<= 4;
#pragma unroll
                    for (int i = 4 * j + 3; i >= 4 * j; --i)
                        below = __builtin_amdgcn_alignbit(below, (uint32_t)(__mul24(acc[i], fix[i]) + neg), 31);
                }
                const uint32_t over = word & ~below & 0x0F0F0F0Fu;
                const uint64_t hits = ballot(over != 0);
                if (hits == 0) continue;
                uint64_t m = hits;
                for (;;) {  // (more lanes than the queue holds go in rounds)
                    const int n = __popcll(m);
                    if (qn > 0 && qn + n > kOwnQueue) drain();
                    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    const bool mine = ((m >> lane) & 1ULL) && rank < kOwnQueue;
                    if (mine) {
                        int4* dst = reinterpret_cast<int4*>(q_val + (qn + rank) * 16);
#pragma unroll
                        for (int j = 0; j < 4; ++j) dst[j] = make_int4(acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]);
                        q_code[qn + rank] = make_uint2(over, (uint32_t)(c | (half << 8) | (s << 9)));
                    }
                    if (n <= kOwnQueue) {
                        qn = __builtin_amdgcn_readfirstlane(qn + n);
                        break;
                    }
                    qn = kOwnQueue;
                    m &= ~ballot(mine);
                }
            }
            if (s == 0) next_rows();
        }
        if (qn > 0) drain();
    }
    report(filling, p.groups);
}

// The first level of such a search, which admits every passing pair: the same products, 64 items (a region) to a
// wavefront.  An item's place among a filter's passing ones is its place in the region, so there are no counters; the
// number of bits of the mask word is the region's count.  Masks are formed from the index in memory (a wavefront has one
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
    const int64_t my0 = p.item_begin + (int64_t)region * 64;
    const int64_t lim = p.item_end < p.n_items ? p.item_end : p.n_items, left = lim - my0;
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
// Up to kOwnBlock queries of rows up to 192 bytes take the form of one block.  Calls with integer bounds and the
// queue -> with it, in us: 2 M x 64, 17 queries 95.8 -> 86.1; 5 M x 64, 24: 184 -> 169; 3.4 M x 96, 16: 144 -> 134;
// 4 M x 128, 16: 177 -> 169; 1.5 M x 192, 32: 109.7 -> 106.9.  At 256 bytes its scores do not fit the registers
// (1.5 M, 32 queries: 133 -> 137).
constexpr bool own_one_block(int d, size_t n_q) { return n_q <= (size_t)kOwnBlock && d <= 192; }
inline auto own_kernel(int d, size_t n_q) -> decltype(&scan_own_kernel<8, false>)
{
    const bool one = own_one_block(d, n_q);
    switch (d) {
    case 64: return one ? &scan_own_kernel<2, true> : &scan_own_kernel<2, false>;
    case 96: return one ? &scan_own_kernel<3, true> : &scan_own_kernel<3, false>;
    case 128: return one ? &scan_own_kernel<4, true> : &scan_own_kernel<4, false>;
    case 192: return one ? &scan_own_kernel<6, true> : &scan_own_kernel<6, false>;
    case 256: return &scan_own_kernel<8, false>;
    default: return nullptr;
    }
}
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
