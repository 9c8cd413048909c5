// Scan for batches whose queries hardly share filters (levels with thresholds in force).
//
// The wavefront dot-product scan gathers one item row per passing pair: at 10 M items x 256 bytes and 256
// filters that pass 5 % each, 2 G 16-byte gathers, 64 cache lines to an instruction.  Here a wavefront holds
// the rows of 64 items in registers and multiplies them with all queries by MFMA, whether a filter
// passes them or not; the filters decide which scores count.  That costs the same for every selectivity, so a
// wavefront whose filters pass few pairs (own_pairs) gathers after all, and one that did so requests the next
// items' rows only when their masks are known.
//
// Eight wavefronts take a segment of 512 items.  Its part of the index (the rows that some filter names, 64 bytes each,
// m <= kOwnRows) is brought to LDS with loads requested a segment ahead, and the mask words of all filters are formed
// there (a filter's rows fetched one by one from memory took longer than the products).  A mask word is what one
// wavefront needs for one query: lane l of the product's result holds query l % 32, and 16 of its items.
// The queries stay in LDS, padded by 16 bytes a row (an odd number of 16-byte pieces: no bank conflicts).
// 10 M x 256 bytes, 256 queries with filters of their own (5 % each), K = 500: the level after the first takes
// 1.33 ms, where gathering took 4.5 (the call 4.93 -> 1.65 ms); 778 k x 96 with 37 filter programs: 38 us.  Bound by
// the tests of the scores (six vector instructions to a pair, 2.6 G pairs) beside the products; two wavefronts to a SIMD
// leave part of the row loads uncovered.
//
// It takes the place of the gathering scan whatever the filters pass, which the host cannot know.  Calls on 3 M
// items, m = 512, K = 100, every query with a filter of its own, gathering -> this scan, in us (d = 256 unless
// said; with rows requested and all index rows staged before the masks were known, 16 queries took 280 to 300 throughout):
//   queries   0.05 % pass   0.2 %        1 %          5 %          the broadest (3 to 16 %)
//     16      112 -> 107    155 -> 122   161 -> 124   216 -> 186   410 -> 225
//     64      244 -> 124    353 -> 129   464 -> 182   527 -> 253   734 -> 269
//    256      909 -> 341   1458 -> 401  1909 -> 620  2127 -> 733  2222 -> 747
//     16, 64 bytes  99 -> 88   129 -> 95   128 -> 88   131 -> 103   200 -> 130
// one filter for 64 queries, 10 M x 192: 447 -> 176 at 0.02 %, 807 -> 339 at 0.5 %, 825 -> 543 at 5 %; behind cluster probing
// (600 of 4096 clusters, 3 M x 128, 32 queries) 326 -> 243.
#pragma once
#include "st_search_kernels.h"

namespace st {

constexpr int kOwnThreads = 512;
constexpr int kOwnSeg = 512;            // items of a segment
constexpr int kOwnWords = kOwnSeg / 64; // one mask word per wavefront
constexpr int kOwnCols = 256;           // queries resident at a time (one row of the grid)
constexpr int kOwnRows = 512;           // signature rows of the index, at most
// Items of a level, at least: two segments to each of the workgroups that are resident.  (Whether the candidate
// regions have room for segments of this size is the plan's to say: level_takes_segments.)
constexpr int64_t kOwnMinItems = 512 * kOwnSeg;
constexpr int kOwnAllRows = 64;         // an index of no more rows is staged whole
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
    return c * (d + 16) + c * kOwnWords * 8 + (size_t)m_bits * kOwnWords * 8 + kOwnRowRefs * 2 + c * (8 + 4 * 5) +
           own_pairs((int)c) * (kOwnThreads / 64) * 2 + kOwnRows * 2 + kOwnRows / 8;
}
static_assert(own_lds_bytes(kOwnCols, 256, kOwnRows) <= 160 * 1024, "LDS of a compute unit");

typedef int own_i4 __attribute__((ext_vector_type(4)));
typedef int own_i16 __attribute__((ext_vector_type(16)));

// LDS exchange without waiting for the global loads in flight (they go to registers of their own).
__device__ inline void own_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// d = 32 * KS.  Grid (workgroups, ceil(queries / kOwnCols)); segments start at multiples of 512 items.  One
// workgroup to a compute unit is resident (registers), so that many are launched and each takes several
// regions in turn: the queries and tables are brought to LDS once.
template <int KS>
__global__ __launch_bounds__(kOwnThreads) void scan_own_kernel(ScanParams p, int n_refs)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char own_lds[];
    constexpr int D = 32 * KS, DP = D + 16;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, half = lane >> 5;
    const int n_q = p.grp_q_off[p.n_groups];
    const int cols = own_cols(n_q), c0 = (int)blockIdx.y * kOwnCols, n_c = min(n_q - c0, cols);
    unsigned char* at = own_lds;
    int8_t* s_q = reinterpret_cast<int8_t*>(at);                  at += (size_t)cols * DP;          // [cols][DP]
    uint64_t* s_mask = reinterpret_cast<uint64_t*>(at);           at += (size_t)cols * kOwnWords * 8;
    uint64_t* s_idx = reinterpret_cast<uint64_t*>(at);            at += (size_t)p.m_bits * kOwnWords * 8;  // [m_bits][kOwnWords]
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
    uint32_t* s_bits = reinterpret_cast<uint32_t*>(at);           // [kOwnRows / 32]

    if (tid < kOwnRows / 32) s_bits[tid] = 0;
    for (int c = tid; c < cols; c += kOwnThreads) {
        const int q = c < n_c ? p.grp_q[c0 + c] : -1;
        uint64_t t = ~0ULL;
        if (q >= 0)
            for (int pp = 0; pp < p.tau_parts; ++pp) t = min(t, p.tau[(int64_t)q * kTauParts + pp]);
        s_query[c] = q;
        s_tau[c] = t;
        s_sq[c] = q >= 0 ? p.qscale[q] : 0.0f;
        s_cnt[c] = 0;
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
        own_barrier();
    }

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
    // its index block: 4 pieces of 16 bytes to a named row, kOwnRows * 4 / kOwnThreads to a thread
    constexpr int kIdx = kOwnRows * 4 / kOwnThreads;
    const int n_idx = n_named * 4;
    own_i4 idx[kIdx];
    int idx_at[kIdx];
#pragma unroll
    for (int u = 0; u < kIdx; ++u) {
        const int x = min(tid + u * kOwnThreads, n_idx - 1);  // (the last piece again: an unconditional load)
        idx_at[u] = x < 0 ? 0 : (p.m_bits <= kOwnAllRows ? x >> 2 : (int)s_named[x >> 2]) * (kTileWords / 2) + (x & 3);
    }
    auto fetch = [&](int64_t sg) __attribute__((always_inline)) {
        const int64_t w0 = (p.item_begin + sg * kOwnSeg) >> 6;
        const own_i4* src = reinterpret_cast<const own_i4*>(p.bloom + (w0 >> 4) * (int64_t)p.m_bits * kTileWords) + ((w0 & 15) >> 1);
#pragma unroll
        for (int u = 0; u < kIdx; ++u) idx[u] = src[idx_at[u]];
    };
    uint32_t last = ~0u;  // pairs that passed among this wavefront's last items; if it multiplied those, the next items' rows are requested before their masks are known
    const int first_region = region;
    settle();
    seg = vs * p.seg_per_visit;
    if (region < p.groups) fetch(seg);
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
            for (int u = 0; u < kIdx; ++u) {
                const int x = tid + u * kOwnThreads;
                if (x < n_idx) reinterpret_cast<own_i4*>(s_idx)[x] = idx[u];
            }
        };
        // This wavefront's item rows (past the end the last row is repeated: no mask names it), and the scales of the
        // items this lane holds results of.  They are requested before the masks are known if the wavefront
        // multiplied its last items, and behind them otherwise: where the filters pass little they are never read.
        own_i4 a[2][KS];
        float si[2][16];
        // (In two forms: whole words of items with vector loads of the scales, and any, for the words that are late.)
        auto rows = [&](auto whole) __attribute__((always_inline)) {
            constexpr bool kWhole = decltype(whole)::value;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                int64_t it = my0 + s * 32 + (lane & 31);
                if (!kWhole) it = min(it, p.n_items - 1);
                const own_i4* row = reinterpret_cast<const own_i4*>(p.items + it * D) + half;
#pragma unroll
                for (int k = 0; k < KS; ++k) a[s][k] = row[2 * k];
            }
            int64_t it0 = my0 + 4 * half;
            if (!kWhole) asm volatile("" : "+v"(it0));  // (32 offsets, kept in registers all the time otherwise)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (kWhole) {
                        const float4 v = *reinterpret_cast<const float4*>(p.iscale + it0 + s * 32 + j * 8);
                        si[s][4 * j] = v.x;
                        si[s][4 * j + 1] = v.y;
                        si[s][4 * j + 2] = v.z;
                        si[s][4 * j + 3] = v.w;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) si[s][4 * j + i] = p.iscale[min(it0 + s * 32 + j * 8 + i, p.n_items - 1)];
                    }
                }
        };
        // (the index block is stored in either branch: behind one where the rows may or may not have been
        // requested, the wait for the block is one for the rows as well)
        const bool early = last > (uint32_t)few && my0 + 64 <= p.n_items;
        if (early) {
            rows(std::true_type{});
            stage();
        } else {
            stage();
        }
        own_barrier();
        advance();
        if (region < p.groups) fetch(seg);
        for (int i = tid; i < cols * kOwnWords; i += kOwnThreads) {
            const int c = i / kOwnWords, w = i % kOwnWords;
            uint64_t m = 0;
            if (c < n_c) {
                const int64_t left = item_lim - (item0 + w * 64);
                m = left >= 64 ? ~0ULL : left > 0 ? ((1ULL << left) - 1ULL) : 0ULL;
                const uint16_t* refs = s_refs + s_r0[c];
                const int rn = s_rn[c];
                int r = 0;
                for (; r + 4 <= rn; r += 4) {
                    const uint64_t m0 = s_idx[refs[r] * kOwnWords + w], m1 = s_idx[refs[r + 1] * kOwnWords + w];
                    const uint64_t m2 = s_idx[refs[r + 2] * kOwnWords + w], m3 = s_idx[refs[r + 3] * kOwnWords + w];
                    m &= (m0 & m1) & (m2 & m3);
                }
                for (; r < rn; ++r) m &= s_idx[refs[r] * kOwnWords + w];
            }
            s_mask[c * kOwnWords + w] = m;
        }
        own_barrier();
        // pairs that pass, over all queries
        uint32_t n_pass = 0;
        for (int c = lane; c < cols; c += 64) n_pass += (uint32_t)__popcll(s_mask[c * kOwnWords + wv]);
        const uint32_t incl = wave_scan_add(n_pass);
        const uint32_t total = lane_value(incl, 63);
        if (total <= (uint32_t)few) {
            last = total;
            uint32_t pos = incl - n_pass;
            for (int c = lane; c < cols; c += 64) {
                uint64_t m = s_mask[c * kOwnWords + wv];
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
        if (!early) rows(std::false_type{});
        last = total;
        for (int b = 0; b < cols; b += 32) {
            const int c = b + (lane & 31);
            const uint64_t word = s_mask[c * kOwnWords + wv];
            if (ballot(word != 0) == 0) continue;
            own_i16 acc[2];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[s][i] = 0;
            const own_i4* qr = reinterpret_cast<const own_i4*>(s_q + (size_t)c * DP) + half;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const own_i4 bq = qr[2 * k];
                acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0][k], bq, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[1][k], bq, acc[1], 0, 0, 0);
            }
            const float sq = s_sq[c];
            const uint64_t tau = s_tau[c];
            // A score below the threshold's cannot be admitted; the others (also where a NaN is involved) are
            // compared as keys.
            const float bound = tau ? bits_score((uint32_t)(tau >> 32)) : -__builtin_inff();
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                // result i of set s is item 32 s + 8 (i / 4) + 4 half + i % 4
                uint32_t over = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float sc = rescale(acc[s][i], sq, si[s][i]);
                    over |= !(sc < bound) ? 1u << (8 * (i >> 2) + (i & 3)) : 0u;
                }
                over &= (uint32_t)(word >> (32 * s)) >> (4 * half);
                if (ballot(over != 0) != 0) {
                    uint32_t it0 = (uint32_t)my0 + 32u * s + 4u * half;
                    asm volatile("" : "+v"(it0));  // (16 ids to a set, kept in registers all the time otherwise)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int bit = 8 * (i >> 2) + (i & 3);
                        if (over >> bit & 1) {
                            const float sc = rescale(acc[s][i], sq, si[s][i]);
                            const uint64_t key = make_key(sc, it0 + bit);
                            if (key >= tau) {
                                const uint32_t slot = atomicAdd(&s_cnt[c], 1u);
                                if (slot < (uint32_t)p.cap) p.cand[((int64_t)s_query[c] * p.groups + at_region) * p.cap + slot] = key;
                            }
                        }
                    }
                }
            }
        }
    }
    report(filling, p.groups);
}

// The kernel for rows of d bytes, or null.  (One copy of the kernel to a length: the lengths the MFMA scan has, as far as
// a workgroup's registers hold the rows of 64 items, and 96 and 192 between them; others go to the gathering scan.)
inline auto own_kernel(int d) -> decltype(&scan_own_kernel<8>)
{
    switch (d) {
    case 64: return &scan_own_kernel<2>;
    case 96: return &scan_own_kernel<3>;
    case 128: return &scan_own_kernel<4>;
    case 192: return &scan_own_kernel<6>;
    case 256: return &scan_own_kernel<8>;
    default: return nullptr;
    }
}

}  // namespace st
