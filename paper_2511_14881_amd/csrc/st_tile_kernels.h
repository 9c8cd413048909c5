// Form of the int8 MFMA scan for the levels that admit by threshold, for batches of up to 32 filters whose
// resident queries leave room for one workgroup to a compute unit (d <= 256): Bloom test
// (Sec. 4.1 Eq. 4), compaction, contraction and admission (Sec. 4.2, Algorithm 1 phase 3) as in
// scan_mfma_kernel, but 64 passing items of one filter are contracted at a time.
//
//   * A unit of 64 items (32 with d = 256) stays in registers while the filter's query rows come by from LDS, 32 at a
//     time (v_mfma_i32_32x32x32_i8): what a unit costs once -- its place in the lists, the scales, the request for
//     the next unit's rows -- is paid for that many items, and an operand read serves two products.
//   * Units are full.  What a filter's list holds beyond a whole number of units is carried, as item numbers, to the
//     wavefront's next segments, and flushed when the wavefront runs out of them.
//   * The rows of the next unit, from whatever segment, are requested before the current one is contracted.
//   * Plain search: a lane holds one query and 16 items of a product, so the bound is one 24-bit multiply to a pair
//     and one compare to 16 pairs: max over the items of dot * F against the query's bound, F the item's
//     scale in fixed point against a power of two above the scales met so far.  A pair can only be admitted if
//     its product reaches the bound (rounded down by more than all roundings involved); lanes in which one does
//     are queued with their 16 dot products, and the exact fp32 score, key and threshold test run where the queue
//     is drained.
//   * Weighted search: the operands change places, so that a lane holds an item and four times four consecutive
//     rows, and the aggregate of a query's tasks stays in the lane, as in scan_mfma_kernel.
//
// Bound, with many query rows to a filter, by the issue of its wavefronts: 60 vector instructions beside 8 products of 32
// cycles to 32 rows x 64 items (two wavefronts to a SIMD; a product hides about six of them), and what a hit costs (queue
// and exact test).  20 M x 128, 1024 queries under two filters: the two levels after the first 1103 + 1554 us with
// 16-item units (scan_mfma_kernel's form), 855 + 1127 here; the call 2.93 -> 2.30 ms.  With few rows to a filter, by the
// round trips of a unit: 5 M x 128, 128 queries x 4 tasks, 8 filters: 156 -> 145 us; 10 M x 256, 256 queries, 8 filters: 272
// -> 256 us.  Measured and not kept: 32 items to a unit and sixteen wavefronts (spills, more instructions to a product:
// 1.55 ms where two and 64 take 1.13); tests of one product beside the next one's within the wavefront (registers for
// both: 1.29 against 1.21 ms); 16 x 16 products (1.32 ms: half the vector instructions hide behind them); the queue
// with whole lanes of 16 results (1.02 instead of 0.84 ms in the level with two hits to 2048 pairs).
#pragma once
#include "st_mfma_kernels.h"

namespace st {

constexpr int kTileWaves = 8;    // wavefronts of a workgroup
constexpr int kTileGroups = 32;  // filters of a launch, at most
constexpr int kTileQueue = 64;   // queued lanes of a wavefront
constexpr int tile_unit(int d) { return d <= 128 ? 64 : 32; }  // items contracted at a time (their rows are held twice over, in registers)
// Items that a filter hands a wavefront over the level, at least (an average over the batch): with fewer, units go out
// partly filled at the end and cost more than they save.
constexpr int tile_min_items(int d) { return d <= 128 ? 48 : 100; }
// Items of the level to a wavefront, whether they pass or not, at least.  The form costs a level some 5 us more than the
// others (set-up, the flush of every filter's last unit), and saves by the items: most where one query row tile comes by
// for many rows of a filter, and less where scores are exact from the start (weighted) or the products of a unit are few (d = 256,
// two 16-row blocks to a filter and row of workgroups).  Both thresholds from 860 calls of this shape, 0.3 to 16 M items, 1 to 24
// filters of 2 to 26 %, each timed with this form wherever it fits and without it.  Calls without -> with it, in us:
//   plain, d <= 128:          8 M x 128, 500 queries, one filter at 10 %   297 -> 227;  0.6 M x 128, 500, 4 at 17 %  158 -> 149
//   weighted, d <= 128:       1 M x 128, 250 x 2 tasks, 3 at 19 %   123 -> 131;  2 M, 3 at 19 %  162 -> 164;  4 M, 4 at 9 %  174 -> 165
//   d = 256, 2 blocks:        3.4 M, 256 queries, 8 at 11 %   218 -> 225;  6.9 M, 200, 8 at 8 %  282 -> 292;  8.8 M, 256, 8 at 4 %  242 -> 237
//            ... 4 tasks and more than 8 filters:  2.7 M, 60 queries, 14 at 9 %   237 -> 227  (2 tasks, 6.7 M, 15 at 7 %: 350 -> 365)
//   d = 256, up to 8 blocks:  1.1 M, 200 queries, 4 at 17 %   130 -> 132;  2 M, 200, 2 at 22 %  141 -> 136
//   d = 256, more:            1.1 M, 256 queries, one at 18 %   131 -> 122
//   d = 256, weighted, T = 1: 2 M, 300 queries, 3 at 19 %   196 -> 202;  4.7 M, 2 at 8 %  202 -> 184
//                      T = 2: 1 M, 250 queries, 4 at 17 %   134 -> 136;  2 M, 4 at 9 %  149 -> 144
//                      T = 4: 0.7 M, 130 queries, 2 at 22 %  127 -> 121
constexpr int tile_min_span(int d, bool weighted, int n_tasks, int n_blocks, int n_groups, int q_split)
{
    if (d <= 128) return !weighted ? 0 : n_tasks == 4 ? 950 : 1000;
    if (n_blocks <= 2 * n_groups * q_split) return n_tasks == 4 && n_groups > kMfmaFilterBatch ? 1000 : 3500;
    if (!weighted) return n_blocks <= 8 * n_groups * q_split ? 700 : 0;
    return n_tasks == 1 ? 1500 : n_tasks == 2 ? 1400 : 0;
}
constexpr int kTileRing = 8;     // units whose items are remembered for the queue

// Byte offsets of the workgroup's LDS (the resident queries are at 0, rows of d + 16 bytes: an odd number of 16-byte
// pieces, no bank conflicts).  Row tables have room for a block more: a tile may reach past the last one.
struct TileLds {
    int32_t bound, sq, tau64, qrow, cnt, prow, grp, list, carry, ids, scl, fix, thr, queue, code, total;
    int32_t lists;  // filters whose lists of a segment are in place at a time
    unsigned long long min_pairs;  // passing pairs of the first level from which the units fill
};

inline TileLds tile_lds(int rows_local, int d, int n_tasks, bool weighted, int n_groups, int slots, int seg_stride, int lists)
{
    constexpr int NW = kTileWaves;
    const int rows = rows_local + 16, unit = tile_unit(d);
    TileLds l;
    l.lists = lists;
    int off = 0;
    auto take = [&](int bytes) { const int o = off; off = (off + bytes + 15) / 16 * 16; return o; };
    take(rows * (d + 16));
    l.bound = take(rows * 4);
    l.sq = take(rows * 4);
    l.tau64 = take((rows / n_tasks + 1) * 8);
    l.qrow = take(rows * 4);
    l.cnt = take((slots * (rows_local / n_tasks + 1) + 1) * 4);  // + the segment counter
    l.prow = take(n_groups * kPrefetchStride * 4);
    l.grp = take((3 * n_groups + 1) * 4);
    l.list = take(NW * lists * seg_stride);
    l.carry = take(NW * n_groups * unit * 4);
    l.ids = take(NW * kTileRing * unit * 4);
    l.scl = take(NW * kTileRing * unit * 4);
    l.fix = take(weighted ? 0 : NW * unit * 4);
    l.thr = take(weighted ? 0 : rows * 4);
    l.queue = take(NW * kTileQueue * (4 / n_tasks) * 4);
    l.code = take(NW * kTileQueue * 4);
    l.total = off;
    return l;
}

typedef int tile_i16 __attribute__((ext_vector_type(16)));

template <int KS, int TT, bool WEIGHTED>
__device__ __forceinline__ void scan_tile_body(const ScanParams& p, const MfmaParams& mp, const TileLds& L)
{
    static_assert(WEIGHTED || TT == 1, "plain search has one task to a query");
    constexpr int D = KS * 64, DP = D + 16;
    constexpr int NW = kTileWaves, kThreads = NW * 64;
    constexpr int KK = 2 * KS;  // contraction steps of 32 bytes
    constexpr int CH = D / 16;
    constexpr int FB = kMfmaFilterBatch;
    constexpr int UNIT = tile_unit(D), NS = UNIT / 32;  // items of a unit, products side by side
    constexpr int RING = kTileRing;
    constexpr int PR = NS == 2 && !WEIGHTED ? 8 : kPrefetchStride;  // signature rows requested a segment ahead (registers)
    constexpr int P = KS == 1 ? 10 : (KS == 2 ? 9 : 8);  // bits of a scale in fixed point: |dot| <= 2^(14 + log2 d), the product at most 2^30
    static_assert(KS == 1 || KS == 2 || KS == 4, "dot products must fit 23 bits for the 24-bit multiply");
    constexpr int NV = 4 / TT;  // values of a queued lane: four dot products (plain) or their aggregates (weighted)
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int seg_stride = mp.seg_stride;
    int8_t* s_q = reinterpret_cast<int8_t*>(lds);
    float* s_bound = reinterpret_cast<float*>(lds + L.bound);  // [rows] tau's score (-inf: none; padding: +inf)
    float* s_sq = reinterpret_cast<float*>(lds + L.sq);
    uint64_t* s_tau64 = reinterpret_cast<uint64_t*>(lds + L.tau64);  // [rows / TT] (padding: above every key)
    int* s_qrow = reinterpret_cast<int*>(lds + L.qrow);
    int* s_thr = reinterpret_cast<int*>(lds + L.thr);          // [rows] plain: integer bounds, for the largest exponent so far
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(lds + L.cnt);
    int* s_prow = reinterpret_cast<int*>(lds + L.prow);  // [groups][kPrefetchStride]
    int* s_glrow = reinterpret_cast<int*>(lds + L.grp);  // [groups] first local query row of the group
    int* s_gnblk = s_glrow + p.n_groups;                 // [groups] local 16-row blocks of the group
    int* s_rowoff = s_gnblk + p.n_groups;                // [groups + 1]

    // (the wavefront's number as the scalar it is: what follows from it stays in scalar registers)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = mp.q_split, y = blockIdx.y;
    const int l32 = lane & 31, half = lane >> 5;
    // wave-private state
    uint8_t* s_list = reinterpret_cast<uint8_t*>(lds + L.list) + wave * L.lists * seg_stride;        // [lists][seg] this segment's passing items
    uint32_t* s_carry = reinterpret_cast<uint32_t*>(lds + L.carry) + wave * p.n_groups * UNIT;       // [groups][UNIT] items carried over
    uint32_t* s_ids = reinterpret_cast<uint32_t*>(lds + L.ids) + wave * RING * UNIT;            // [RING][UNIT] items of a unit
    float* s_scl = reinterpret_cast<float*>(lds + L.scl) + wave * RING * UNIT;                  // [RING][UNIT] their scales
    int* s_fix = reinterpret_cast<int*>(lds + L.fix) + wave * UNIT;                                  // [UNIT] ... in fixed point
    uint32_t* q_val = reinterpret_cast<uint32_t*>(lds + L.queue) + wave * kTileQueue * NV;           // [queue][NV]
    uint32_t* q_code = reinterpret_cast<uint32_t*>(lds + L.code) + wave * kTileQueue;

    // ---- schedule: as in scan_mfma_kernel (visits dealt to workgroups, segments drawn by the wavefronts from a
    // counter in LDS)
    const int seg_items = p.seg_items;
    const int SW = seg_items >> 6;
    const int spv = p.seg_per_visit;
    const int64_t item_lim = p.item_end < p.n_items ? p.item_end : p.n_items;
    const int n_seg = (int)((p.item_end - p.item_begin + seg_items - 1) / seg_items);
    const int n_visit = (n_seg + spv - 1) / spv;
    const int wg_visits = (int)blockIdx.x < n_visit ? (n_visit - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x : 0;
    const int wg_segs = wg_visits * spv;
    const int R = mp.region_slots;
    const int nq_pad = mp.rows_local / TT + 1;
    const int nf = p.n_groups;  // at most kTileGroups
    const int n_batches = (nf + FB - 1) / FB;  // a segment is taken FB filters at a time
    uint32_t* s_work = s_cnt + R * nq_pad;
    auto seg_first = [&](int num) -> int64_t {
        const int i = num / spv;
        return p.item_begin + (int64_t)(((int)blockIdx.x + i * (int)gridDim.x) * spv + (num - i * spv)) * seg_items;
    };
    auto in_sample = [&](int64_t first) -> bool {  // the 64-item word at `first` belongs to the first level's sample
        if (p.samp_role != 2) return false;
        const uint32_t fw = (uint32_t)(first >> 6), sw = (uint32_t)(p.samp_stride_items >> 6);  // in words: 32 bits do
        const uint32_t j = fw / sw;
        return j < (uint32_t)p.samp_segs && fw - j * sw < (uint32_t)(p.samp_seg_items >> 6);
    };

    // ---- workgroup-wide set-up: tables and the resident-query image (written by an earlier launch of the search)
    // into LDS; all reads of a share are issued before anything is stored
    const int n_prow = nf * kPrefetchStride;
    const int n_piece = mp.rows_local * CH;
    const int n_imgrow = mp.rows_local;
    const int4* gq = reinterpret_cast<const int4*>(mp.img_q + (int64_t)y * mp.rows_local * D);
    auto piece = [&](int i) {  // where piece i of the image belongs (the image is laid out for scan_mfma_kernel)
        const int r = i / CH, c = (i % CH) ^ swz<KS>(r);
        return reinterpret_cast<int4*>(s_q + r * DP + c * 16);
    };
    auto row_tau = [&](int lr) -> uint64_t {
        uint64_t t64 = ~0ULL;
        for (int pp = 0; pp < p.tau_parts; ++pp)
            t64 = min(t64, mp.img_tau[(int64_t)(y * (mp.rows_local / TT) + lr / TT) * kTauParts + pp]);
        return t64;
    };
    auto row_store = [&](int lr, int qrow, float sq, uint64_t t64) {
        s_qrow[lr] = qrow;
        s_sq[lr] = sq;
        s_bound[lr] = qrow < 0 ? __builtin_inff() : t64 ? key_score(t64) : -__builtin_inff();
        if ((lr % TT) == 0) s_tau64[lr / TT] = qrow >= 0 ? t64 : ~0ULL;
        if (!WEIGHTED) s_thr[lr] = 0x7FFFFFFF;
    };
    {
        static_assert(kTileGroups * kPrefetchStride <= kThreads && kTileGroups <= 64, "a table entry per thread, a filter per lane");
        const int v_prow = mp.prow[tid < n_prow ? tid : 0];
        const int gc = tid <= nf ? tid : 0;
        const int v_rowoff = p.grp_row_off[gc];
        const int v_b0 = mp.grp_blk_off[gc < nf ? gc : 0], v_b1 = mp.grp_blk_off[gc < nf ? gc + 1 : 0];
        int4 v_img[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = tid + u * kThreads;
            v_img[u] = i < n_piece ? gq[i] : make_int4(0, 0, 0, 0);
        }
        int v_qrow = -1;
        float v_sq = 0.0f;
        uint64_t v_tau = 0;
        if (tid < n_imgrow) {
            v_qrow = mp.img_qrow[y * mp.rows_local + tid];
            v_sq = mp.img_sq[y * mp.rows_local + tid];
            v_tau = row_tau(tid);
        }
        if (tid < n_prow) s_prow[tid] = v_prow;
        if (tid <= nf) {
            s_rowoff[tid] = v_rowoff;
            if (tid < nf) {  // the group's 16-row blocks that live in this row of workgroups
                const int bf = v_b0 + ((y - v_b0) % S + S) % S;
                s_gnblk[tid] = bf < v_b1 ? (v_b1 - bf + S - 1) / S : 0;
                s_glrow[tid] = (bf / S) * 16;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = tid + u * kThreads;
            if (i < n_piece) *piece(i) = v_img[u];
        }
        if (tid < n_imgrow) row_store(tid, v_qrow, v_sq, v_tau);
    }
    for (int i = tid; i < R * nq_pad; i += kThreads) s_cnt[i] = 0;
    if (tid == 0) *s_work = (uint32_t)NW;
    for (int i = tid + 8 * kThreads; i < n_piece; i += kThreads) *piece(i) = gq[i];
    for (int lr = tid + kThreads; lr < n_imgrow; lr += kThreads)
        row_store(lr, mp.img_qrow[y * mp.rows_local + lr], mp.img_sq[y * mp.rows_local + lr], row_tau(lr));
    __syncthreads();

    // ---- Bloom words: lane (gi * SW + w) owns word w of filter gi of a batch.
    const int pr_gi = lane / SW, pr_w = lane - pr_gi * SW;
    const int glrow = lane < nf ? s_glrow[lane] : 0;
    const int gnblk = lane < nf ? s_gnblk[lane] : 0;
    const int all_rows = (int)lane_value(wave_max_u32((uint32_t)(lane < nf ? s_rowoff[lane + 1] - s_rowoff[lane] : 0)), 63);  // of the longest filter
    struct Stage {
        int num;    // segment number within the workgroup (>= wg_segs: none, the work has run out)
        int batch;  // filter batch
    };
    uint64_t pre[PR];  // the first rows' words of the stage to come
    // (rows are requested eight at a time; a shorter filter repeats its first one)
    auto bloom_eight = [&](const uint64_t* base, int g, int r0, uint64_t* v) {
        const int* rows = s_prow + g * kPrefetchStride;
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = base[(int64_t)max(rows[r0 + r] >= 0 ? rows[r0 + r] : rows[0], 0) * kTileWords];
    };
    auto bloom_request = [&](const Stage& st) {
        const int64_t gw = (seg_first(st.num) >> 6) + pr_w;
        const int g = st.batch * FB + pr_gi;
        if (pr_gi >= FB || g >= nf || st.num >= wg_segs || gw * 64 >= item_lim) return;
        const uint64_t* base = p.bloom + ((gw >> 4) * (int64_t)p.m_bits) * kTileWords + (gw & 15);
        bloom_eight(base, g, 0, pre);
        if (PR > 8 && all_rows > 8) bloom_eight(base, g, 8, pre + PR - 8);
    };
    auto bloom_word = [&](const Stage& st) -> uint64_t {  // my mask word of the stage
        const int64_t gw = (seg_first(st.num) >> 6) + pr_w;
        const int64_t first = gw * 64;
        const int g = st.batch * FB + pr_gi;
        if (pr_gi >= FB || g >= nf || first >= item_lim || in_sample(first)) return 0ULL;
        const int64_t left = item_lim - first;
        uint64_t mask = left >= 64 ? ~0ULL : ((1ULL << left) - 1ULL);
        const int r_at = s_rowoff[g], n_rows = s_rowoff[g + 1] - r_at;
        if (n_rows == 0) return mask;
#pragma unroll
        for (int r = 0; r < 8; ++r) mask &= pre[r];
        if (all_rows > 8) {
            const uint64_t* base = p.bloom + ((gw >> 4) * (int64_t)p.m_bits) * kTileWords + (gw & 15);
            uint64_t late[8];
            if (PR == 8) bloom_eight(base, g, 8, late);
#pragma unroll
            for (int r = 0; r < 8; ++r) mask &= PR == 8 ? late[r] : pre[PR - 8 + r];
            for (int r = kPrefetchStride; r < n_rows; ++r) mask &= base[(int64_t)p.grp_rows[r_at + r] * kTileWords];
        }
        return mask;
    };
    Stage stage{wave, 0};  // the next one, whose words are requested
    int next_num = 0;      // segment behind the stage's
    bloom_request(stage);

    // ---- lists of the segment in place, and the position in them
    int64_t item0 = 0;     // first item of the segment in place
    uint32_t* cnt_s = s_cnt;
    int region = 0;
    bool flush = false;    // the wavefront's last segment: partial units too
    int gcur = 0;          // lane f: this segment's passing items of filter f of the batch ...
    int glow = 0;          // ... of its lower 256 items
    int gnc = 0;           // lane f: items carried over in front of those of filter f (of all)
    uint64_t seg_mask = 0; // mask word of my (filter, word) pair
    int seg_pos = 0;       // ... and the place of its items in the filter's list
    bool seg_full = false; // many items pass
    int batch_g0 = 0, batch_end = 0;  // filters of the batch in place
    int list_g0 = 0;       // first filter whose list is in place
    int gen_gi = 0, gen_b0 = 0, gen_tot = 0, gen_nc = 0, gen_low = 0;  // next unit: filter, place in its items
    auto gen_fetch = [&]() {
        gen_nc = __builtin_amdgcn_readlane(gnc, gen_gi);
        gen_tot = gen_nc + __builtin_amdgcn_readlane(gcur, gen_gi - batch_g0);
        gen_low = __builtin_amdgcn_readlane(glow, gen_gi - batch_g0);
        gen_b0 = 0;
    };
    // Item `at` of filter f: carried ones, then this segment's.  One 4-byte LDS read either way (a carried item
    // number, or the aligned word that holds the list's byte).
    auto entry_item = [&](int f, int at, int nc, int low) -> uint32_t {
        const int cj = at - nc;  // place in this segment's list (negative: a carried entry)
        const unsigned char* src = cj < 0 ? reinterpret_cast<const unsigned char*>(s_carry + f * UNIT + at)
                                          : s_list + (f - list_g0) * seg_stride + (cj & ~3);
        const uint32_t v = *reinterpret_cast<const uint32_t*>(src);
        const uint32_t here = (uint32_t)item0 + ((v >> ((cj & 3) * 8)) & 255u) + (cj >= low ? 256u : 0u);
        return cj < 0 ? v : here;
    };
    auto build_lists = [&](int g0) {  // set bits of the filters from g0 on into their lists, in item order
        list_g0 = g0;
        const int l0 = g0 - batch_g0;
        if (seg_full) {  // word by word, a lane to a bit
            const int w1 = min(l0 + L.lists, batch_end - batch_g0) * SW;
            for (int w = l0 * SW; w < w1; ++w) {
                const uint32_t lo = lane_value((uint32_t)seg_mask, w), hi = lane_value((uint32_t)(seg_mask >> 32), w);
                const int rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
                const int gi = w / SW;
                uint8_t* list = s_list + (gi - l0) * seg_stride + (int)lane_value((uint32_t)seg_pos, w);
                if ((((uint64_t)hi << 32) | lo) >> lane & 1) list[rank] = (uint8_t)((w - gi * SW) * 64 + lane);
            }
        } else if (pr_gi >= l0 && pr_gi < l0 + L.lists) {  // a lane to a word
            uint8_t* list = s_list + (pr_gi - l0) * seg_stride + seg_pos;
            for (uint64_t m = seg_mask; m; m &= m - 1) *list++ = (uint8_t)(pr_w * 64 + __ffsll((long long)m) - 1);
        }
    };
    // Positions on the wavefront's next unit, through as many segments as it takes; false: none is left.
    auto next_unit = [&]() -> bool {
        for (;;) {
            while (gen_gi < batch_end) {
                const int left = gen_tot - gen_b0;
                if (left >= UNIT || (flush && left > 0)) return true;
                if (!flush && left > 0 && (gen_b0 > 0 || gen_tot > gen_nc)) {
                    // what is left over goes to the front of the filter's items (reads before writes: the same wavefront)
                    const uint32_t v = entry_item(gen_gi, min(gen_b0 + lane, gen_tot - 1), gen_nc, gen_low);
                    if (lane < left) s_carry[gen_gi * UNIT + lane] = v;
                }
                if (lane == gen_gi) gnc = flush ? 0 : left;
                if (++gen_gi < batch_end) {
                    if (gen_gi == list_g0 + L.lists) build_lists(gen_gi);
                    gen_fetch();
                }
            }
            if (stage.num >= wg_segs) return false;
            seg_mask = bloom_word(stage);
            item0 = seg_first(stage.num);
            const int slot = R == 1 ? 0 : stage.num % R;
            region = (int)blockIdx.x + slot * (int)gridDim.x + y * (int)gridDim.x * R;
            cnt_s = s_cnt + slot * nq_pad;
            batch_g0 = stage.batch * FB;
            batch_end = min(batch_g0 + FB, nf);
            if (stage.batch == 0) {  // the wavefront's next segment
                uint32_t drawn = 0;
                if (lane == 0) drawn = atomicAdd(s_work, 1u);
                next_num = __builtin_amdgcn_readfirstlane((int)drawn);
            }
            flush = next_num >= wg_segs;
            stage = stage.batch + 1 < n_batches ? Stage{stage.num, stage.batch + 1} : Stage{next_num, 0};
            bloom_request(stage);
            const int c = __popcll(seg_mask);
            int incl = c;
            // (the words of a filter sit in neighbouring lanes of one 16-lane row: register moves, no shuffles)
            if (SW > 1) { const int v = (int)row_shr<1>((uint32_t)incl); if (pr_w >= 1) incl += v; }
            if (SW > 2) { const int v = (int)row_shr<2>((uint32_t)incl); if (pr_w >= 2) incl += v; }
            if (SW > 4) { const int v = (int)row_shr<4>((uint32_t)incl); if (pr_w >= 4) incl += v; }
            seg_pos = incl - c;
            // (a turn of the loop over a lane's bits costs about as much as one over the words, and the longest
            // lane's bits count)
            seg_full = (int)lane_value(wave_max_u32((uint32_t)c), 63) > (batch_end - batch_g0) * SW;
            build_lists(batch_g0);
            const int last_word = __shfl(incl, (lane * SW + SW - 1) & 63);
            const int low_words = __shfl(incl, (lane * SW + (SW > 4 ? 3 : SW - 1)) & 63);
            // (a filter without blocks in this row of workgroups has nothing to do here)
            const int blocks = __shfl(gnblk, (batch_g0 + lane) & 63);
            gcur = lane < batch_end - batch_g0 && blocks > 0 ? last_word : 0;
            glow = low_words;
            gen_gi = batch_g0;
            gen_fetch();
        }
    };

    // ---- queue of lanes in which an admission is possible: NV values each, and where their rows and items are (first
    // local row of the tile << 12 | unit's place in the ring and the product << 8 | which four of the lane's results << 6 |
    // lane).  The store is issued in assembly so that the compiler keeps counting loads only when it
    // waits for a unit's rows (see scan_mfma_kernel).
    constexpr int kNoUnit = 0x7FFFFFFF;
    int qn = 0, oldest = kNoUnit;  // the oldest unit that the queue refers to
    auto drain = [&]() {
        if (lane < qn) {
            const uint32_t code = q_code[lane];
            const int s32 = (int)(code & 31u), sh = (int)(code >> 5) & 1, g = (int)(code >> 6) & 3;
            const int at0 = (int)((code >> 8) & (uint32_t)(RING * NS - 1)) * 32, lrow = (int)(code >> 12);
            const uint32_t* src = q_val + lane * NV;
            auto store = [&](int row, uint64_t key) {
                const uint32_t at = atomicAdd(&cnt_s[row / TT], 1u);
                if (at < (uint32_t)p.cap) {
                    uint64_t* dst = p.cand + ((int64_t)(s_qrow[row] / TT) * p.groups + region) * p.cap + at;
                    asm volatile("global_store_dwordx2 %0, %1, off" : : "v"(dst), "v"(key) : "memory");
                }
            };
            if constexpr (!WEIGHTED) {
                const int row = lrow + s32, at = at0 + 8 * g + 4 * sh;
                const int4 v4 = *reinterpret_cast<const int4*>(src);
                const uint4 id4 = *reinterpret_cast<const uint4*>(s_ids + at);
                const float4 si4 = *reinterpret_cast<const float4*>(s_scl + at);
                const float sq = s_sq[row];
                const uint64_t tau = s_tau64[row];
                const int v[4] = {v4.x, v4.y, v4.z, v4.w};
                const uint32_t id[4] = {id4.x, id4.y, id4.z, id4.w};
                const float si[4] = {si4.x, si4.y, si4.z, si4.w};
                uint64_t key[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    key[i] = make_key(rescale(v[i], sq, si[i]), id[i]);
                    if (id[i] == ~0u) key[i] = 0;  // (padding)
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (key[i] >= tau && key[i]) store(row, key[i]);
            } else {
                const uint32_t id = s_ids[at0 + s32];
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    const int row = lrow + 8 * g + 4 * sh + j * TT;
                    const uint64_t key = make_key(__uint_as_float(src[j]), id);
                    if (id != ~0u && key >= s_tau64[row / TT]) store(row, key);
                }
            }
        }
        qn = 0;
        oldest = kNoUnit;
    };
    auto push = [&](uint64_t m, uint32_t code, const uint32_t* val) {  // m: lanes to queue, not 0
        const int n = __popcll(m);
        if (qn + n > kTileQueue) drain();
        if ((m >> lane) & 1ULL) {
            const int at = qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if constexpr (NV == 4) *reinterpret_cast<int4*>(q_val + at * NV) = make_int4((int)val[0], (int)val[1], (int)val[2], (int)val[3]);
            else if constexpr (NV == 2) *reinterpret_cast<int2*>(q_val + at * NV) = make_int2((int)val[0], (int)val[1]);
            else q_val[at] = val[0];
            q_code[at] = code | (uint32_t)lane;
        }
        qn = __builtin_amdgcn_readfirstlane(qn + n);  // (a scalar, which the compiler does not see by itself)
    };

    // ---- units
    v4i rows[NS][KK], next[NS][KK];
    float next_si = 0.0f;
    int next_lrow = 0, next_nblk = 0;  // of the unit requested last (0 blocks: none)
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int k = 0; k < KK; ++k) next[s][k] = v4i{0, 0, 0, 0};
    int unit_no = 0;  // units requested
    // plain search: every scale that this wavefront's factors cover is below 2^cur_E (none yet)
    int cur_E = -1000;
    float fix_scale = 0.0f;  // 2^(P - cur_E)
    bool more = true;
    while (more || next_nblk > 0) {
        // the requested unit becomes the current one (its rows are waited for here)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int k = 0; k < KK; ++k) rows[s][k] = next[s][k];
        const float si = next_si;
        const int lrow0 = next_lrow, nblk = next_nblk, ring = (unit_no - 1) & (RING - 1);
        // the next one
        next_nblk = 0;
        more = more && next_unit();
        if (more) {
            uint32_t id[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) id[s] = entry_item(gen_gi, min(gen_b0 + 32 * s + l32, gen_tot - 1), gen_nc, gen_low);
            const uint32_t own = half ? id[NS - 1] : id[0];  // item `lane` of the unit
            next_si = p.iscale[own];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const char* row = reinterpret_cast<const char*>(p.items) + (uint64_t)id[s] * D + half * 16;
#pragma unroll
                for (int k = 0; k < KK; ++k) {
                    const int4 v = *reinterpret_cast<const int4*>(row + 32 * k);
                    next[s][k] = v4i{v.x, v.y, v.z, v.w};
                }
            }
            if (unit_no - RING >= oldest) drain();
            if (NS == 2 || half == 0) s_ids[(unit_no & (RING - 1)) * UNIT + lane] = gen_b0 + lane < gen_tot ? own : ~0u;
            next_lrow = __builtin_amdgcn_readlane(glrow, gen_gi);
            next_nblk = __builtin_amdgcn_readlane(gnblk, gen_gi);
            gen_b0 += UNIT;
        }
        const int this_unit = unit_no - 1;
        if (more) ++unit_no;
        if (nblk == 0) continue;

        // scales: the exact ones for the queue, and the plain search's fixed-point factors
        if (NS == 2 || half == 0) s_scl[ring * UNIT + lane] = si;
        int4 fix[NS][4];
        float si_s[NS];
        bool cull = true;
        if (!WEIGHTED) {
            // the largest of the unit: scales are positive, so their bit patterns order as they do (a negative or
            // non-finite scale comes out on top and switches the bound off for the unit)
            const float smax = __uint_as_float(lane_value(wave_max_u32(__float_as_uint(si)), 63));
            cull = smax > 0x1p-90f && smax < 0x1p90f;
            const int E = (int)(__float_as_uint(smax) >> 23) - 126;  // 2^E > smax
            if (cull && E > cur_E) {  // (a handful of times to a launch)
                // The workgroup's bounds come down to this exponent at least: a bound for a larger one is smaller,
                // and lets more pairs through.
                cur_E = E;
                fix_scale = __uint_as_float((uint32_t)(P - E + 127) << 23);
                const float thr_scale = fix_scale * 0.99999618530273f;  // (1 - 2^-18) * 2^(P-E)
                for (int row = lane; row < mp.rows_local; row += 64)
                    if (s_qrow[row] >= 0)  // (not for padding)
                        atomicMin(&s_thr[row], (int)__builtin_amdgcn_fmed3f(__builtin_floorf(bound_quotient(s_bound[row], s_sq[row]) * thr_scale),
                                                                            -2147483648.0f, 2147483520.0f));
            }
            // (at least 1: the product of a tiny scale may round to zero, its ceiling does not)
            if (NS == 2 || half == 0) s_fix[lane] = cull ? max(__float2int_ru(si * fix_scale), 1) : 0;
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int g = 0; g < 4; ++g) fix[s][g] = *reinterpret_cast<const int4*>(s_fix + 32 * s + 8 * g + 4 * half);
        } else {
#pragma unroll
            for (int s = 0; s < NS; ++s) si_s[s] = s_scl[ring * UNIT + 32 * s + l32];
        }
        const int8_t* qp = s_q + (lrow0 + l32) * DP + half * 16;
        for (int j = 0; j < nblk; j += 2) {
            const int lrow = lrow0 + 16 * j;
            const bool one = j + 1 >= nblk;  // only the first block of the tile is the filter's
            v4i q[KK];
#pragma unroll
            for (int k = 0; k < KK; ++k) {
                const int4 v = *reinterpret_cast<const int4*>(qp + 32 * k);
                q[k] = v4i{v.x, v.y, v.z, v.w};
            }
            qp += 32 * DP;
            int thr = 0;
            if (!WEIGHTED) {
                thr = s_thr[lrow + l32];
                if (!cull) thr = (int)0x80000000;
                if (one && (lane & 16)) thr = 0x7FFFFFFF;
            }
            tile_i16 acc[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[s][i] = 0;
#pragma unroll
            for (int k = 0; k < KK; ++k)
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    acc[s] = WEIGHTED ? __builtin_amdgcn_mfma_i32_32x32x32_i8(q[k], rows[s][k], acc[s], 0, 0, 0)
                                      : __builtin_amdgcn_mfma_i32_32x32x32_i8(rows[s][k], q[k], acc[s], 0, 0, 0);
            uint32_t val[NS][4][NV];
            uint64_t hits[NS][4], any = 0;
            if constexpr (!WEIGHTED) {
                int m[NS][4];
#pragma unroll
                for (int s = 0; s < NS; ++s) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int t0 = __mul24(acc[s][4 * g], fix[s][g].x), t1 = __mul24(acc[s][4 * g + 1], fix[s][g].y);
                        const int t2 = __mul24(acc[s][4 * g + 2], fix[s][g].z), t3 = __mul24(acc[s][4 * g + 3], fix[s][g].w);
                        m[s][g] = max(max(max(t0, t1), t2), t3);
#pragma unroll
                        for (int i = 0; i < NV; ++i) val[s][g][i] = (uint32_t)acc[s][4 * g + i];
                    }
                    any |= ballot(max(max(max(m[s][0], m[s][1]), m[s][2]), m[s][3]) >= thr);
                }
                if (any == 0) continue;
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int g = 0; g < 4; ++g) hits[s][g] = ballot(m[s][g] >= thr);
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 sq4 = *reinterpret_cast<const float4*>(s_sq + lrow + 8 * g + 4 * half);
                    const float4 tf4 = *reinterpret_cast<const float4*>(s_bound + lrow + 8 * g + 4 * half);
                    const float sqv[4] = {sq4.x, sq4.y, sq4.z, sq4.w};
                    const float tfv[4] = {tf4.x, tf4.y, tf4.z, tf4.w};
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        float sc[4];
                        bool hit = false;
#pragma unroll
                        for (int r = 0; r < 4; ++r) sc[r] = rescale(acc[s][4 * g + r], sqv[r], si_s[s]);
#pragma unroll
                        for (int q0 = 0; q0 < 4; q0 += TT) {
                            float agg = 0.0f;
#pragma unroll
                            for (int tt = 0; tt < TT; ++tt) agg = __fmaf_rn(p.w[tt], sc[q0 + tt], agg);
                            hit = hit || agg >= tfv[q0];
                            val[s][g][q0 / TT] = __float_as_uint(agg);
                        }
                        hits[s][g] = g >= 2 && one ? 0ULL : ballot(hit);
                        any |= hits[s][g];
                    }
                }
                if (any == 0) continue;
            }
            const uint32_t code = (uint32_t)((lrow << 12) | (ring * NS << 8));
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (hits[s][g]) push(hits[s][g], code + (uint32_t)(s << 8) + (uint32_t)(g << 6), val[s][g]);
            oldest = min(oldest, this_unit);
        }
    }
    if (qn > 0) drain();
    __syncthreads();
    // region fill counts: real ones for the queries this workgroup row owns, zero for the others
    for (int i = tid * TT; i < mp.n_blocks * 16; i += kThreads * TT) {
        const int grow = mp.blk_row[i];
        if (grow < 0) continue;
        const int q = grow / TT;
        const int b = i >> 4;
        for (int j = 0; j < R; ++j) {
            uint32_t c = 0;
            if (b % S == y) c = s_cnt[j * nq_pad + ((b / S) * 16 + (i & 15)) / TT];
            const int region_j = (int)blockIdx.x + j * (int)gridDim.x + y * (int)gridDim.x * R;
            p.cnt[(int64_t)q * p.groups + region_j] = c < (uint32_t)p.cap ? c : (uint32_t)p.cap;
            if (c > (uint32_t)p.cap) p.ovf[q] = 1u;
        }
    }
}

// Whether a launch with these parameters can be served by this form, its LDS, and from which count of the first
// level's passing pairs on it is.
inline bool scan_tile_applies(const ScanParams& sp, const MfmaParams& mp, int gx, TileLds* lds)
{
    lds->total = 0;
    if (!mp.density_acc || sp.n_groups > kTileGroups) return false;
    const double items = (double)(sp.item_end - sp.item_begin) / ((double)gx * kTileWaves);  // of a wavefront
    if (items < tile_min_span(sp.d, sp.weighted != 0, sp.n_tasks, mp.n_blocks, sp.n_groups, mp.q_split)) return false;
    const double pairs = (double)mp.density_pairs * tile_min_items(sp.d) / (items > 1.0 ? items : 1.0);
    for (int lists = sp.n_groups < kMfmaFilterBatch ? sp.n_groups : kMfmaFilterBatch;; lists = (lists + 1) / 2) {
        *lds = tile_lds(mp.rows_local, sp.d, sp.n_tasks, sp.weighted != 0, sp.n_groups, mp.region_slots, mp.seg_stride, lists);
        lds->min_pairs = pairs < 9e18 ? (unsigned long long)pairs : 9000000000000000000ULL;
        if (lds->total <= 160 * 1024) return true;
        if (lists == 1) {
            lds->total = 0;
            return false;
        }
    }
}

}  // namespace st
