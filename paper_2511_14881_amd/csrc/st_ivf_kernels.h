// Cluster probing (Sec. 4.2; Sec. 4.3, Alg. 1).
//
// Items are stored cluster by cluster; cluster c is the item range [off[c], off[c+1]).
// Phase 1 (ivf_probe_kernel): one workgroup per query scores every centroid like an item
// (int8 dot, two fp32 multiplies), and an exact top-n_p by (score descending, cluster id
// ascending) gives the probed clusters.
// Phases 2-4, up to kQueryProbes probes (ivf_query_kernel): the workgroups of a query filter and
// score the items of its probed ranges alone, ivf_merge_kernel selects and orders the top K (or a lone
// workgroup itself, where it has few words).
// Phase 2, any number of probes (ivf_mask_kernel): 32 threads per (query, probed cluster) run the
// query's filter program only over the words of that cluster's range and OR the result into the
// query's row of a bit-sliced mask index (zeroed beforehand), laid out like the Bloom index; phases
// 3-4 are then the ordinary fused scan and selection reading that mask index: items outside the
// probed ranges have mask bit 0 and are never loaded.
#pragma once
#include "st_bloom_kernels.h"
#include "st_search_kernels.h"

namespace st {

constexpr int kProbeThreads = 256;

struct IvfParams {
    const int8_t* queries;        // [batch][d]
    const float* qscale;          // [batch]
    const int8_t* centroids;      // [n_clusters][d]
    const float* cscale;          // [n_clusters]
    const int64_t* cluster_off;   // [n_clusters + 1]
    int32_t d, n_clusters, n_probe, k_pad, batch;
    int64_t n_items;
    uint64_t* keys;               // [batch][n_clusters]  scratch: centroid keys
    int32_t* probes;              // [batch][n_probe]     probed clusters in rank order, -1 = none
    int32_t* user_probes;         // the same for the caller, or null
    StageCopy tables;             // the filter programs' tables, brought over by the first workgroup of phase 1
};

// Dynamic LDS: sorted keys [k_pad], histogram [256], misc [8], reduction [2 * waves].
inline size_t probe_lds_bytes(int k_pad) { return (size_t)k_pad * 8 + 256 * 4 + 8 * 4 + 2 * (kProbeThreads / 64) * 8 + 16; }

__global__ __launch_bounds__(kProbeThreads) void ivf_probe_kernel(IvfParams p)
{
    extern __shared__ uint64_t probe_lds[];
    uint64_t* s_sorted = probe_lds;                                       // [k_pad]
    uint64_t* s_red = s_sorted + p.k_pad;                                 // [2 * waves]
    uint32_t* s_hist = reinterpret_cast<uint32_t*>(s_red + 2 * (kProbeThreads / 64));  // [256]
    uint32_t* s_misc = s_hist + 256;                                      // [8]
    const int tid = threadIdx.x, b = blockIdx.x;
    if (b == 0 && p.tables.src) stage_copy(p.tables);
    const float sq = p.qscale[b];
    uint64_t* keys = p.keys + (int64_t)b * p.n_clusters;
    int64_t qoff[kRowBlock];
#pragma unroll
    for (int r = 0; r < kRowBlock; ++r) qoff[r] = (int64_t)b * p.d;
    for (int c = tid; c < p.n_clusters; c += kProbeThreads) {
        // (query chunks through the scalar cache, centroid chunks four loads at a time)
        int acc[kRowBlock] = {0, 0, 0, 0, 0, 0, 0, 0};
        dot_block<1>(reinterpret_cast<const int4*>(p.centroids + (int64_t)c * p.d), p.queries, qoff, p.d >> 4, acc);
        const float s = rescale(acc[0], sq, p.cscale[c]);
        keys[c] = make_key(s, (uint32_t)c);
    }
    __threadfence_block();
    __syncthreads();
    const int want = p.n_probe < p.n_clusters ? p.n_probe : p.n_clusters;
    const int n_out = wg_topk(keys, p.n_clusters, want, s_sorted, p.k_pad, s_hist, s_misc, s_red);
    __syncthreads();
    for (int j = tid; j < p.n_probe; j += kProbeThreads) {
        const int32_t c = j < n_out ? (int32_t)key_item(s_sorted[j]) : -1;
        p.probes[(int64_t)b * p.n_probe + j] = c;
        if (p.user_probes) p.user_probes[(int64_t)b * p.n_probe + j] = c;
    }
}

// Phase 1 for many centroids, in two kernels.  Part kernel, grid (batch, parts): a workgroup
// scores its slice of the centroids (at most kTopkRegs * kProbeThreads of them) into LDS, keeps the
// best min(n_probe, slice) keys with the register-resident select and leaves them, unordered, at
// the head of its slice of the key scratch.  Merge kernel, one workgroup per query: the parts'
// survivors (at most kTopkRegs * kProbeMergeThreads in all: the host chooses the number of parts
// accordingly) are selected and sorted in LDS and the probed ids written.
constexpr int kProbeParts = 16;
constexpr int kProbeMergeThreads = 512;

__global__ __launch_bounds__(kProbeThreads) void ivf_probe_part_kernel(IvfParams p, int chunk, uint32_t* part_cnt)
{
    __shared__ uint64_t s_keys[kTopkRegs * kProbeThreads];
    __shared__ uint64_t s_sorted[kLdsSortMax];
    __shared__ uint32_t s_hist[3 * 256], s_misc[8];
    __shared__ uint64_t s_red[32];
    const int tid = threadIdx.x, b = blockIdx.x, part = blockIdx.y;
    if (b == 0 && part == 0 && p.tables.src) stage_copy(p.tables);
    const int c0 = part * chunk;
    int n = p.n_clusters - c0;
    n = n < 0 ? 0 : (n > chunk ? chunk : n);
    const float sq = p.qscale[b];
    int64_t qoff[kRowBlock];
#pragma unroll
    for (int r = 0; r < kRowBlock; ++r) qoff[r] = (int64_t)b * p.d;
    for (int i = tid; i < n; i += kProbeThreads) {
        const int c = c0 + i;
        int acc[kRowBlock] = {0, 0, 0, 0, 0, 0, 0, 0};
        dot_block<1>(reinterpret_cast<const int4*>(p.centroids + (int64_t)c * p.d), p.queries, qoff, p.d >> 4, acc);
        s_keys[i] = make_key(rescale(acc[0], sq, p.cscale[c]), (uint32_t)c);
    }
    __syncthreads();
    const int want = p.n_probe < n ? p.n_probe : n;
    int kept = 0;
    if (n > 0) {
        uint64_t kth;
        kept = lds_topk(s_keys, n, want, s_sorted, p.k_pad, s_hist, s_misc, s_red, false, kth);
        __syncthreads();
    }
    uint64_t* dst = p.keys + (int64_t)b * p.n_clusters + c0;  // kept <= n: inside this part's slice
    for (int i = tid; i < kept; i += kProbeThreads) dst[i] = s_sorted[i];
    if (tid == 0) part_cnt[b * kProbeParts + part] = (uint32_t)kept;
}

__global__ __launch_bounds__(kProbeMergeThreads) void ivf_probe_merge_kernel(IvfParams p, int chunk, int parts,
                                                                           const uint32_t* part_cnt)
{
    __shared__ uint64_t s_keys[kTopkRegs * kProbeMergeThreads];
    __shared__ uint64_t s_sorted[kLdsSortMax];
    __shared__ uint32_t s_hist[3 * 256], s_misc[8];
    __shared__ uint64_t s_red[32];
    const int tid = threadIdx.x, b = blockIdx.x;
    uint32_t at = 0;
    for (int pp = 0; pp < parts; ++pp) {
        uint32_t c = part_cnt[b * kProbeParts + pp];
        c = c < (uint32_t)p.n_probe ? c : (uint32_t)p.n_probe;  // (a part keeps at most n_probe, whatever the memory says)
        const uint64_t* src = p.keys + (int64_t)b * p.n_clusters + (int64_t)pp * chunk;
        if (at + c > (uint32_t)(kTopkRegs * kProbeMergeThreads)) c = (uint32_t)(kTopkRegs * kProbeMergeThreads) - at;
        for (uint32_t i = tid; i < c; i += kProbeMergeThreads) s_keys[at + i] = src[i];
        at += c;
    }
    __syncthreads();
    const int want = p.n_probe < p.n_clusters ? p.n_probe : p.n_clusters;
    uint64_t kth;
    const int n_out = lds_topk(s_keys, (int)at, want, s_sorted, p.k_pad, s_hist, s_misc, s_red, true, kth);
    __syncthreads();
    for (int j = tid; j < p.n_probe; j += kProbeMergeThreads) {
        const int32_t c = j < n_out ? (int32_t)key_item(s_sorted[j]) : -1;
        p.probes[(int64_t)b * p.n_probe + j] = c;
        if (p.user_probes) p.user_probes[(int64_t)b * p.n_probe + j] = c;
    }
}

// grid (ceil(n_probe / kMaskProbes), batch): a workgroup takes kMaskProbes probed clusters of one
// query, 32 threads per cluster (a cluster of a thousand items is 16 words).  prog_off / code /
// leaf_rows as for bloom_expr_kernel, one program per query.  mask_rows: bit-sliced index with
// `batch` rows; row b belongs to query b.
constexpr int kMaskProbes = 8;
__global__ __launch_bounds__(256) void ivf_mask_kernel(const uint64_t* __restrict__ bloom, int32_t m_bits,
                                                       int32_t k_hashes, IvfParams p,
                                                       const int32_t* __restrict__ prog_off,
                                                       const int32_t* __restrict__ code,
                                                       const int32_t* __restrict__ leaf_rows,
                                                       uint64_t* __restrict__ mask_rows)
{
    __shared__ uint64_t s_stack[kExprDepth][256];
    __shared__ int32_t s_code[kExprOps];
    __shared__ int32_t s_rows[kExprOps * kExprHashes];
    const int tid = threadIdx.x, b = blockIdx.y;
    const int sub = tid >> 5, wl = tid & 31;
    const int j = (int)blockIdx.x * kMaskProbes + sub;
    const int32_t c = j < p.n_probe ? p.probes[(int64_t)b * p.n_probe + j] : -1;
    // the range, kept inside the corpus whatever the offsets say (empty when there is no cluster)
    int64_t lo = 0, hi = 0;
    if (c >= 0) {
        lo = p.cluster_off[c];
        hi = p.cluster_off[c + 1];
        lo = lo < 0 ? 0 : (lo > p.n_items ? p.n_items : lo);
        hi = hi < lo ? lo : (hi > p.n_items ? p.n_items : hi);
    }
    const int i0 = prog_off[b], n_ops = prog_off[b + 1] - i0;
    for (int i = tid; i < n_ops; i += 256) s_code[i] = code[i0 + i];
    for (int i = tid; i < n_ops * k_hashes; i += 256) s_rows[i] = leaf_rows[(int64_t)i0 * k_hashes + i];
    __syncthreads();  // the only barrier: threads without work may leave below
    if (lo >= hi) return;
    const int64_t w_first = lo >> 6, w_last = (hi - 1) >> 6;
    for (int64_t gw = w_first + wl; gw <= w_last; gw += 32) {
        // bits of this word that belong to [lo, hi)
        const int64_t first = gw * 64;
        uint64_t in = ~0ULL;
        if (first < lo) in &= ~0ULL << (lo - first);
        if (first + 64 > hi) in &= ~0ULL >> (first + 64 - hi);
        const uint64_t* base = bloom + ((gw >> 4) * (int64_t)m_bits) * kTileWords + (gw & 15);
        const uint64_t res = expr_eval_word(s_code, s_rows, n_ops, k_hashes, base, s_stack, tid) & in;
        // neighbouring clusters of one query share their boundary word: OR, not store
        if (res) atomicOr((unsigned long long*)&mask_rows[((gw >> 4) * (int64_t)p.batch + b) * kTileWords + (gw & 15)],
                          (unsigned long long)res);
    }
}

// ------------------------------------------------------------------------------------------
// Phases 2-4 for up to kQueryProbes probes: the workgroups of a query (its parts) walk the words of
// its probed clusters (all of them laid end to end, one word per thread and round, the parts taking
// rounds in turn), run the filter program on each word, score the items that pass themselves (one
// v_dot4 row product per set bit) and append their keys to their share of the query's buffer,
// which is pruned to the best K whenever it cannot take another round.  A merge kernel selects and orders what
// the parts kept.  The work is proportional to the probed items, nothing is written for the rest of
// the corpus, and no candidate can be lost (no regions, no thresholds from elsewhere).
//
// Bound by chains of memory round trips (program leaves, then item rows), so it wants many short
// parts with all wavefronts scoring: 20 M x 128, 16 queries, K = 2048, 32 of 4096 clusters probed take
// 65 us a call with 16 parts a query, against 162 us with 4 (what a merge in LDS had room for) and a
// list of passing items per wavefront.
constexpr int kQueryThreads = 512;
constexpr int kQueryProbes = 512;   // one probe per thread when the ranges are laid out
// A lone workgroup with no more words to walk than this (by the average cluster) orders its keys itself: as a rule fewer than
// 4096, which its own LDS selection takes.  (256 queries, 20,000 items, K = 500, 64 of 1024 clusters, 64 words: 43 us a call,
// 46 to 48 with the merge; 1024 queries, 100,000 items, 128 words: 150 against 135.)
constexpr int kQueryFewWords = 64;
constexpr int kQueryParts = 16;     // workgroups per query, at most (powers of two)

struct IvfQueryParams {
    IvfParams ivf;
    const uint64_t* bloom;
    int32_t m_bits, k_hashes;
    const int8_t* items;
    const float* iscale;
    const int32_t *prog_off, *code, *leaf_rows;
    uint64_t* gath;            // [batch][gath_cap] key buffer
    int64_t gath_cap;
    int64_t part_cap;          // keys of one part's share of the buffer
    int64_t part_keys;         // ... of which keys are gathered in; the rest (several parts, k_pad above the LDS sort size) is the prune's scratch
    int32_t finish;            // 1: a lone part writes the result rows itself (k_pad within the LDS sort size), no merge follows
    int32_t part_keep;         // a part hands on all its keys if they are no more than this (>= K), else its best K
    uint64_t* srt;             // [batch][k_pad] when k_pad > kLdsSortMax, else null (merge's general way, prune of a lone part)
    int32_t K, k_pad;
    int64_t* out_ids;
    float* out_scores;
    int32_t* out_count;
    uint32_t* ovf;             // [batch] "took the slow exact path" flags of the workspace: reset (this path has none)
    uint32_t* part_cnt;        // [batch][kQueryParts] keys each part kept
};

__global__ __launch_bounds__(kQueryThreads) void ivf_query_kernel(IvfQueryParams p)
{
    __shared__ uint64_t s_stack[kExprDepth][kQueryThreads];
    __shared__ int32_t s_code[kExprOps];
    __shared__ int32_t s_rows[kExprOps * kExprHashes];
    __shared__ uint64_t s_sorted[kLdsSortMax];
    __shared__ int64_t s_lo[kQueryProbes], s_hi[kQueryProbes];
    __shared__ uint32_t s_first[kQueryProbes + 1];  // first word (in the laid-out order) of each probe
    __shared__ uint32_t s_hist[3 * 256], s_misc[8], s_wsum[kQueryThreads / 64];
    __shared__ uint64_t s_red[32];
    __shared__ int64_t s_word[kQueryThreads];  // first item of the word each thread evaluated this round
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, b = blockIdx.x;
    const IvfParams& v = p.ivf;
    static_assert(sizeof(s_stack) >= (size_t)kTopkRegs * kQueryThreads * 8, "the stack doubles as a key buffer");
    static_assert(sizeof(s_stack) >= (size_t)kQueryThreads * 64 * 2, "... and as the list of a round's passing items");
    static_assert(kQueryThreads * 64 <= 65536, "an entry of that list has 16 bits");

    // the program, and the item ranges of the probed clusters (clipped to the corpus)
    const int i0 = p.prog_off[b], n_ops = p.prog_off[b + 1] - i0;
    for (int i = tid; i < n_ops; i += kQueryThreads) s_code[i] = p.code[i0 + i];
    for (int i = tid; i < n_ops * p.k_hashes; i += kQueryThreads) s_rows[i] = p.leaf_rows[(int64_t)i0 * p.k_hashes + i];
    uint32_t words = 0;
    if (tid < kQueryProbes) {
        int64_t lo = 0, hi = 0;
        const int32_t c = tid < v.n_probe ? v.probes[(int64_t)b * v.n_probe + tid] : -1;
        if (c >= 0) {
            lo = v.cluster_off[c];
            hi = v.cluster_off[c + 1];
            lo = lo < 0 ? 0 : (lo > v.n_items ? v.n_items : lo);
            hi = hi < lo ? lo : (hi > v.n_items ? v.n_items : hi);
        }
        s_lo[tid] = lo;
        s_hi[tid] = hi;
        words = hi > lo ? (uint32_t)(((hi - 1) >> 6) - (lo >> 6) + 1) : 0u;
    }
    // exclusive prefix sum of the word counts over the workgroup
    uint32_t incl = words;
    incl = wave_scan_add(incl);
    if (lane == 63) s_wsum[wv] = incl;
    if (tid == 0) {
        s_misc[4] = 0;  // keys in the buffer
        p.ovf[b] = 0u;
    }
    __syncthreads();
    uint32_t base = 0, total = 0;
    for (int w = 0; w < kQueryThreads / 64; ++w) {
        const uint32_t t = s_wsum[w];
        if (w < wv) base += t;
        total += t;
    }
    if (tid < kQueryProbes) s_first[tid] = base + incl - words;
    if (tid == 0) s_first[kQueryProbes] = total;
    __syncthreads();

    const int part = blockIdx.y, parts = gridDim.y;
    const int64_t cap = p.part_keys;
    uint64_t* buf = p.gath + (int64_t)b * p.gath_cap + part * p.part_cap;
    uint64_t* sorted = p.k_pad <= kLdsSortMax ? s_sorted : parts > 1 ? buf + cap : p.srt + (int64_t)b * p.k_pad;
    uint32_t* s_n = &s_misc[4];
    int64_t qoff[kRowBlock];
#pragma unroll
    for (int r = 0; r < kRowBlock; ++r) qoff[r] = (int64_t)b * v.d;
    const float sq = v.qscale[b];
    uint64_t tau = 0;
    // words per round: as many as the buffer is sure to hold beside the K keys kept
    int64_t wpr = (cap - p.K) / 64;
    wpr = wpr > kQueryThreads ? kQueryThreads : (wpr < 1 ? 1 : wpr);
    {   // no longer than an even share of the query's words (whole wavefronts), so that every part has work
        const int64_t share = (((int64_t)total + parts - 1) / parts + 63) & ~63LL;
        if (share < wpr) wpr = share < 64 ? 64 : share;
    }
    for (uint32_t w0 = (uint32_t)(part * wpr); w0 < total; w0 += (uint32_t)(parts * wpr)) {
        if ((int64_t)*s_n + wpr * 64 > cap) {  // uniform: *s_n is stable between barriers
            const int n_out = wg_topk(buf, (int64_t)*s_n, p.K, sorted, p.k_pad, s_hist, s_misc, s_red, false, &tau);
            for (int i = tid; i < n_out; i += kQueryThreads) buf[i] = sorted[i];
            __syncthreads();
            if (tid == 0) *s_n = (uint32_t)n_out;
            __syncthreads();
        }
        const uint32_t wi = w0 + tid;
        uint64_t m = 0;
        int64_t first = 0;
        if (tid < wpr && wi < total) {
            // the probe this word belongs to: last j with s_first[j] <= wi
            int a = 0, z = kQueryProbes;
            while (z - a > 1) {
                const int mid = (a + z) >> 1;
                if (s_first[mid] <= wi) a = mid; else z = mid;
            }
            const int64_t lo = s_lo[a], hi = s_hi[a];
            const int64_t gw = (lo >> 6) + (wi - s_first[a]);
            first = gw * 64;
            uint64_t in = ~0ULL;
            if (first < lo) in &= ~0ULL << (lo - first);
            if (first + 64 > hi) in &= ~0ULL >> (first + 64 - hi);
            const uint64_t* wbase = p.bloom + ((gw >> 4) * (int64_t)p.m_bits) * kTileWords + (gw & 15);
            m = expr_eval_word(s_code, s_rows, n_ops, p.k_hashes, wbase, s_stack, tid) & in;
        }
        // The round's passing items, dealt out evenly over the workgroup's threads: every thread lists
        // its set bits as (thread, bit) pairs in the stack's memory, which is free once all words are
        // evaluated.  (A part with few words has them in its first wavefronts alone; a list per
        // wavefront left the others without items to score.)
        s_word[tid] = first;
        const uint32_t cnt = (uint32_t)__popcll(m);
        const uint32_t inc = wave_scan_add(cnt);
        if (lane == 63) s_wsum[wv] = inc;
        __syncthreads();
        uint32_t at = inc - cnt, n_pairs = 0;
        for (int w = 0; w < kQueryThreads / 64; ++w) {
            const uint32_t t = s_wsum[w];
            if (w < wv) at += t;
            n_pairs += t;
        }
        uint16_t* pairs = reinterpret_cast<uint16_t*>(&s_stack[0][0]);
        while (m) {
            const int bit = __ffsll((long long)m) - 1;
            m &= m - 1;
            pairs[at++] = (uint16_t)((tid << 6) | bit);
        }
        const uint32_t n_before = *s_n;
        __syncthreads();
        for (uint32_t k = tid; k < n_pairs; k += kQueryThreads) {
            const uint32_t pr = pairs[k];
            const int64_t item = s_word[pr >> 6] + (pr & 63);
            // (query chunks through the scalar cache, item chunks four loads at a time)
            int acc[kRowBlock] = {0, 0, 0, 0, 0, 0, 0, 0};
            dot_block<1>(reinterpret_cast<const int4*>(p.items + item * v.d), v.queries, qoff, v.d >> 4, acc);
            const float sc = rescale(acc[0], sq, p.iscale[item]);
            const uint64_t key = make_key(sc, (uint32_t)item);
            // (without a threshold every key stays: its place is known)
            if (tau == 0) buf[n_before + k] = key;
            else if (key >= tau) buf[atomicAdd(s_n, 1u)] = key;
        }
        if (tau == 0 && tid == 0) *s_n = n_before + n_pairs;
        __syncthreads();
    }
    uint32_t n_keys = *s_n;
    if (p.finish) {
        uint64_t kth;
        int n_out;
        if (n_keys <= (uint32_t)(kTopkRegs * kQueryThreads)) {
            uint64_t* s_keys = &s_stack[0][0];
            for (uint32_t i = tid; i < n_keys; i += kQueryThreads) s_keys[i] = buf[i];
            __syncthreads();
            n_out = lds_topk(s_keys, (int)n_keys, p.K, s_sorted, p.k_pad, s_hist, s_misc, s_red, true, kth);
        } else {
            n_out = wg_topk(buf, (int64_t)n_keys, p.K, s_sorted, p.k_pad, s_hist, s_misc, s_red);
        }
        write_result(s_sorted, n_out, p.K, p.out_ids + (int64_t)b * p.K, p.out_scores + (int64_t)b * p.K, p.out_count + b);
        return;
    }
    if (n_keys > (uint32_t)p.part_keep) {
        // keep this part's best K (unordered) at the head of its share
        uint64_t kth;
        int kept;
        if (p.k_pad <= kLdsSortMax && n_keys <= (uint32_t)(kTopkRegs * kQueryThreads)) {  // register-resident select on a copy in LDS
            uint64_t* s_keys = &s_stack[0][0];
            for (uint32_t i = tid; i < n_keys; i += kQueryThreads) s_keys[i] = buf[i];
            __syncthreads();
            kept = lds_topk(s_keys, (int)n_keys, p.K, s_sorted, p.k_pad, s_hist, s_misc, s_red, false, kth);
            __syncthreads();
        } else {
            kept = wg_topk(buf, (int64_t)n_keys, p.K, sorted, p.k_pad, s_hist, s_misc, s_red, false, &kth);
        }
        for (int i = tid; i < kept; i += kQueryThreads) buf[i] = sorted[i];
        n_keys = (uint32_t)kept;
    }
    // the merge is a kernel of its own (ivf_merge_kernel): a device-wide fence here, for a
    // last-finisher merge in this kernel, measured 30 us per workgroup
    if (tid == 0) p.part_cnt[b * kQueryParts + part] = n_keys;
}

// Keys the parts of a query hand on together, as a target (each at least K): the merge reads them three times.
constexpr int kMergeKeys = 16384;

// Selection and order of what the parts of a query handed on: one workgroup per query, by buckets of the
// score over the keys where they lie, a share of the wavefronts to each part; a thread's first 16 keys stay in registers
// for the passes.  Bound by the latency of its passes (16 x 1000 keys: 24.6 us, 27.1 with the keys read in every pass).
constexpr int kMergeThreads = 1024;
constexpr uint32_t kMergeRegs = 16;  // keys of a thread held in registers
constexpr int kMergeRoom = 8192;
static_assert(kOrderBins * 4 >= kLdsSortMax * 8, "the general way's result borrows the counters");
__global__ __launch_bounds__(kMergeThreads) void ivf_merge_kernel(IvfQueryParams p, int parts)
{
    __shared__ uint64_t s_keys[kMergeRoom];
    __shared__ uint64_t s_bins[kOrderBins / 2];
    __shared__ uint32_t s_hist[256], s_misc[8], s_wsum[kMergeThreads / 64];
    __shared__ uint64_t s_red[32];
    constexpr int NW = kMergeThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, b = blockIdx.x;
    uint64_t* keys = p.gath + (int64_t)b * p.gath_cap;
    auto held = [&](int pp) {  // (a part hands on no more than its share holds, whatever the memory says)
        const uint32_t c = p.part_cnt[b * kQueryParts + pp];
        return c < (uint32_t)p.part_keys ? c : (uint32_t)p.part_keys;
    };
    static_assert(kQueryParts <= NW, "every part has a wavefront of its own");
    uint32_t total = 0;
    for (int pp = 0; pp < parts; ++pp) total += held(pp);
    const int per = NW / parts, mine = wv / per;  // (parts is a power of two)
    const uint32_t n_mine = held(mine);
    const uint64_t* src = keys + mine * p.part_cap;
    const uint32_t first = (uint32_t)((wv % per) * 64 + lane), step = (uint32_t)per * 64;
    auto each_from = [&](uint32_t i0, auto&& f) {
        for (; ballot(i0 < n_mine) != 0; i0 += 8 * step) {
            uint64_t v[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u)
                if (i0 + u * step < n_mine) v[u] = src[i0 + u * step];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u)
                if (i0 + u * step < n_mine) f(v[u]);
        }
    };
    const uint32_t want = total < (uint32_t)p.K ? total : (uint32_t)p.K;
    int64_t* ids = p.out_ids + (int64_t)b * p.K;
    float* scores = p.out_scores + (int64_t)b * p.K;
    auto order = [&](auto&& each) {
        return bucket_order<kMergeThreads>(each, want, (uint32_t)kMergeRoom, s_keys, reinterpret_cast<uint32_t*>(s_bins), s_misc,
                                           s_red, s_wsum, [&](uint32_t rank, uint64_t key) {
                                               if (rank < want) {
                                                   ids[rank] = (int64_t)key_item(key);
                                                   scores[rank] = key_score(key);
                                               }
                                           });
    };
    // With more keys than one round of loads takes, a thread's first 16 stay in registers for all passes (0: none; no key
    // is 0).  With fewer a pass is one round trip as it is and the unrolled code costs more than it saves (2 queries x 2
    // parts of 21 keys: 7.5 us with registers, 6.6 without).
    bool ordered = want == 0;
    if (total > 8 * kMergeThreads) {
        uint64_t kr[kMergeRegs];
        const uint32_t held_regs = (uint32_t)__builtin_amdgcn_readfirstlane((int)min((n_mine + step - 1) / step, (uint32_t)kMergeRegs));
#pragma unroll
        for (uint32_t u = 0; u < kMergeRegs; ++u) kr[u] = first + u * step < n_mine ? src[first + u * step] : 0ULL;
        ordered = order([&](auto&& f) {
#pragma unroll
            for (uint32_t u = 0; u < kMergeRegs; ++u)
                if (u < held_regs && kr[u]) f(kr[u]);
            each_from(first + kMergeRegs * step, f);
        });
    } else if (!ordered) {
        ordered = order([&](auto&& f) { each_from(first, f); });
    }
    if (ordered) {
        for (int i = (int)want + tid; i < p.K; i += kMergeThreads) {
            ids[i] = -1;
            scores[i] = -__builtin_inff();
        }
        if (tid == 0) p.out_count[b] = (int32_t)want;
        return;
    }
    // many equal scores: the general way over the keys moved together (a step's keys are read before any of
    // them is written; they only move down)
    int64_t at = 0;
    for (int pp = 0; pp < parts; ++pp) {
        const uint32_t c = held(pp);
        for (uint32_t i0 = 0; i0 < c; i0 += kMergeThreads) {
            __syncthreads();
            const uint64_t k = i0 + tid < c ? keys[pp * p.part_cap + i0 + tid] : 0ULL;
            __syncthreads();
            if (i0 + tid < c) keys[at + i0 + tid] = k;
        }
        at += c;
    }
    __threadfence_block();
    __syncthreads();
    uint64_t* sorted = p.srt ? p.srt + (int64_t)b * p.k_pad : s_bins;
    const int n_out = wg_topk(keys, at, p.K, sorted, p.k_pad, s_hist, s_misc, s_red);
    write_result(sorted, n_out, p.K, ids, scores, p.out_count + b);
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint64_t* __restrict__ dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] = 0ULL;
}

}  // namespace st
