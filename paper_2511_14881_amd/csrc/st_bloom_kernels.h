// Bloom index kernels: build (Sec. 4.1), item-major export and the stand-alone mask export.
//
// Index layout in HBM ("rotated" / bit-sliced, Sec. 4.1, blocked for 128-byte lines):
//   word(tile, row, w) = bloom[(tile * m_bits + row) * 16 + w],  tile = item / 1024,
//   w = (item % 1024) / 64, bit (item % 64) of that word = bit `row` of the item's signature.
// One row segment of a tile is 16 words = 128 bytes; a filter that sets r signature bits
// touches r such lines per tile.
#pragma once
#include <type_traits>

#include "st_device.h"

namespace st {

// Position of a hash modulo m <= 65536, for the build kernel's inner loop (the same value as
// bloom_bit).  A power of two needs the low bits of the hash alone, so the second product of
// splitmix64 is formed only as far as they reach; other sizes reduce the two halves of the hash with a
// multiply-high by floor(2^32 / m), which is at most one short of the quotient.
struct BuildMod {
    uint32_t m, magic, two32;  // magic = floor(2^32 / m), two32 = 2^32 mod m
};
inline BuildMod build_mod(int32_t m_bits)
{
    BuildMod b;
    b.m = (uint32_t)m_bits;
    b.magic = m_bits > 1 ? (uint32_t)((1ULL << 32) / (uint64_t)m_bits) : 0u;
    b.two32 = (uint32_t)((1ULL << 32) % (uint64_t)m_bits);
    return b;
}
template <bool POW2>
__device__ inline uint32_t build_pos(uint64_t x, const BuildMod& b)
{
    uint64_t z = x + 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z ^= z >> 27;
    constexpr uint32_t kLo = 0x133111EBu, kHi = 0x94D049BBu;
    if (POW2) {
        // bits 0 .. 15 of w ^ (w >> 31), w = z * (kHi:kLo): the cross products count from bit 32 on, and
        // their low 15 bits depend on the low bits of the factors only (24-bit multiplies)
        const uint64_t lo = (uint64_t)(uint32_t)z * kLo;
        uint32_t c0 = __umul24((uint32_t)z & 0xFFFFFFu, kHi & 0xFFFFFFu), c1 = __umul24((uint32_t)(z >> 32) & 0xFFFFFFu, kLo & 0xFFFFFFu);
        // (nobody is to see how few of their bits count: the masks would go, and with them the 24-bit form, for full
        // products at a quarter of the rate.  3 M items x 6 ids, 8 hashes: 183 -> 170 us; 3 M x 16, 8: 366 -> 350)
        asm("" : "+v"(c0));
        asm("" : "+v"(c1));
        const uint32_t hi = (uint32_t)(lo >> 32) + c0 + c1;
        return ((uint32_t)lo ^ (((uint32_t)lo >> 31) | (hi << 1))) & (b.m - 1u);
    }
    z *= ((uint64_t)kHi << 32) | kLo;
    z ^= z >> 31;
    auto mod = [&](uint32_t v) {
        const uint32_t r = v - __umulhi(v, b.magic) * b.m;
        return r >= b.m ? r - b.m : r;
    };
    return mod(mod((uint32_t)(z >> 32)) * b.two32 + mod((uint32_t)z));  // < m * m <= 2^32
}

// One workgroup per 1024-item tile, one item per thread.  The tile's block of the index -- m rows of
// 128 bytes -- is assembled in LDS (in slabs of kBuildSlabRows rows where m is larger): every thread
// hashes the ids of its item once per slab (k positions each, Sec. 4.1), sets the item's bit in the rows
// the positions name with LDS atomic ORs, and the finished rows go out as one contiguous, coalesced
// copy.  Hash work is therefore independent of m up to the slab size, and HBM sees the feature
// lists once and the index once.
constexpr int kBuildThreads = kTileItems;
constexpr int kBuildSlabRows = 1024;  // 128 KB of LDS

// Two neighbouring ids (a list may start at any multiple of 8 bytes).
struct __attribute__((packed, aligned(8))) BuildPair {
    uint64_t a, b;
};

// Word w32 (32 items) of LDS row r lies at w32 ^ (r & 31): the 64 lanes of a wavefront hold two words'
// worth of items, and without the swizzle their updates of any rows would meet in two to four banks.
__device__ inline int build_word(int r, int w32) { return r * 32 + (w32 ^ (r & 31)); }

// LANES: lanes to an item's list.  A load is paid by the lines that it touches, 64 where every lane reads a list of its own; with
// four lanes to a list it is 16, but the items come in four passes, and lists of a few ids leave lanes idle.
// K: hashes of an id (0: as many as k_hashes says), written out so that two of them are in flight and no loop is counted.
// ONE: the rows fit one slab, and no position is compared with it.  Bound by the instructions of the hashes (some 20 to each,
// two products among them) beside the LDS updates.  10 M items x 16 ids, 4 hashes, 512 rows: 0.70 ms with a counted loop, a
// test against the slab and four steps to an address; the whole of a pass with the export 915 us, 820 with
// two ids to a load, 718 with four lanes to a list, 690 with 24-bit products (the kernel 0.48 ms).
// PAIRS: two ids to a load, but for short lists, where finding out whether there is a second one costs more than a load.
template <bool POW2, int K, bool ONE, int LANES, bool PAIRS = true>
__global__ __launch_bounds__(kBuildThreads, 8) void bloom_build_kernel(const int64_t* __restrict__ feat_offsets,
                                                                    const uint64_t* __restrict__ feat_ids,
                                                                    int64_t n_items, BuildMod bm,
                                                                    int32_t k_hashes, uint64_t* __restrict__ bloom)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t s_bits[];  // [rows][32]: the 16 words of a row as 32-bit halves
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x;
    const int m_bits = (int)bm.m;
    constexpr int kWide = PAIRS ? 2 : 1, kLoads = LANES == 1 ? 8 / kWide : 2;  // ids to a load, loads in flight per thread
    constexpr int kStep = kLoads * kWide * LANES;
    for (int slab0 = 0; slab0 < m_bits; slab0 += kBuildSlabRows) {
        const int rows = min(kBuildSlabRows, m_bits - slab0);
        for (int i = tid; i < rows * 8; i += kBuildThreads) reinterpret_cast<int4*>(s_bits)[i] = make_int4(0, 0, 0, 0);
        __syncthreads();
        for (int pass = 0; pass < LANES; ++pass) {
            const int it = (tid & ~63) + pass * (64 / LANES) + (tid & 63) / LANES, w32 = it >> 5;  // item of the tile
            const int64_t item = tile * kTileItems + it;
            const uint32_t bit = 1u << (it & 31);
            const int64_t f_begin = item < n_items ? feat_offsets[item] : 0, f_end = item < n_items ? feat_offsets[item + 1] : 0;
            auto mark = [&](uint64_t id, int j) __attribute__((always_inline)) {
                const int r = (int)build_pos<POW2>(id ^ (uint64_t)j, bm) - (ONE ? 0 : slab0);
                if (ONE || (uint32_t)r < (uint32_t)rows) atomicOr(&s_bits[build_word(r, w32)], bit);
            };
            for (int64_t e = f_begin + kWide * (tid & (LANES - 1)); e < f_end; e += kStep) {
                BuildPair f[kLoads];
                const int left = (int)min(f_end - e, (int64_t)kStep);
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    const int at = u * kWide * LANES;
                    f[u] = {0, 0};
                    if (PAIRS && at + 1 < left) f[u] = *reinterpret_cast<const BuildPair*>(feat_ids + e + at);
                    else if (at < left) f[u].a = feat_ids[e + at];
                }
#pragma unroll
                for (int u = 0; u < kLoads; ++u)
#pragma unroll
                    for (int i = 0; i < kWide; ++i)
                        if (u * kWide * LANES + i < left) {
                            const uint64_t id = i ? f[u].b : f[u].a;
                            if constexpr (K > 0) {
#pragma unroll
                                for (int j = 0; j < K; ++j) mark(id, j);
                            } else {
                                for (int j = 0; j < k_hashes; ++j) mark(id, j);
                            }
                        }
            }
        }
        __syncthreads();
        int4* dst = reinterpret_cast<int4*>(bloom + (tile * (int64_t)m_bits + slab0) * kTileWords);
        for (int i = tid; i < rows * 8; i += kBuildThreads) {
            const int r = i >> 3, c = i & 7;  // the four words of a piece lie in one piece, their order depends on the row
            const int4 v = reinterpret_cast<const int4*>(s_bits)[r * 8 + (c ^ ((r >> 2) & 7))];
            int4 o = (r & 1) ? make_int4(v.y, v.x, v.w, v.z) : v;
            if (r & 2) o = make_int4(o.z, o.w, o.x, o.y);
            dst[i] = o;
        }
        __syncthreads();
    }
}

// The kernel for an index: written out for two to five hashes and up to one slab of rows.
// Four lanes to a list from 12 ids to an item on, where the tiles fill the chip and the positions need no division. One lane -> four, a
// build and an export in us:
//   1.1 M items x 21 ids 126 -> 101;  4.5 M x 19 391 -> 368;  1.5 M x 13 122.9 -> 120.4
//   but 2.2 M x 7 88 -> 95;  6.0 M x 3 196 -> 367;  44,000 x 18 75 -> 85;  100 rows, 2.9 M x 18, 5 hashes 402 -> 460
// An id to a load where the hashes are counted and an item has fewer than four ids. Two ids -> one:
//   5 M items x 3 ids, 1 hash 123.5 -> 115.2, 7 hashes 154.6 -> 150.8;  x 2, 6 hashes 132.7 -> 128.2;  but 4 M x 4, 16 hashes 240 -> 242
constexpr int64_t kBuildLongList = 12, kBuildLongTiles = 512, kBuildShortList = 4;
template <bool POW2, int LANES>
inline auto build_kernel(int k_hashes) -> decltype(&bloom_build_kernel<POW2, 0, false, 1>)
{
    switch (k_hashes) {
    case 2: return &bloom_build_kernel<POW2, 2, true, LANES>;
    case 3: return &bloom_build_kernel<POW2, 3, true, LANES>;
    case 4: return &bloom_build_kernel<POW2, 4, true, LANES>;
    case 5: return &bloom_build_kernel<POW2, 5, true, LANES>;
    default: return &bloom_build_kernel<POW2, 0, true, LANES>;
    }
}
inline auto build_kernel(int m_bits, int k_hashes, int64_t n_ids, int64_t n_items, int64_t n_tiles) -> decltype(&bloom_build_kernel<true, 0, false, 1>)
{
    const bool pow2 = (m_bits & (m_bits - 1)) == 0;
    if (m_bits > kBuildSlabRows) return pow2 ? &bloom_build_kernel<true, 0, false, 1> : &bloom_build_kernel<false, 0, false, 1>;
    if (pow2 && n_ids >= kBuildLongList * n_items && n_tiles >= kBuildLongTiles) return build_kernel<true, 4>(k_hashes);
    if (pow2 && (k_hashes < 2 || k_hashes > 5) && n_ids < kBuildShortList * n_items) return &bloom_build_kernel<true, 0, true, 1, false>;
    return pow2 ? build_kernel<true, 1>(k_hashes) : build_kernel<false, 1>(k_hashes);
}

// In-register transpose of a 32 x 32 bit matrix: bit j of a[i] and bit i of a[j] change places.
// (The steps at distance 16 and 8 exchange whole bytes: one byte permute per word.)
__device__ inline void transpose32(uint32_t (&a)[32])
{
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t lo = a[k], hi = a[k + 16];
        a[k] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
        a[k + 16] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
    }
#pragma unroll
    for (int k0 = 0; k0 < 32; k0 += 16)
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k) {
            const uint32_t lo = a[k], hi = a[k + 8];
            a[k] = __builtin_amdgcn_perm(hi, lo, 0x06020400u);
            a[k + 8] = __builtin_amdgcn_perm(hi, lo, 0x07030501u);
        }
    auto step = [&](auto dist, uint32_t mask) {
        constexpr int j = decltype(dist)::value;
#pragma unroll
        for (int k = 0; k < 32; ++k)
            if ((k & j) == 0) {
                const uint32_t t = ((a[k] >> j) ^ a[k + j]) & mask;
                a[k + j] ^= t;
                a[k] ^= t << j;
            }
    };
    step(std::integral_constant<int, 4>{}, 0x0F0F0F0Fu);
    step(std::integral_constant<int, 2>{}, 0x33333333u);
    step(std::integral_constant<int, 1>{}, 0x55555555u);
}

// Item-major signatures: out[item][word j] gathers bit `item` of 64 rows, i.e. every tile is
// transposed.  A thread takes a block of 32 rows x 32 items: it reads its 32-bit column of the 32
// rows (32 neighbouring lanes cover a row's whole 128-byte line), transposes the block in registers
// and leaves 32 row-bits per item in LDS, from where the items' words go out in order.  A workgroup
// has 16 row blocks: 512 rows of one tile, or all rows of `tiles_per` tiles where a tile has fewer.
// Bound by memory (the index read once, the signatures written once).  One thread per item, gathering
// a bit from every row, took 4.77 ms for 10 M items x 512 bits (each word read 64 times, 64 shifts and
// masks per output word); the transpose takes 0.22 ms, 5.8 TB/s.
constexpr int kExportThreads = 512;
constexpr int kExportBlocks = kExportThreads / 32;  // 32-row blocks of a workgroup
// LDS words of one tile with `blocks` row blocks: the items of neighbouring lanes lie 32 * blocks words
// apart, four words of padding per 32 items spread them over the banks
constexpr int export_tile_words(int blocks) { return kTileItems * blocks + 32 * 4; }
inline int export_tiles_per(int m_bits)
{
    const int blocks = 2 * ((m_bits + 63) / 64);
    return blocks >= kExportBlocks ? 1 : kExportBlocks / blocks;
}
inline int export_lds_bytes(int m_bits)
{
    const int blocks = 2 * ((m_bits + 63) / 64);
    return 4 * export_tiles_per(m_bits) * export_tile_words(blocks < kExportBlocks ? blocks : kExportBlocks);
}

__global__ __launch_bounds__(kExportThreads) void bloom_export_kernel(const uint64_t* __restrict__ bloom,
                                                                      int64_t n_items, int32_t m_bits,
                                                                      int32_t tiles_per, uint64_t* __restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t s_out[];
    const int tid = threadIdx.x;
    const int n_slabs = (m_bits + 63) >> 6, all_blocks = 2 * n_slabs;
    const int64_t tile0 = (int64_t)blockIdx.x * tiles_per;
    const uint32_t* rows = reinterpret_cast<const uint32_t*>(bloom);
    for (int c0 = 0; c0 < all_blocks; c0 += kExportBlocks) {
        const int blocks = min(kExportBlocks, all_blocks - c0);  // (an even number)
        const int unit = tid >> 5, w32 = tid & 31;
        const int tl = unit / blocks, blk = unit - tl * blocks;
        const int64_t item0 = (tile0 + tl) * kTileItems;
        if (tl < tiles_per && item0 < n_items) {
            const int row0 = (c0 + blk) * 32;
            const uint32_t* src = rows + ((tile0 + tl) * (int64_t)m_bits + row0) * 32 + w32;
            uint32_t a[32];
#pragma unroll
            for (int j = 0; j < 32; ++j) a[j] = row0 + j < m_bits ? src[j * 32] : 0u;
            transpose32(a);
            uint32_t* dst = s_out + tl * export_tile_words(blocks) + w32 * (32 * blocks + 4) + blk;
#pragma unroll
            for (int i = 0; i < 32; ++i) dst[i * blocks] = a[i];
        }
        __syncthreads();
        const int words = blocks >> 1;  // 64-bit words per item in this pass
        for (int t = 0; t < tiles_per; ++t) {
            const int64_t first = (tile0 + t) * kTileItems;
            const int n = first >= n_items ? 0 : (n_items - first < kTileItems ? (int)(n_items - first) : kTileItems);
            for (int e = tid; e < n * words; e += kExportThreads) {
                const int it = e / words, w = e - it * words;
                const uint32_t* src = s_out + t * export_tile_words(blocks) + it * blocks + (it >> 5) * 4 + 2 * w;
                out[(first + it) * n_slabs + (c0 >> 1) + w] = *reinterpret_cast<const uint64_t*>(src);
            }
        }
        __syncthreads();
    }
}

// Mask word of one filter: AND of the rows its signature sets, limited to real items.
__device__ inline uint64_t bloom_mask_word(const uint64_t* __restrict__ bloom, int32_t m_bits,
                                           int64_t gw, int64_t n_items,
                                           const int32_t* __restrict__ rows, int n_rows)
{
    const int64_t first = gw * 64;
    if (first >= n_items) return 0;
    const int64_t left = n_items - first;
    uint64_t mask = left >= 64 ? ~0ULL : ((1ULL << left) - 1ULL);
    const uint64_t* base = bloom + ((gw >> 4) * (int64_t)m_bits) * kTileWords + (gw & 15);
    // four independent loads at a time, so that their latencies overlap
    int r = 0;
    for (; r + 4 <= n_rows; r += 4) {
        const uint64_t a = base[(int64_t)rows[r] * kTileWords], b = base[(int64_t)rows[r + 1] * kTileWords];
        const uint64_t c = base[(int64_t)rows[r + 2] * kTileWords], e = base[(int64_t)rows[r + 3] * kTileWords];
        mask &= (a & b) & (c & e);
    }
    for (; r < n_rows; ++r) mask &= base[(int64_t)rows[r] * kTileWords];
    return mask;
}

// dev_mask[f][w] for every filter f and word w (Eq. 4, 64 items per AND).
__global__ __launch_bounds__(256) void bloom_mask_kernel(const uint64_t* __restrict__ bloom,
                                                         int32_t m_bits, int64_t n_items,
                                                         int64_t n_words,
                                                         const int32_t* __restrict__ row_off,
                                                         const int32_t* __restrict__ rows,
                                                         int32_t n_filters,
                                                         uint64_t* __restrict__ out)
{
    const int64_t gw = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    if (gw >= n_words || f >= n_filters) return;
    const int r0 = row_off[f], r1 = row_off[f + 1];
    out[(int64_t)f * n_words + gw] = bloom_mask_word(bloom, m_bits, gw, n_items, rows + r0, r1 - r0);
}

// Boolean filter expressions over per-feature Bloom results (Sec. 4: a query is a conjunction of
// OR-groups of feature = value terms, possibly negated; Sec. 4.3: the per-feature results and the
// operators sit in an operation array that is run in order on a stack).  One thread per 64-item
// word and expression: a leaf pushes the AND of the k signature rows of its feature, NOT / AND /
// OR work on the top of the stack, which lives in LDS (one column per thread, so the dynamic
// depth costs no register indexing).  The host has checked every program: depth <= kExprDepth,
// no pop from an empty stack, one result left.
//   code[i]       operator of entry i (0 leaf, 1 and, 2 or, 3 not)
//   leaf_rows     k_hashes rows per entry (read for leaves only), entry-major
//   prog_off      [n_exprs + 1] entries of each expression; an empty one passes every item
//   out_tile_rows > 0: the result becomes row e of a bit-sliced index of that many rows in the
//                 layout above (the scan kernels read it like a Bloom index whose "signature bit"
//                 e is the whole expression); 0: plain [n_exprs][n_words] masks (Sec. 4.3: 1 bit
//                 per item)
constexpr int kExprDepth = 16;
constexpr int kExprOps = 256;    // entries of one program, at most
constexpr int kExprHashes = 16;  // rows of a leaf, at most

// One program on one 64-item word: s_code / s_rows hold the program (LDS), base points at word w
// of row 0 of the word's tile, column tid of s_stack (NT columns, one per thread) is this thread's stack.  Returns the raw
// result (all ones for the empty program); the caller masks the bits that are not items.
template <int NT>
__device__ inline uint64_t expr_eval_word(const int32_t* s_code, const int32_t* s_rows, int n_ops, int k_hashes,
                                          const uint64_t* __restrict__ base, uint64_t (*s_stack)[NT], int tid)
{
    int top = 0;
    for (int i = 0; i < n_ops; ++i) {
        const int op = s_code[i];
        if (op == 0) {
            // four rows at a time, so that their latencies overlap (a short leaf repeats its last row)
            uint64_t w = ~0ULL;
            const int32_t* rows = s_rows + i * k_hashes;
            for (int j = 0; j < k_hashes; j += 4) {
                const int j1 = j + 1 < k_hashes ? j + 1 : k_hashes - 1, j2 = j + 2 < k_hashes ? j + 2 : k_hashes - 1,
                          j3 = j + 3 < k_hashes ? j + 3 : k_hashes - 1;
                const uint64_t a = base[(int64_t)rows[j] * kTileWords], b = base[(int64_t)rows[j1] * kTileWords];
                const uint64_t c = base[(int64_t)rows[j2] * kTileWords], e = base[(int64_t)rows[j3] * kTileWords];
                w &= (a & b) & (c & e);
            }
            s_stack[top++][tid] = w;
        } else if (op == 3) {
            s_stack[top - 1][tid] = ~s_stack[top - 1][tid];
        } else {
            const uint64_t rhs = s_stack[--top][tid];
            const uint64_t lhs = s_stack[top - 1][tid];
            s_stack[top - 1][tid] = op == 1 ? (lhs & rhs) : (lhs | rhs);
        }
    }
    return n_ops > 0 ? s_stack[0][tid] : ~0ULL;
}

__global__ __launch_bounds__(256) void bloom_expr_kernel(const uint64_t* __restrict__ bloom, int32_t m_bits,
                                                         int32_t k_hashes, int64_t n_items, int64_t n_words,
                                                         const int32_t* __restrict__ prog_off,
                                                         const int32_t* __restrict__ code,
                                                         const int32_t* __restrict__ leaf_rows,
                                                         int32_t out_tile_rows, uint64_t* __restrict__ out)
{
    __shared__ uint64_t s_stack[kExprDepth][256];
    __shared__ int32_t s_code[kExprOps];
    __shared__ int32_t s_rows[kExprOps * kExprHashes];
    const int tid = threadIdx.x;
    const int64_t gw = (int64_t)blockIdx.x * 256 + tid;
    const int e = blockIdx.y;
    // the workgroup's program, fetched once (the tables may sit in pinned host memory: one round
    // trip for the whole workgroup instead of one per entry)
    const int i0 = prog_off[e], n_ops = prog_off[e + 1] - i0;
    for (int i = tid; i < n_ops; i += 256) s_code[i] = code[i0 + i];
    for (int i = tid; i < n_ops * k_hashes; i += 256) s_rows[i] = leaf_rows[(int64_t)i0 * k_hashes + i];
    __syncthreads();
    if (gw >= n_words) return;  // (no barrier below: a thread's stack column is its own)
    const int64_t first = gw * 64;
    const int64_t left = n_items - first;
    const uint64_t valid = left >= 64 ? ~0ULL : (left > 0 ? ((1ULL << left) - 1ULL) : 0ULL);
    const uint64_t* base = bloom + ((gw >> 4) * (int64_t)m_bits) * kTileWords + (gw & 15);
    const uint64_t raw = expr_eval_word(s_code, s_rows, n_ops, k_hashes, base, s_stack, tid);
    // bits past the last item stay 0, also under a NOT
    const uint64_t res = raw & valid;
    if (out_tile_rows > 0)
        out[((gw >> 4) * (int64_t)out_tile_rows + e) * kTileWords + (gw & 15)] = res;
    else
        out[(int64_t)e * n_words + gw] = res;
}

}  // namespace st
