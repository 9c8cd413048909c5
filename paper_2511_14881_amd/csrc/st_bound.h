// Where a scan may test a pair by integers before it computes the pair's score, and a test that the product itself makes.
//
// A score is ((float)dot * s_q) * s_i with both products rounded, and the tests ask whether dot * s_i, with s_i rounded
// up to fixed point, reaches tau / s_q less 2^-18 of it.  No pair at or above tau is lost by that as long as every
// rounding between is relative (2^-24 of the value):
//   * the first product is an integer times s_q: exact, or at or above 2^-126 and relative, whatever s_q is -- unless it
//     overflows, and then the score is infinite however small s_i may be;
//   * the second one is relative if it reaches a tau of 2^-126 or more.  Below that, half a unit of 2^-149 may be
//     any part of the score: with s_q = s_i = 2^-75 the dots 99,999 and 100,000 give the same one;
//   * a quotient below 2^-126 gives a bound of 0 (the fixed point's factor is below 2^101), which every pair with a
//     positive score meets.
//
// The test within the product.  A pair can only be admitted if dot >= T with T = (tau / s_q) / s_i, a product of a
// number of the query and one of the item.  Both are written as 32 int8 digits, a slice, such that the slices' inner
// product is at most T (every term is rounded down): the query's slice goes behind its row and the
// item's, negated, behind the item's, one contraction step more, and what the matrix unit returns is dot - bound.  Its sign
// is the test; no vector instruction is spent on a pair's scale.  With a reference H of the same size as the items'
// 1 / s_i:
//   u = (tau / s_q) * H / 128, in sixteenths: U + f / 16, U up to 28 * 127     g = (1 / s_i) * 128 / H: g1 + r / 128, below 128
//   u * g >= U * g1 + (U >> 7) * r + ((U & 127) >> 3) * (r >> 4) + f * (g1 >> 4)
// The first term takes 28 digits (U dealt out evenly over them), each of the others one.  Items with 1 / s_i above H count as if it
// were H: a lower bound than theirs, which lets more pairs through.  H is the largest 1 / s_i of a sample of the items,
// less if the largest u would not fit: 28 * 127 * 128 = 455,168 is as large as the digits' product gets.  Relative
// error of the bound below 2 % for U from 128 on and g from 32 on (tests/test_admission_bound.py).
//
// Bounds above that.  Rows with a common mean have dot products, and with them bounds, far beyond 455,168 (rows of 256 bytes
// that fill the int8 range, with a mean cosine of 0.7 between them: 1 M).  H is lowered for want of room then, all bounds stop at
// 455,168 or the query's share of it, and most pairs pass them.  So a part of the bound that all items of a unit share comes first: h is
// 1 / (the unit's largest s_i), the accumulators start at -base with base <= (tau / s_q) * h, a number of the query
// and the unit, and the items' digits are those of 1 / s_i - h.  An item's bound is then below T only where 1 / s_i
// exceeds h + H.  Units whose item of the largest scale needs a dot product of no more than 0.909 * 455,168 have no shared part: there a
// bound that stops at the limit cuts nearly all pairs, too, and the starting values cost some 4 % of a call.
#pragma once
#include <stdint.h>

namespace st {

// tau / s_q for the score of a query's threshold (-infinity: none), or -infinity: no bound, all pairs are tested exactly.
constexpr float bound_quotient(float tau, float s_q)
{
    // (|dot| <= 2^26 for d up to 4096)
    return tau >= 0x1p-126f && s_q <= 0x1p100f && tau / s_q < __builtin_inff() && tau / s_q > 0.0f ? tau / s_q : -__builtin_inff();
}

constexpr int kSliceBytes = 32;
constexpr int kSliceSlots = 28;                             // digits of the first term
constexpr int kSliceTop = kSliceSlots * 127 * 16 + 15;      // largest u, in sixteenths
constexpr float kSliceSlack = 0.99951171875f;               // 1 - 2^-11: more than all roundings of either number

// Whether the digits' range does not do for the largest 1 / s_i of the sample and the largest tau / s_q.
constexpr bool slice_wide(float h_max, float tq_max) { return h_max * (tq_max / 455168.0f) > 1.0f; }
// Units whose largest scale is below this one have a shared part then.
constexpr float slice_shared_below(float tq_max) { return tq_max / (455168.0f * 0.909f); }
// H from the largest 1 / s_i of the sample (0: none is usable) and the largest tau / s_q (0: none).
constexpr float slice_ref(float h_max, float tq_max)
{
    float h = h_max > 0.0f ? h_max : 1.0f;
    if (tq_max > 0.0f && h * (tq_max / 455168.0f) > 1.0f) h = 455168.0f / tq_max;
    return h < 0x1p-90f ? 0x1p-90f : h > 0x1p90f ? 0x1p90f : h;
}
// u in sixteenths; tq > 0.
constexpr int slice_query(float tq, float ref)
{
    const float u = tq * ref * (kSliceSlack * 0.125f);
    return u < (float)kSliceTop ? (int)u : kSliceTop;
}
// g in 128ths from 1 / s_i and 128 * 128 / H * kSliceSlack; 0 for what is not a positive number.
constexpr float slice_factor(float ref) { return 16384.0f * kSliceSlack / ref; }
constexpr int slice_item(float inv, float factor)
{
    const float g = inv * factor;
    return g > 0.0f ? g < 16383.0f ? (int)g : 16383 : 0;
}
// h from the unit's largest scale (0: no shared part), which is below 2^90.
constexpr float slice_shared(float inv_top) { return inv_top < 0x1p90f ? inv_top : 0x1p90f; }
// The part of a unit's bounds that its items share: of a query's u and 8 * h / H, rounded down (2^23 is above any dot product).
constexpr float slice_base_factor(float h, float factor)
{
    const float f = h * (factor * 0x1p-11f);
    return f < 0x1p24f ? f : 0x1p24f;
}
constexpr int slice_base(int u, float base_factor)
{
    const float b = (float)u * base_factor;
    return b < 0x1p23f ? (int)b : 1 << 23;
}
// The slices' inner product.
constexpr int slice_bound(int u, int g)
{
    const int whole = u >> 4, g1 = g >> 7, r = g & 127;
    return whole * g1 + (whole >> 7) * r + ((whole & 127) >> 3) * (r >> 4) + (u & 15) * (g1 >> 4);
}
// Word w of a query's slice, four digits, and of an item's, whose digits are negated.
constexpr int slice_query_word(int u, int w)
{
    const int whole = u >> 4;
    if (w == 7) return whole >> 7 | ((whole & 127) >> 3) << 8 | (u & 15) << 16;
    // (digit j is (whole + j) / 28: the last whole % 28 ones are one larger than the others)
    const int from = kSliceSlots - whole % kSliceSlots - 4 * w;  // first larger one, from this word on
    const uint32_t larger = from <= 0 ? 0x01010101u : from >= 4 ? 0u : 0x01010101u << (8 * from);
    return (int)((uint32_t)(whole / kSliceSlots) * 0x01010101u + larger);
}
constexpr int slice_item_word(int g, int w)
{
    const int g1 = g >> 7, r = g & 127;
    return w < 7 ? (int)((uint32_t)(-g1 & 255) * 0x01010101u) : (-r & 255) | (-(r >> 4) & 255) << 8 | (-(g1 >> 4) & 255) << 16;
}

}  // namespace st
