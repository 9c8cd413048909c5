// Where a scan may test a pair by integers before it computes the pair's score.
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
#pragma once

namespace st {

// tau / s_q for the score of a query's threshold (-infinity: none), or -infinity: no bound, all pairs are tested exactly.
constexpr float bound_quotient(float tau, float s_q)
{
    // (|dot| <= 2^26 for d up to 4096)
    return tau >= 0x1p-126f && s_q <= 0x1p100f && tau / s_q < __builtin_inff() && tau / s_q > 0.0f ? tau / s_q : -__builtin_inff();
}

}  // namespace st
