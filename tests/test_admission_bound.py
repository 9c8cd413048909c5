"""The integer tests that the scans put in front of a pair's score, on the host: whatever the scales (finite and > 0),
a pair whose score reaches the threshold's must pass.  The arithmetic of the kernels is repeated here around the
library's own bound_quotient."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_14881_amd", "csrc")

_PROGRAM = r"""
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>
#include "st_bound.h"

static float score(int dot, float sq, float si)
{
    volatile float a = (float)dot * sq;
    volatile float b = a * si;
    return b;
}
// dot * factor against the threshold's bound, the factor of P bits (scan_tile, scan_mfma2)
static bool passes(int dot, float tq, float si, int E, int P)
{
    const float fix = std::ldexp(1.0f, P - E);
    const int f = std::max((int)std::ceil(si * fix), 1);
    const int thr = std::min((int)std::floor(std::fmin(tq * (fix * 0.99999618530273f), 1.2e9f)), (1 << 30) + 1);
    return (int64_t)dot * f >= thr;
}
// the high half of dot * factor (scan_mfma)
static bool passes_high(int dot, float tq, float si, int E)
{
    const int64_t f = (int64_t)std::ceil(si * std::ldexp(1.0f, 31 - E));
    const int thr = (int)std::floor(std::fmin(tq * std::ldexp(0.99999618530273f, -(E + 1)), 2.0e9f));
    return (int)(((int64_t)dot * f) >> 32) >= thr;
}
int main()
{
    std::mt19937_64 rng(5);
    auto uni = [&](double a, double b) { return a + (b - a) * (double)(rng() >> 11) * 0x1p-53; };
    const int dims[4] = {64, 128, 256, 512};
    long tested = 0, bounded = 0, cut = 0;
    for (long it = 0; it < 4000000; ++it) {
        const int d = dims[it & 3], P = d == 64 ? 10 : d == 128 ? 9 : 8, top = 127 * 127 * d;
        // the threshold's pair, then another one with a score near it
        const double es = uni(-148, 127);
        const float sq = std::fmin((float)std::exp2(es), 3.4e38f);
        double ei = uni(-100, 100);
        if (it & 4) ei = uni(-149.5, -95) - es;  // its score near or below the smallest normal number
        else if (it & 8) ei = uni(80, 127) - es; // ... near or above the largest
        const float si = (float)std::exp2(std::min(std::max(ei, -148.0), 126.9));
        const int dot = (int)std::exp2(uni(0, std::log2((double)top)));
        const float tau = score(dot, sq, si);
        float si2 = si * (it & 16 ? 1.0f : (float)std::exp2(uni(-12, 12)));
        if (!(si2 > 0.0f) || std::isinf(si2)) si2 = si;
        int dot2 = (int)std::min((double)top, std::max(1.0, (double)dot * si / si2 * uni(0.9999, 1.0001) - (it & 32 ? 1 : 0)));
        if (it % 7 == 0) dot2 = (int)std::exp2(uni(0, std::log2((double)top)));
        const float sc2 = score(dot2, sq, si2);
        const float tq = st::bound_quotient(tau, sq);
        const float smax = std::max(si, si2);
        if (!(smax > 0x1p-90f && smax < 0x1p90f)) continue;  // (no integer test then)
        ++tested;
        if (!(tq > 0.0f)) continue;
        ++bounded;
        const int E = std::ilogb(smax) + 1 + (it % 3 == 0 ? (int)uni(0, 8) : 0);  // a wavefront may have met larger scales
        if (E >= 90) continue;
        const bool p = d <= 256 ? passes(dot2, tq, si2, E, P) : true, h = passes_high(dot2, tq, si2, E);
        cut += !p;
        if (sc2 >= tau && !(p && h)) {
            std::printf("cut: d=%d dot=%d dot2=%d sq=%a si=%a si2=%a tau=%a score=%a\n", d, dot, dot2, sq, si, si2, tau, sc2);
            return 1;
        }
    }
    std::printf("ok %ld %ld %ld\n", tested, bounded, cut);
    return 0;
}
"""


def test_integer_bounds_never_cut_a_pair_that_reaches_the_threshold(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "bound.cpp", str(tmp_path / "bound")
    src.write_text(_PROGRAM)
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    assert run.returncode == 0, run.stdout + run.stderr
    ok, tested, bounded, cut = run.stdout.split()
    # ordinary scales keep their bound, and the bound does cut
    assert ok == "ok" and int(bounded) > 0.3 * int(tested) and int(cut) > 0.03 * int(tested), run.stdout


_SLICES = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>
#include "st_bound.h"

int main()
{
    std::mt19937_64 rng(7);
    auto uni = [&](double a, double b) { return a + (b - a) * (double)(rng() >> 11) * 0x1p-53; };
    // the words are the digits, and their products add up to the bound: 32 int8 products, as the matrix unit sums them
    for (int it = 0; it < 200000; ++it) {
        const int u = it < 3 ? (it == 0 ? 0 : it == 1 ? st::kSliceTop : 15) : (int)(rng() % (st::kSliceTop + 1)), g = it % 5 ? (int)(rng() % 16384) : 16383;
        int sum = 0;
        for (int w = 0; w < st::kSliceBytes / 4; ++w)
            for (int j = 0; j < 4; ++j) sum += (int)(int8_t)(st::slice_query_word(u, w) >> (8 * j)) * (int)(int8_t)(st::slice_item_word(g, w) >> (8 * j));
        if (sum != -st::slice_bound(u, g)) return std::printf("words: u=%d g=%d sum=%d bound=%d\n", u, g, sum, st::slice_bound(u, g)), 1;
    }
    // never above tau / s_q / s_i, whatever the reference; and within 2 % of it where both numbers are large enough
    double worst = 0;
    long close = 0;
    for (int it = 0; it < 2000000; ++it) {
        const float si = (float)std::exp2(uni(-100, 89)), T = (float)std::exp2(uni(0, 22)), tq = T * si;
        if (!(tq > 0x1p-126f) || std::isinf(tq)) continue;
        const float h_max = it % 3 ? (float)(uni(0.2, 4) / si) : (float)std::exp2(uni(-100, 100));
        const float ref = st::slice_ref(h_max, tq * (float)uni(1, 3));
        const int u = st::slice_query(tq, ref), g = st::slice_item(1.0f / si, st::slice_factor(ref));
        if (u < 0 || u > st::kSliceTop || g < 0 || g > 16383) return std::printf("range: u=%d g=%d\n", u, g), 1;
        const double exact = (double)tq / si, bound = st::slice_bound(u, g);
        if (bound > exact * (1 - 0x1p-18)) return std::printf("above: si=%a tq=%a ref=%a bound=%g exact=%g\n", si, tq, ref, bound, exact), 1;
        if (u >= 128 * 16 && u < st::kSliceTop && g >= 32 * 128 && g < 16383) {
            ++close;
            worst = std::fmax(worst, 1 - bound / exact);
        }
    }
    std::printf("ok %ld %.5f\n", close, worst);
    return worst < 0.02 ? 0 : 1;
}
"""


def test_the_products_bound_lies_just_below_the_threshold(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "slices.cpp", str(tmp_path / "slices")
    src.write_text(_SLICES)
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    assert run.returncode == 0, run.stdout + run.stderr
    assert int(run.stdout.split()[1]) > 50_000, run.stdout  # most of what is tested has both numbers in their good range


_SHARED = r"""
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>
#include "st_bound.h"

int main()
{
    std::mt19937_64 rng(11);
    auto uni = [&](double a, double b) { return a + (b - a) * (double)(rng() >> 11) * 0x1p-53; };
    // the two parts together: never above tau / s_q / s_i, for scales up to the unit's largest one, whatever the reference
    for (int it = 0; it < 2000000; ++it) {
        const float top = (float)std::exp2(uni(-100, 89)), si = it % 4 ? top * (float)uni(0.01, 1) : top * (float)std::exp2(uni(-40, 0));
        const float tq = (float)std::exp2(uni(0, 23)) * si;
        if (!(tq > 0x1p-126f) || std::isinf(tq) || !(si > 0)) continue;
        const float ref = st::slice_ref(it % 3 ? (float)(uni(0.2, 4) / si) : (float)std::exp2(uni(-100, 100)), tq * (float)uni(1, 30)), factor = st::slice_factor(ref);
        const int u = st::slice_query(tq, ref);
        // (a reciprocal within one unit of its last place)
        const float off[3] = {1.0f - 0x1p-23f, 1.0f, 1.0f + 0x1p-23f};
        const float h = st::slice_shared(1.0f / top * off[it % 3]), inv = 1.0f / si * off[it / 3 % 3];
        const int g = st::slice_item(inv - h, factor), base = st::slice_base(u, st::slice_base_factor(h, factor));
        if (base < 0 || base > 1 << 23 || g < 0 || g > 16383) return std::printf("range: base=%d g=%d\n", base, g), 1;
        const double exact = (double)tq / si, bound = (double)base + st::slice_bound(u, g);
        if (bound > exact * (1 - 0x1p-18)) return std::printf("above: top=%a si=%a tq=%a ref=%a bound=%g exact=%g\n", top, si, tq, ref, bound, exact), 1;
    }
    // how much is let through: rows with a common mean, units of 64 items, thresholds at the 40th of 6,400 items
    for (int form = 0; form < 6; ++form) {
        const int d = form % 2 ? 128 : 256, n = 6400, n_q = 12;
        const double c = form < 2 ? 0.5 : 0.75;
        const bool same = form >= 4;  // all scales alike, as of a table that was quantised with one
        std::vector<int> mu(d), x((size_t)n * d), q((size_t)n_q * d);
        auto row = [&](int* to) {
            for (int i = 0; i < d; ++i) to[i] = (int)std::lrint(std::max(-127.0, std::min(127.0, std::sqrt(c) * mu[i] + std::sqrt(1 - c) * uni(-127, 127))));
        };
        for (int& v : mu) v = (int)uni(-127, 127);
        for (int i = 0; i < n; ++i) row(&x[(size_t)i * d]);
        for (int i = 0; i < n_q; ++i) row(&q[(size_t)i * d]);
        std::vector<float> si(n);
        for (float& s : si) s = same ? 0.01f : (float)uni(0.5, 1.5);
        std::vector<std::vector<int>> dot(n_q, std::vector<int>(n));
        std::vector<float> tq(n_q);
        for (int j = 0; j < n_q; ++j) {
            std::vector<float> sc(n);
            for (int i = 0; i < n; ++i) {
                int a = 0;
                for (int t = 0; t < d; ++t) a += x[(size_t)i * d + t] * q[(size_t)j * d + t];
                dot[j][i] = a;
                sc[i] = (float)a * si[i];
            }
            std::nth_element(sc.begin(), sc.begin() + 40, sc.end(), std::greater<float>());
            tq[j] = sc[40];
        }
        const float h_max = 1.0f / *std::min_element(si.begin(), si.end()), tq_max = *std::max_element(tq.begin(), tq.end());
        const float ref = st::slice_ref(h_max, tq_max), factor = st::slice_factor(ref);
        const float below = st::slice_wide(h_max, tq_max) ? st::slice_shared_below(tq_max) : 0.0f;
        long through = 0, units = 0;
        for (int i0 = 0; i0 < n; i0 += 64) {
            const float top = *std::max_element(si.begin() + i0, si.begin() + i0 + 64), h = top < below ? st::slice_shared(1.0f / top) : 0.0f;
            units += h > 0;
            for (int j = 0; j < n_q; ++j) {
                const int u = st::slice_query(tq[j], ref), base = st::slice_base(u, st::slice_base_factor(h, factor));
                for (int i = i0; i < i0 + 64; ++i) through += dot[j][i] >= base + st::slice_bound(u, st::slice_item(1.0f / si[i] - h, factor));
            }
        }
        std::printf("d %d mean %.2f: %.4f of the pairs, %ld units with a shared part\n", d, c, (double)through / n / n_q, units);
        if (through > n / 50 * n_q || (d == 256 && units == 0)) return 1;  // 0.6 % reach the threshold
    }
    return 0;
}
"""


def test_bounds_beyond_the_digits_range_hold_and_cut(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "shared.cpp", str(tmp_path / "shared")
    src.write_text(_SHARED)
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    assert run.returncode == 0, run.stdout + run.stderr
