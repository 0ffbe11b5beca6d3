"""The two functions of a photon's random words (csrc/fastmath.hpp: direction,
minus_log_product) against the C library's long-double versions, on the CPU.
Bound: two units in the last place, as for the general functions."""
from __future__ import annotations

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0908_4403_amd", "csrc")

HARNESS = r"""
#define __host__
#define __device__
#include <cmath>
#include <cstdio>
#include <cstdint>
#include <random>
#include <vector>
#include "fastmath.hpp"

static double ulp_err(double got, long double ref) {
    int e; std::frexp((double)ref, &e);
    return (double)(std::fabs((long double)got - ref) / std::ldexp(1.0L, e - 53));
}

int main() {
    using namespace heget::fm;
    const long double pi = 3.141592653589793238462643383279502884L;
    std::mt19937 rng(4321);
    std::vector<uint32_t> words;
    // the ends of the 128 sectors and of the 128 mantissa bins, and their neighbours
    for (uint32_t k = 0; k < 256; ++k)
        for (int d = -2; d <= 2; ++d) words.push_back((k << 24) + d);
    for (int b = 0; b < 32; ++b)
        for (int d = -1; d <= 1; ++d) words.push_back((1u << b) + d);
    const size_t edges = words.size();
    for (int i = 0; i < 1000000; ++i) words.push_back(rng());
    double worst[3] = {0, 0, 0};
    for (uint32_t w : words) {
        double c, s;
        direction(w, kPhotonTables, &c, &s);
        // nearest quarter turn out first: exact in long double
        const long double t = (w + 0.5L) * 0x1p-30L;  // in quarter turns
        const int q = (int)std::nearbyint(t);
        const long double a = (t - q) * pi / 2, s0 = std::sin(a), c0 = std::cos(a);
        const long double rs = (q & 3) == 0 ? s0 : (q & 3) == 1 ? c0 : (q & 3) == 2 ? -s0 : -c0;
        const long double rc = (q & 3) == 0 ? c0 : (q & 3) == 1 ? -s0 : (q & 3) == 2 ? -c0 : s0;
        worst[0] = std::fmax(worst[0], ulp_err(c, rc));
        worst[1] = std::fmax(worst[1], ulp_err(s, rs));
    }
    auto logs = [&](uint32_t a, uint32_t b) {
        const double p = ((a + 0.5) * 0x1p-32) * ((b + 0.5) * 0x1p-32);  // rounded, as the function takes it
        const long double ref = p > 0.5 ? -std::log1p((long double)p - 1) : -std::log((long double)p);
        if (p < 1.0) worst[2] = std::fmax(worst[2], ulp_err(minus_log_product(a, b, kPhotonTables), ref));
    };
    for (size_t i = 0; i < edges; ++i)
        for (size_t j = 0; j <= i; ++j) logs(words[i], words[j]);
    for (size_t i = edges; i + 1 < words.size(); ++i) logs(words[i], words[i + 1]);
    for (uint32_t d = 0; d < 100000; ++d) logs(0xffffffffu - d * 331u, 0xffffffffu - (d & 1023u));
    std::printf("%.3f %.3f %.3f\n", worst[0], worst[1], worst[2]);
    return 0;
}
"""


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    d = tmp_path_factory.mktemp("fmp")
    src = d / "fmp.cpp"
    src.write_text(HARNESS)
    exe = d / "fmp"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    return [float(v) for v in
            subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]


@pytest.mark.parametrize("which, name", [(0, "cos"), (1, "sin"), (2, "-log of a product")])
def test_within_two_ulp(errors, which, name):
    assert errors[which] <= 2.0, (name, errors)
