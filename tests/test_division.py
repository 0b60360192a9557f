"""The division by a constant of the context (div_by, lf_kernels.hip): its
source, taken as it stands and built for the host, against the binary32
division, bit for bit -- every quotient halfway between two subnormal numbers
of short divisors, neighbours of halfway points of normal quotients, random
bits, zeros, infinities and subnormal divisors."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2402_14670_amd", "csrc", "lf_kernels.hip")

DRIVER = r'''
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#define __host__
#define __device__
#define __forceinline__ inline
%s
static uint64_t state = 12345;
static uint32_t rnd() { state = state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(state >> 32); }
static float from(uint32_t u) { float f; std::memcpy(&f, &u, 4); return f; }
static uint32_t bits(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }
static long bad = 0, n = 0;
static void check(float a, float b, double r) {
    volatile float va = a, vb = b;
    const float q = va / vb, p = div_by(a, r);
    ++n;
    if (bits(q) != bits(p) && !(std::isnan(q) && std::isnan(p)) && bad++ < 10)
        std::printf("%%a / %%a: %%a, not %%a\n", a, b, p, q);
}
int main() {
    const float special[] = {0.0f, INFINITY, from(1), from(0x007fffff), from(0x00800000), from(0x7f7fffff), 1.0f, 3.0f};
    for (int it = 0; it < 6000; ++it) {
        // short divisors, which have many exact halfway quotients; random bits
        const float b = it %% 2 ? std::ldexp((float)(2 * (rnd() %% 4096) + 1) * (it %% 4 == 1 ? 1 : -1), (int)(rnd() %% 140) - 40)
                      : it < 16 ? special[it / 2] : from(rnd());
        if (std::isnan(b)) continue;
        const double r = recip(b);
        for (float a : special) { check(a, b, r); check(-a, b, r); }
        for (int j = 0; j < 500; ++j) {
            check(from(rnd()), b, r);
            for (int e : {-150, -130, -40, 60}) {   // halfway quotients k 2^e and their neighbours
                const double k = 2.0 * (rnd() >> (e == -150 ? 9 + rnd() %% 20 : 9)) + 1.0;
                const float a = (float)(k * std::ldexp(1.0, e) * (double)b);
                check(a, b, r);
                check(from(bits(a) + 1), b, r);
                check(from(bits(a) - 1), b, r);
            }
        }
    }
    std::printf("checked %%ld bad %%ld\n", n, bad);
    return bad != 0;
}
'''


def test_division_by_a_constant_is_correctly_rounded(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++ on this host")
    src = open(SRC).read()
    a = src.index("__device__ __forceinline__ double as_double(uint64_t u)")
    b = src.index("// Flags of event ev: of the part")
    prog = tmp_path / "div.cpp"
    prog.write_text(DRIVER % src[a:b])
    exe = tmp_path / "div"
    build = subprocess.run([gxx, "-std=c++17", "-O2", "-ffp-contract=off", str(prog), "-o", str(exe)],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:]
