"""Division by a prepared constant (hs_internal.h) against the machine's own, for
every small divisor, divisors of every size, and numerators at each multiple's
edge and at random."""
import subprocess

from paper_cs_9809105_amd import build

_SRC = r"""
#include <cstdio>
#include <initializer_list>
#include <cstdint>
#include "hs_internal.h"
using namespace hs;
static uint64_t state = 88172645463325252ull;
static uint32_t rnd() { state ^= state << 13; state ^= state >> 7; state ^= state << 17; return (uint32_t)(state >> 16); }
static int bad = 0;
static void check(uint32_t n, const FastDiv &v) { if (fast_div(n, v) != n / v.d && ++bad < 5) printf("%u / %u\n", n, v.d); }
static void divisor(uint32_t d) {
    const FastDiv v = fast_div_by(d);
    for (uint32_t n : {0u, 1u, d - 1, d, d + 1, 0x7fffffffu, 0x80000000u, 0xfffffffeu, 0xffffffffu}) check(n, v);
    const uint32_t top = 0xffffffffu / d * d;
    check(top, v);
    check(top - 1, v);
    for (int i = 0; i < 60; ++i) {
        const uint32_t r = rnd(), q = r / d * d;
        check(r, v);
        check(q, v);
        check(q - 1, v);
    }
}
int main() {
    for (uint32_t d = 1; d <= 70000; ++d) divisor(d);
    for (int s = 0; s < 32; ++s)
        for (int e = -3; e <= 3; ++e) {
            const uint32_t d = (1u << s) + (uint32_t)e;
            if (d) divisor(d);
        }
    for (int i = 0; i < 200000; ++i) {
        const uint32_t d = rnd() >> (rnd() & 31);
        if (d) divisor(d);
    }
    divisor(0x7fffffffu);
    divisor(0xffffffffu);
    return bad != 0;
}
"""


def test_fast_div(tmp_path):
    src = tmp_path / "t.cpp"
    src.write_text(_SRC)
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
