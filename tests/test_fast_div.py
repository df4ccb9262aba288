"""The divisions that the work decomposition uses, against the divide operator and their definitions, on the host."""
import subprocess

from paper_2512_07011_amd import build

SRC = r"""
#include "bsfa_internal.h"
#include <cstdio>
int main()
{
    unsigned long long bad = 0, seen = 0, rng = 88172645463325252ull;
    auto next = [&] { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return (uint32_t)(rng & 0x7fffffffu); };
    auto check = [&](uint32_t d) {
        const bsfa::FastDiv f = bsfa::fast_div(d);
        auto one = [&](uint32_t n) { if (n <= 0x7fffffffu) { ++seen; bad += f.of(n) != n / d; } };
        const uint32_t top = 0x7fffffffu / d * d;
        for (uint32_t n : {0u, 1u, d - 1, d, d + 1, top - 1, top, 0x7ffffffeu, 0x7fffffffu}) one(n);
        for (int i = 0; i < 100; ++i) { one(next()); const uint32_t m = next() / d * d; one(m); if (m) one(m - 1); }
    };
    for (uint32_t d = 1; d <= 5000; ++d) check(d);
    for (int s = 1; s < 31; ++s) for (int e = -1; e <= 1; ++e) if ((1ll << s) + e > 0) check((uint32_t)((1ll << s) + e));
    check(0x7fffffffu);
    for (int i = 0; i < 5000; ++i) check(next() | 1u);
    std::printf("%llu %llu\n", bad, seen);
}
"""


def run_on_host(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run([build.HIPCC, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-std=c++17", "-O2", "-I" + build.CSRC,
                    "-I/opt/rocm/include", "-o", str(exe), str(src)], check=True, capture_output=True)
    return map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())


def test_fast_div_is_exact_below_2_31(tmp_path):
    bad, seen = run_on_host(tmp_path, SRC)
    assert bad == 0 and seen > 1000000


ROW_SRC = r"""
#include "bsfa_internal.h"
#include <cstdio>
int main()
{
    // every item of rows of k items, with shorter runs above them: S(t) = sum - k t, item x is in the last row with S(t) > x
    unsigned long long bad = 0, seen = 0, rng = 88172645463325252ull;
    auto next = [&] { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return (uint32_t)rng; };
    for (int k = 1; k <= 16; ++k)
        for (int i = 0; i < 2000000; ++i) {
            const long sum = 1 + (long)(next() % (i & 1 ? 1u << 30 : 1u << (4 + i % 26))), x = i & 2 ? next() % sum : sum - 1 - (long)(next() % 64) * k % sum;
            const long t = bsfa::counted_row((int)sum, (int)x, k);
            ++seen;
            bad += !(t >= 0 && sum - k * t > x && sum - k * (t + 1) <= x);
        }
    std::printf("%llu %llu\n", bad, seen);
}
"""


def test_row_of_a_counted_item_is_exact(tmp_path):
    """The row of work items that an item is in, for totals up to 2^30 (the largest that lengths below 2^31 give)."""
    bad, seen = run_on_host(tmp_path, ROW_SRC)
    assert bad == 0 and seen > 1000000
