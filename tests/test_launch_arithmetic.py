"""The kernels' index divisions on the CPU, from the header that the kernels include: division by a launch constant
as a multiplication, and the rounded quotient of planes beyond its range.  Both against the integer division, at the
quotients' edges and at random operands over their whole ranges."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <random>
#include "kvx_internal.h"

static long long wrong = 0, checked = 0;

static void short_division(int64_t n, int64_t d, const kvx::Divisor &by) {
    if (n < 0 || n > INT32_MAX)
        return;
    ++checked;
    if (kvx::divide(static_cast<int>(n), by) != n / d && wrong++ < 5)
        std::printf("divide(%lld, %lld) = %d\n", (long long)n, (long long)d, kvx::divide(static_cast<int>(n), by));
}

static void long_division(int64_t n, int64_t d) {
    if (n < 0 || n >= (int64_t{1} << 53) || n / d > INT32_MAX - 1)
        return;
    ++checked;
    if (kvx::divide_long(n, static_cast<int>(d)) != n / d && wrong++ < 5)
        std::printf("divide_long(%lld, %lld) = %d\n", (long long)n, (long long)d, kvx::divide_long(n, (int)d));
}

int main() {
    std::mt19937_64 rng(12345);
    auto below = [&](int64_t most) {  // spread over the logarithm: 1 <= value <= most
        const int bits = static_cast<int>(rng() % 63);
        const int64_t v = static_cast<int64_t>(rng() >> 1 >> bits) % most + 1;
        return v;
    };
    for (int step = 0; step < 60000; ++step) {
        const int64_t d = step < 2048 ? step + 1 : step < 2112 ? (int64_t{1} << (step - 2048) % 31) + (step % 3 - 1)
                          : below(INT32_MAX);
        if (d < 1)
            continue;
        const kvx::Divisor by = kvx::divisor(d);
        for (int64_t n : {int64_t{0}, int64_t{1}, d - 1, d, d + 1, int64_t{INT32_MAX} - 1, int64_t{INT32_MAX},
                          INT32_MAX / d * d, INT32_MAX / d * d - 1})
            short_division(n, d, by);
        for (int k = 0; k < 32; ++k) {
            const int64_t q = below(INT32_MAX) % (INT32_MAX / d + 1), n = q * d;
            for (int64_t e : {n - 1, n, n + 1, n + d - 1, static_cast<int64_t>(rng() >> 33)})
                short_division(e, d, by);
        }
        // A slab has at most 2^26 vectors, and a plane's first vectors of tiles are multiples of 256.
        const int64_t slab = d % (int64_t{1} << 26) + 1;
        for (int k = 0; k < 32; ++k) {
            const int64_t n = below(INT32_MAX - 1) * slab;
            for (int64_t e : {n - 1, n, n + 1, n + slab - 1, n / 256 * 256, n / 256 * 256 + 256})
                long_division(e, slab);
        }
    }
    std::printf("%lld checked, %lld wrong\n", checked, wrong);
    return wrong != 0;
}
"""


def test_index_divisions_are_exact(tmp_path):
    src, exe = tmp_path / "divide.cpp", tmp_path / "divide"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2609_15021_amd", "csrc"),
                    "-I", "/opt/rocm/include", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 10_000_000, r.stdout
