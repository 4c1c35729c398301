"""The kernels' index arithmetic, built for the host, against integer division:
the split of a workgroup's index into (token, slice) for every slice count up
to 4096 and at the ends of the index range, and the small division for every
dividend below 2^17 at divisors over its range."""
import subprocess

from paper_2609_36959_amd import build as hip_build

DRIVER = r"""
#include <cstdio>
#include "internal.hpp"
using namespace cobalt;
int main() {
    const uint32_t top = (1u << 31) - 1u;
    for (uint32_t n = 1; n <= 4096; ++n) {
        const Slices s = cut_row((int64_t)n * 64, 1);
        if (s.slices != n) return std::printf("slices of %u\n", n), 1;
        auto bad = [&](uint32_t b) {
            uint32_t t, g;
            s.split(b, &t, &g);
            return t != b / n || g != b % n;
        };
        for (uint32_t k = 0; k < 64; ++k) {  // around multiples of n over the whole range
            const uint32_t q = (uint32_t)((uint64_t)(top / n) * k / 63);
            for (int d = -2; d <= 2; ++d) {
                const int64_t b = (int64_t)q * n + d;
                if (b >= 0 && b <= top && bad((uint32_t)b)) return std::printf("split %u\n", n), 1;
            }
        }
        for (uint32_t b = top - 3; b <= top; ++b)
            if (bad(b)) return std::printf("split %u at the top\n", n), 1;
    }
    for (int64_t y = 1; y <= 1 << 17; y = y < 600 ? y + 1 : y + y / 7) {
        const SmallDiv d = divide_by(y);
        for (int x = 0; x < 1 << 17; ++x)
            if (d(x) != x / y) return std::printf("%d / %d\n", x, (int)y), 1;
    }
    return 0;
}
"""


def test_index_math(tmp_path):
    src, exe = tmp_path / "driver.hip", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run([hip_build.HIPCC, *hip_build.HIPFLAGS, str(src), "-o", str(exe)], check=True,
                   capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
