"""The cover search of the assignment kernel (csrc/cover.hpp), built for the
host, against its definition: the first set of nodes in the order (size,
value) that meets every mask, found by trying all sets in that order."""
import subprocess

import numpy as np
import pytest

from paper_2609_36959_amd import build as hip_build

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "cover.hpp"
template <int KM>
static void solve(const std::vector<uint32_t>& in, std::vector<uint32_t>& out) {
    for (size_t i = 0; i * KM < in.size(); ++i) {
        uint32_t m[KM];
        for (int j = 0; j < KM; ++j) m[j] = in[i * KM + j];
        out.push_back(cobalt::first_cover<KM>(m));
    }
}
int main(int, char** argv) {
    std::vector<uint32_t> in, out;
    FILE* f = std::fopen(argv[1], "rb");
    uint32_t v;
    while (std::fread(&v, 4, 1, f) == 1) in.push_back(v);
    std::fclose(f);
    argv[3][0] == '8' ? solve<8>(in, out) : solve<16>(in, out);
    f = std::fopen(argv[2], "wb");
    std::fwrite(out.data(), 4, out.size(), f);
    std::fclose(f);
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("cover")
    src, exe = d / "driver.hip", d / "driver"
    src.write_text(DRIVER)
    subprocess.run([hip_build.HIPCC, *hip_build.HIPFLAGS, str(src), "-o", str(exe)], check=True,
                   capture_output=True)

    def run(masks):
        masks = np.ascontiguousarray(masks, np.uint32)
        masks.tofile(d / "in")
        subprocess.run([str(exe), str(d / "in"), str(d / "out"), str(masks.shape[1])], check=True)
        return np.fromfile(d / "out", np.uint32)
    return run


def by_definition(masks, bits):
    """Tries every non-empty set of the `bits` nodes in order, all rows at once."""
    sets = sorted(range(1, 1 << bits), key=lambda b: (bin(b).count("1"), b))
    out = np.zeros(len(masks), np.uint32)
    todo = np.arange(len(masks))
    for b in sets:
        met = ((masks[todo] & b) != 0) | (masks[todo] == 0)
        hit = met.all(axis=1)
        out[todo[hit]] = b
        todo = todo[~hit]
        if not len(todo):
            break
    return out


@pytest.mark.parametrize("KM", [8, 16])
@pytest.mark.parametrize("bits", [1, 2, 3, 7, 8, 12, 15])
def test_first_cover(driver, KM, bits):
    rng = np.random.default_rng(100 * KM + bits)
    rows = []
    for size in (1, 2, 2, 2, 3, 5, bits):  # nodes per mask; two where replicas are few
        m = np.zeros((150, KM), np.uint32)
        for _ in range(size):
            m |= np.uint32(1) << rng.integers(0, bits, m.shape).astype(np.uint32)
        # some slots without a mask: at the end, as for K < KM, or anywhere
        k = rng.integers(1, KM + 1, len(m))
        m[np.arange(KM) >= k[:, None]] = 0
        m[50:100][rng.random((50, KM)) < 0.3] = 0
        rows.append(m)
    m = np.concatenate(rows)
    m = m[(m != 0).any(axis=1)]
    assert np.array_equal(driver(m), by_definition(m, bits))


def test_first_cover_small_exhaustive(driver):
    """Every triple of masks over four nodes."""
    a = np.arange(1, 16, dtype=np.uint32)
    m = np.zeros((15 ** 3, 8), np.uint32)
    m[:, 0], m[:, 3], m[:, 7] = (v.ravel() for v in np.meshgrid(a, a, a))
    assert np.array_equal(driver(m), by_definition(m, 4))
