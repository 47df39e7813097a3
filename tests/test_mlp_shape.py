"""Launch of the MLP stage for every 32-bit count of samples, the last 15 among
them (n + 15 does not fit 32 bits there): csrc/internal.hpp's formulas, compiled
for the host, against whole numbers of any size (CPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = """
#include <cstdio>
#include "internal.hpp"
int main() {
  unsigned n, cu, per;
  while (std::scanf("%u %u %u", &n, &cu, &per) == 3) {
    const vrn::MlpShape s = vrn::mlp_shape(n, cu, per);
    std::printf("%u %u %u\\n", vrn::mlp_tiles(n), s.grid, s.threads);
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2311_02542_amd", "csrc"),
                    str(d / "main.cpp"), "-o", exe], check=True)

    def ask(calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


def test_every_sample_has_a_wave(shapes):
    counts = [1, 15, 16, 17, 4 * 256 * 16, 4 * 256 * 16 + 1, 100003, 1 << 21, (1 << 31) + 5, (1 << 32) - 17, (1 << 32) - 16]
    counts += [(1 << 32) - k for k in range(15, 0, -1)]
    calls = [(n, cu, per) for n in counts for cu in (1, 104, 256) for per in (1, 3)]
    for (n, cu, per), (tiles, grid, threads) in zip(calls, shapes(calls)):
        assert tiles == -(-n // 16)
        waves = threads // 64
        assert threads % 64 == 0 and 4 <= waves <= 8 and 1 <= grid <= cu * per
        # as many blocks as there are tiles for, until the chip is full
        assert grid == min(-(-tiles // waves), cu * per)
        # a block is no larger than its share of the tiles asks for
        assert waves == 4 or waves - 1 < -(-tiles // cu)
