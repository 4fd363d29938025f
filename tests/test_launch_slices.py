"""The slices of a launch (``csrc/launch_slices.hpp``) cover every workgroup
once and keep each launch's threads below 2^32, which a corrector call of more
than 67 million elements (241 GB at degree 0 with six quantities) exceeds."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2108_10565_amd", "csrc")
DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "launch_slices.hpp"
int main(int argc, char** argv) {
  const int64_t blocks = std::atoll(argv[1]), fail_at = std::atoll(argv[3]);
  const int threads = std::atoi(argv[2]);
  int64_t calls = 0;
  const int r = stp::for_slices(blocks, threads, 0, [&](int64_t first, unsigned count) {
    std::printf("%lld %u\n", static_cast<long long>(first), count);
    return ++calls == fail_at ? 7 : 0;
  });
  std::printf("result %d\n", r);
}
"""

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("slices")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", d / "driver", d / "driver.cpp"], check=True)

    def run(blocks, threads, fail_at=0):
        out = subprocess.run([d / "driver", str(blocks), str(threads), str(fail_at)], check=True, capture_output=True,
                             text=True).stdout.splitlines()
        return [tuple(map(int, line.split())) for line in out[:-1]], int(out[-1].split()[1])
    return run


@pytest.mark.parametrize("blocks", [0, 1, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, 5 * (1 << 24) + 3])
def test_slices_cover_the_grid(driver, blocks):
    slices, result = driver(blocks, 256)
    assert result == 0
    at = 0
    for first, count in slices:
        assert first == at and count > 0 and count * 256 < 1 << 32
        at += count
    assert at == blocks


def test_first_error_ends_the_slices(driver):
    slices, result = driver(5 * (1 << 24), 256, fail_at=2)
    assert len(slices) == 2 and result == 7
