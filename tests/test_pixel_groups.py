"""Batches of more pixels than 32 bits count are split into launches of whole
images (the splitting is plain C++, compiled here on its own)."""
import pathlib
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2305_05600_amd" / "csrc"
MAIN = """
#include <cstdio>
#include <cstdlib>
#include "pixel_groups.hpp"
int main(int, char** a) {
  hvpic::for_pixel_groups(atoll(a[1]), atoll(a[2]), [](int64_t p, int64_t n) { printf("%lld %lld\\n", (long long)p, (long long)n); });
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("groups")
    (d / "m.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(d / "m.cpp"), "-o", str(d / "m")], check=True)
    return d / "m"


# images x pixels: one launch; just at, and above, 2^31; the largest grids and batches that the entry points admit
@pytest.mark.parametrize("images,P", [(1, 1), (8, 131072), (16384, 131072), (16385, 131072), (4096, (1 << 28) - 1),
                                      (17, (1 << 28) - 1), (40, 214748365), (2147483647, 3)])
def test_groups_cover_the_batch(exe, images, P):
    N = images * P
    rows = [tuple(map(int, r.split())) for r in subprocess.run([exe, str(N), str(P)], check=True, capture_output=True,
                                                               text=True).stdout.splitlines()]
    at = 0
    for p, n in rows:
        assert p == at and n % P == 0 and 0 < n <= 1 << 31
        at += n
    assert at == N
    assert len(rows) == -(-images // max(1, (1 << 31) // P))
