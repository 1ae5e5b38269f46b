"""Index and launch arithmetic of the kernels (csrc/launch_rules.h), compiled for the
host and checked against exact integers over the range of grids that the interface
takes (6 N <= 2^31: columns of up to 3.5e8 planes)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_08447_amd", "csrc")
NZ_MAX = (1 << 31) // 6

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "launch_rules.h"
using namespace hkp;
int main() {
  char what[32];
  long long a, b, c;
  const float c0[3] = {2.0f, 2.2f, 2.6f};   // the kernels' kinds
  while (std::scanf("%31s %lld %lld %lld", what, &a, &b, &c) == 4) {
    if (!std::strcmp(what, "range")) std::printf("%d\n", range_begin((int)a, (int)b, (int)c));
    if (!std::strcmp(what, "fold")) std::printf("%zu\n", fold_offset((int)a));
    if (!std::strcmp(what, "room")) std::printf("%d\n", z_split(a, (int)b, c != 0, c0[1]).room);
    if (!std::strcmp(what, "fixed")) std::printf("%d\n", z_split(a, (int)b, c != 0, c0[1]).fixed);
    for (int k = 0; k < 3; ++k)   // ranges of `c` live workgroups in a launch over `a`
      if (!std::strcmp(what, "live"))
        std::printf("%d\n", z_ranges((int)c, (int)b, z_split(a, (int)b, true, c0[k]).room, c0[k]));
  }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def ask(lines):
        r = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, q)) for q in lines),
                           capture_output=True, text=True, check=True)
        return [int(v) for v in r.stdout.split()]

    return ask


def test_z_ranges_tile_every_column(rules):
    """The ranges' bounds are floor(zc nz / zs), from a single plane to the longest column."""
    q = [("range", zc, nz, zs) for nz in (1, 2, 7, 48, 1000, 178956971, NZ_MAX)
         for zs in range(1, 13) if zs <= nz for zc in range(zs + 1)]
    assert rules(q) == [zc * nz // zs for _, zc, nz, zs in q]


def test_phase_rows_beyond_32_bits(rules):
    z = [0, 1, 47, (1 << 31) // 24 - 1, (1 << 31) // 24 + 1, 178956971, NZ_MAX - 1]
    assert rules([("fold", v, 0, 0) for v in z]) == [24 * v for v in z]


def test_few_live_members_of_a_large_batch_are_split(rules):
    """64 members of 16 vectors in 30 tiles each: with few vectors left the launch has to
    spread over the CUs; with all of them alive it is not split."""
    all_ = 64 * 16 * 30
    for left in (1, 2, 4, 8):
        assert all(z >= 2 for z in rules([("live", all_, 40, left * 30)])), left
    assert rules([("live", all_, 40, all_)]) == [1, 1, 1]


def test_room_for_z_ranges(rules):
    """A split decided on the host is the one that the grid holds; one decided on the
    device has room for two ranges wherever the grid's size allows them."""
    sizes = [(n, nz) for n in (1, 30, 480, 4095, 4096, 30720, 1 << 30) for nz in (1, 5, 48)]
    host = [("room", n, nz, 0) for n, nz in sizes], [("fixed", n, nz, 0) for n, nz in sizes]
    assert rules(host[0]) == rules(host[1])
    assert all(r >= 2 for (n, _), r in zip(sizes, rules([("room", n, nz, 1) for n, nz in sizes]))
               if n * 2 < 1 << 31)
    assert rules([("room", (1 << 31) - 1, 48, 1), ("fixed", (1 << 31) - 1, 48, 1)]) == [1, 1]
