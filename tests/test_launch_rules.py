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
  while (std::scanf("%31s %lld %lld %lld", what, &a, &b, &c) == 4) {
    if (!std::strcmp(what, "range")) std::printf("%d\n", range_begin((int)a, (int)b, (int)c));
    if (!std::strcmp(what, "fold")) std::printf("%zu\n", fold_offset((int)a));
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
