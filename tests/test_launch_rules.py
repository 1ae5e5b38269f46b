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
  long long a, b, c, d;
  const float c0[3] = {2.0f, 2.2f, 2.6f};   // the kernels' kinds
  while (std::scanf("%31s %lld %lld %lld %lld", what, &a, &b, &c, &d) == 5) {
    if (!std::strcmp(what, "tune")) {
      TuneShape t[kMaxTuneShapes];
      const int n = tune_shapes((int)a, (int)b, (int)c, d != 0, t);
      for (int i = 0; i < n; ++i)
        std::printf("%d %d %d %d\n", t[i].tile_y, t[i].vgroup, t[i].dma, t[i].zsplit);
    }
    if (!std::strcmp(what, "range")) std::printf("%d\n", range_begin((int)a, z_cut((int)b, ZRanges{(int)c, 1.0f / (float)c})));
    if (!std::strcmp(what, "fold")) std::printf("%zu\n", fold_offset((int)a));
    if (!std::strcmp(what, "room")) std::printf("%d\n", z_split(a, (int)b, c != 0, c0[1], d ? (int)d : kCUs).room);
    if (!std::strcmp(what, "fixed")) std::printf("%d\n", z_split(a, (int)b, c != 0, c0[1], d ? (int)d : kCUs).fixed.zs);
    if (!std::strcmp(what, "ranges"))   // a live workgroups, b planes, at most c ranges, d CUs
      std::printf("%d\n", z_ranges((int)a, (int)b, (int)c, c0[1], (float)d, 1.0f / (float)d).zs);
    if (!std::strcmp(what, "vectors")) std::printf("%lld\n", table_vectors(a, b, c));
    if (!std::strcmp(what, "anew")) std::printf("%d\n", record_anew((int)a, (int)b, c, kCUs) ? 1 : 0);
    for (int k = 0; k < 3; ++k)   // ranges of `c` live workgroups in a launch over `a`
      if (!std::strcmp(what, "live"))
        std::printf("%d\n", z_ranges((int)c, (int)b, z_split(a, (int)b, true, c0[k], kCUs).room, c0[k],
                                     kCUs, 1.0f / kCUs).zs);
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
        r = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, (q + (0, 0, 0))[:5])) for q in lines),
                           capture_output=True, text=True, check=True)
        return [int(v) for v in r.stdout.split()]

    return ask


def test_z_ranges_tile_every_column(rules):
    """The ranges' bounds are floor(zc nz / zs), from a single plane to the longest column."""
    q = [("range", zc, nz, zs) for nz in list(range(1, 60)) + [1000, 178956971, NZ_MAX]
         for zs in range(1, 13) if zs <= nz for zc in range(zs + 1)]
    assert rules(q) == [zc * nz // zs for _, zc, nz, zs in q]


def test_phase_rows_beyond_32_bits(rules):
    z = [0, 1, 47, (1 << 31) // 24 - 1, (1 << 31) // 24 + 1, 178956971, NZ_MAX - 1]
    assert rules([("fold", v, 0, 0) for v in z]) == [24 * v for v in z]


def test_few_live_members_of_a_large_batch_are_split(rules):
    """64 members of 16 vectors in 30 tiles each: with few vectors left the launch has to
    spread over the CUs, whether the host counts them or a recorded launch is made for the
    members left; with all of them alive it is not split."""
    tiles, nb, batch = 30, 16, 64
    all_ = batch * nb
    for left in (1, 2, 4, 8):
        n = rules([("vectors", all_, left, 0)])[0]
        assert n == left
        assert rules([("fixed", n * tiles, 40, 0)])[0] >= 2, left
    for members in (1, 3):
        n = rules([("vectors", all_, -1, members * nb)])[0]
        assert n == members * nb
        assert all(z >= 2 for z in rules([("live", n * tiles, 40, 4 * tiles)]))
    assert rules([("vectors", all_, -1, 0), ("fixed", all_ * tiles, 40, 0)]) == [all_, 1]


def test_recorded_iterations_follow_the_members_left(rules):
    """64 -> 16 -> 4 -> 1 where the launches are large; never for small ones, whose
    recording costs more than it gives."""
    wgs = 16 * 30
    at = [a for a in range(64, 0, -1) if rules([("anew", 64, a, wgs)])[0]]
    assert at == list(range(16, 0, -1))
    assert rules([("anew", 8, 2, 4096 // 8 - 1), ("anew", 8, 2, 4096 // 8), ("anew", 8, 0, 1 << 20)]) == [0, 1, 0]


def test_room_for_z_ranges(rules):
    """A split decided on the host is the one that the grid holds; one decided on the
    device has room for two ranges, unless the launch is too large to be split."""
    sizes = [(n, nz) for n in (1, 30, 480, 4095, 4096, 30720, (1 << 31) - 1) for nz in (1, 5, 48)]
    host = [("room", n, nz, 0) for n, nz in sizes], [("fixed", n, nz, 0) for n, nz in sizes]
    assert rules(host[0]) == rules(host[1])
    room = rules([("room", n, nz, 1) for n, nz in sizes])
    assert all((r >= 2) == (n < 4096) for (n, _), r in zip(sizes, room))
    assert all(n * r < 1 << 31 for (n, _), r in zip(sizes, room))


@pytest.mark.parametrize("cus", [32, 64, 256, 304])
def test_launches_are_balanced_for_the_device(rules, cus):
    """The split minimises planes on the fullest CU of the device's count, whole or a
    partition: against the rule in exact integers."""
    def cost(n, nz, zs):
        return max(-(-n * zs // cus), 2.2) * (nz / zs + 2)
    q = [(n, nz) for n in (1, 7, 30, 31, 32, 33, 100, 255, 256, 257, 480, 511, 513, 2000, 4095)
         for nz in (1, 5, 40, 48)]
    for (n, nz), zs in zip(q, rules([("ranges", n, nz, 8, cus) for n, nz in q])):
        best = min(cost(n, nz, z) for z in range(1, min(8, nz) + 1))
        assert 1 <= zs <= min(8, nz) and cost(n, nz, zs) <= best * (1 + 1e-5), (n, nz, zs)
    # a launch that fills a partition is not split there, but is on the whole GPU
    assert rules([("fixed", 16 * 32, 48, 0, 32)]) == [1]
    assert rules([("fixed", 100, 48, 0, 256)])[0] > 1


@pytest.mark.parametrize("nb", [1, 2, 3, 4, 5, 24])
@pytest.mark.parametrize("ny", [1, 2, 40])
@pytest.mark.parametrize("nx", [64, 75, 192])
@pytest.mark.parametrize("fp64", [0, 1])
def test_tuner_times_the_launches_that_a_filter_makes(rules, nx, ny, nb, fp64):
    """Every shape once, with the z split of the solver's launches; row copies (dma) are a
    choice only where both forms exist, and otherwise the form that the launch takes."""
    v = rules([("tune", nx, ny, nb, fp64)])
    shapes = [tuple(v[i:i + 4]) for i in range(0, len(v), 4)]
    dmas = [0] if nx % 64 else ([0, 1] if fp64 else [1])
    want = [(ty, vg, dma, 1) for dma in dmas for vg in sorted({1, 2, 4, nb}) if vg <= nb
            for ty in (1, 2, 4) if ty <= 2 or ty <= 2 * ny]
    assert sorted(shapes) == sorted(want)
