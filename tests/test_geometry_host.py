"""The library's choice of tiles and K-slices for plans that name neither (choose_geometry),
run on the CPU: the choice at shapes that select each compiled tile, and what holds for
every choice over a sweep of shapes."""
import os
import subprocess

import pytest

from paper_2601_20595_amd import build as libbuild

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "exec_tables.hpp"
int main() {
  int bf16, slots, min_bn, may_split, n_groups;
  long long N, K, ws, rows;
  while (scanf("%d %lld %lld %d %d %d %lld %d", &bf16, &N, &K, &slots, &min_bn, &may_split, &ws, &n_groups) == 8) {
    std::vector<int64_t> groups;
    for (int i = 0; i < n_groups && scanf("%lld", &rows) == 1; ++i) groups.push_back(rows);
    const csg::Geometry g = csg::choose_geometry(bf16, groups, N, K, slots, min_bn, may_split, ws);
    printf("%d %d %d\n", g.bm, g.bn, g.split);
  }
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("geometry")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run([libbuild.hipcc(), "-std=c++17", "-O1", "-I", libbuild.CSRC, "-I",
                    os.path.join(libbuild.ROOT, "include"), str(d / "driver.cpp"),
                    os.path.join(libbuild.CSRC, "exec_tables.cpp"), "-o", exe], check=True, stdout=subprocess.PIPE,
                   stderr=subprocess.STDOUT)

    def run(asked):
        """asked: (bf16, groups, N, K, slots, min_bn, may_split, ws_bytes) each."""
        text = "".join("%d %d %d %d %d %d %d %d %s\n" % (b, n, k, slots, bn, sp, ws, len(g), " ".join(map(str, g)))
                       for b, g, n, k, slots, bn, sp, ws in asked)
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split()
        got = list(map(int, out))
        assert len(got) == 3 * len(asked)
        return [tuple(got[i:i + 3]) for i in range(0, len(got), 3)]
    return run


GIB, MIB16 = 1 << 30, 1 << 24
CHOICES = [
    # bf16, rows per group, N, K, slots, narrowest tile, may split, partial sums -> bm, bn, slices
    (1, [4], 132, 128, 256, 64, 1, GIB, (128, 64, 1)),
    (1, [128], 1792, 4096, 256, 64, 1, GIB, (128, 64, 4)),
    (1, [128], 1792, 4096, 256, 64, 0, GIB, (128, 64, 1)),       # split_k 1 named
    (1, [128], 1792, 4096, 256, 128, 0, GIB, (128, 128, 1)),     # all-reduce
    (1, [1024], 1284, 4096, 256, 64, 1, GIB, (128, 128, 2)),
    (1, [1280], 772, 4096, 256, 64, 1, GIB, (128, 128, 3)),
    (1, [2048], 1792, 4096, 256, 64, 1, GIB, (128, 128, 1)),
    (1, [2048], 2052, 4096, 256, 64, 1, GIB, (256, 256, 3)),
    (1, [4096], 1792, 4096, 256, 64, 1, GIB, (256, 256, 2)),
    (1, [8192], 1792, 4096, 256, 64, 1, GIB, (256, 256, 1)),     # 224 tiles: nothing to cut
    (1, [201, 5, 306], 1792, 4096, 256, 64, 1, GIB, (128, 128, 3)),
    (1, [512], 1792, 4096, 192, 64, 1, GIB, (128, 128, 3)),      # 64 workgroups copy
    (1, [512], 1792, 4096, 256, 64, 1, GIB, (128, 64, 2)),
    (1, [1280], 772, 4096, 256, 64, 1, MIB16, (128, 128, 3)),    # 210 slices of 64 KiB
    (1, [600], 260, 640, 0, 64, 1, GIB, (0, 0, 1)),              # every slot copies: no choice
    (0, [256], 256, 2048, 256, 64, 1, GIB, (64, 64, 8)),
    (0, [256], 256, 256, 256, 64, 1, GIB, (64, 64, 1)),
    (0, [2048], 1024, 1024, 256, 64, 1, GIB, (64, 64, 1)),
]


def test_choices(choose):
    got = choose([c[:8] for c in CHOICES])
    assert got == [c[8] for c in CHOICES]


def test_every_choice_fits(choose):
    """Cut launches run all at once (a unit per slot), slices hold two K steps at least and
    fit their partial sums, and small tiles appear only where all of them run at once."""
    asked = [(b, [m], n, k, slots, bn, sp, ws)
             for b in (0, 1) for m in (1, 64, 129, 700, 2048, 16384) for n in (4, 132, 1028, 4096)
             for k in (64, 640, 4096) for slots in (8, 192, 256) for bn in (64, 128) for sp in (0, 1)
             for ws in (MIB16, GIB) if b or bn == 64]
    for (b, (m,), n, k, slots, bn, sp, ws), (bm, tn, s) in zip(asked, choose(asked)):
        units = -(-m // bm) * -(-n // tn) * s
        assert (bm, tn) in (((256, 256), (128, 128), (128, 64)) if b else ((64, 64),)) and tn >= min(bn, 64 if not b else bn)
        if s > 1:
            assert sp and units <= slots and units * bm * tn * 4 <= ws and k // (64 if b else 16) >= 2 * s
        if b and bm < 256:
            assert units <= slots
