"""CPU check of the rules that pick the passes of a run (lbm_pick.h, compiled
here for the host): which shape a D2Q9 grid starts with, and where two-step
passes replace it because its columns leave most of a wave idle."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1603_09577_amd", "csrc")
F64, F32, F16 = 0, 1, 2
MAIN = r"""
#include <cstdio>
#include "lbm_pick.h"
int main(int argc, char **argv) {
    if (argc > 1 && argv[1][0] == 'b') {
        int prec; unsigned long long nodes, blocks, tiles;
        while (std::scanf("%d %llu %llu %llu", &prec, &nodes, &blocks, &tiles) == 4)
            std::printf("%d\n", (int)lbm::batch_passes_win(prec, nodes, blocks, tiles, 256));
        return 0;
    }
    if (argc > 1) {
        int prec; unsigned nx, n, src, wall;
        while (std::scanf("%d %u %u %u %u", &prec, &nx, &n, &src, &wall) == 5)
            std::printf("%d\n", (int)lbm::pick_pass3(prec, nx, n, src, wall));
        return 0;
    }
    int prec; unsigned nx, ny, ncu, large, sb, plain;
    while (std::scanf("%d %u %u %u %u %u %u", &prec, &nx, &ny, &ncu, &large, &sb, &plain) == 7) {
        const int s = lbm::pick_multi(prec, nx, ny, ncu);
        std::printf("%d %d\n", s, (int)lbm::two_steps_fit_better(prec, s, nx, ny, ncu, large, sb, plain));
    }
}
"""


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("pick")
    src, exe = d / "pick.cc", d / "pick"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(rows, *mode):
        out = subprocess.run([str(exe), *mode], input="\n".join(" ".join(str(int(v)) for v in r) for r in rows), text=True,
                             capture_output=True, check=True).stdout.split("\n")
        return [tuple(int(v) for v in line.split()) for line in out if line]
    return run


def test_grids_of_the_rule(pick):
    cases = {(F64, 64, 64): 5, (F64, 128, 128): 6, (F32, 128, 128): 6, (F64, 1024, 1024): 4, (F32, 1024, 1024): 3,
             (F16, 1024, 1024): 4, (F16, 4000, 2500): 3, (F32, 512, 512): 3, (F64, 512, 512): 3, (F32, 1000, 723): 4}
    got = pick([(*k, 256, 0, 0, 1) for k in cases])
    assert got == [(v, 0) for v in cases.values()]


def test_ragged_columns(pick):
    """Narrow tall grids: (type, nx, ny, state beyond the cache) -> two-step
    passes instead; FP32 takes the narrower halo of four steps."""
    cases = {(F64, 60, 2200, 0): 0, (F64, 60, 3000, 0): 1, (F64, 60, 20000, 0): 1, (F64, 60, 60000, 1): 1,
             (F64, 58, 20000, 0): 0, (F64, 63, 20000, 0): 0, (F64, 120, 20000, 0): 0, (F64, 62, 1000, 0): 0,
             (F16, 60, 6000, 0): 0, (F16, 60, 8000, 0): 1, (F16, 60, 150000, 1): 1, (F16, 58, 20000, 0): 0,
             (F16, 120, 6000, 0): 0, (F16, 120, 14000, 0): 1, (F16, 120, 60000, 1): 0, (F16, 186, 20000, 0): 0,
             (F32, 60, 20000, 0): 0, (F32, 60, 100000, 1): 0}
    got = pick([(p, nx, ny, 256, b, 0, 1) for p, nx, ny, b in cases])
    assert [g[1] for g in got] == list(cases.values())
    # a step that costs more: Scheme B; walls or rates other than 1
    cases = {(F32, 60, 20000, 0, 1, 1): 1, (F32, 62, 60000, 1, 1, 0): 1, (F32, 60, 20000, 0, 0, 0): 1,
             (F32, 60, 100000, 1, 0, 0): 0, (F32, 60, 8000, 0, 1, 0): 0, (F32, 120, 14000, 0, 1, 0): 0,
             (F64, 120, 14000, 0, 1, 1): 1, (F64, 120, 14000, 0, 0, 0): 0, (F64, 120, 30000, 1, 1, 0): 0}
    got = pick([(p, nx, ny, 256, *rest) for p, nx, ny, *rest in cases])
    assert [g[1] for g in got] == list(cases.values())
    four = pick([(F32, nx, 30000, 256, 0, 0, 1) for nx in (54, 55, 58, 59, 62, 108, 109, 116, 117, 163, 174, 175, 216, 220, 1024)])
    assert [g[0] for g in four] == [3, 4, 4, 3, 3, 3, 4, 4, 3, 4, 4, 3, 3, 3, 3]


def test_wide_and_small_grids_keep_their_passes(pick):
    rows = [(p, nx, ny, 256, b, sb, plain) for p in (F64, F32, F16) for nx in (1, 2, 8, 33, 54, 125, 187, 250, 512, 1000, 4001)
            for ny in (1, 2, 7, 64, 300, 723, 2500, 30000) for b in (0, 1)
            for sb in (0, 1) for plain in (0, 1)]
    rows += [(p, nx, ny, 256, 0, 1, 0) for p in (F64, F32, F16) for nx in (55, 60, 62, 110, 124) for ny in (1, 20, 64, 300, 700)]
    got = pick(rows)
    assert all(0 <= s < 8 and not t for s, t in got)


def test_d3q19_passes(pick):
    """(type, grid, source, walls) -> 0 single sweeps, 1 two steps in 62-node
    columns, 2 in 64-node lines.  FP64 counts the fill of the columns it takes:
    60 nodes fill 62-node ones better than lines."""
    cases = {(F64, (60, 60, 60), 0, 1): 1, (F64, (60, 60, 60), 1, 1): 1, (F64, (60, 60, 60), 0, 0): 1,
             (F64, (58, 58, 58), 0, 1): 0, (F64, (58, 58, 58), 0, 0): 1,
             (F64, (58, 58, 58), 1, 0): 1, (F64, (56, 56, 56), 1, 0): 0, (F64, (60, 60, 30), 0, 0): 0, (F64, (56, 56, 56), 1, 1): 0, (F64, (72, 72, 72), 1, 1): 0,
             (F64, (64, 64, 64), 1, 1): 2, (F64, (62, 62, 62), 1, 1): 1, (F64, (128, 128, 128), 1, 1): 2,
             (F64, (200, 180, 160), 0, 1): 1, (F64, (40, 40, 40), 0, 1): 0,
             (F32, (60, 60, 60), 0, 1): 0, (F32, (64, 64, 64), 0, 1): 2, (F32, (100, 80, 60), 1, 0): 1, (F32, (60, 80, 80), 0, 0): 1, (F32, (96, 96, 96), 0, 1): 2,
             (F32, (256, 256, 256), 0, 1): 2, (F32, (216, 157, 128), 0, 1): 1,
             (F16, (100, 100, 100), 0, 1): 2, (F16, (216, 157, 128), 1, 1): 1, (F16, (100, 100, 100), 0, 0): 0}
    got = pick([(p, n[0], n[0] * n[1] * n[2], s, w) for p, n, s, w in cases], "3")
    assert [g[0] for g in got] == list(cases.values())


def test_batches_of_narrow_or_tiny_instances(pick):
    """(type, nx, ny, instances) -> whether the batch starts with passes."""
    cases = {(F32, 2, 500, 400): 0, (F64, 2, 500, 400): 0, (F16, 500, 2, 400): 0, (F64, 500, 2, 400): 0,
             (F32, 8, 8, 5000): 0, (F32, 4, 4, 20000): 0, (F32, 10, 300, 300): 0, (F64, 16, 16, 4000): 0,
             (F16, 16, 16, 4000): 0, (F16, 24, 24, 2000): 0, (F32, 4, 4, 64): 1, (F64, 8, 8, 400): 1,
             (F32, 32, 32, 1500): 1, (F16, 32, 32, 1500): 1, (F64, 32, 32, 1500): 1, (F64, 64, 64, 400): 1,
             (F16, 64, 64, 400): 1, (F32, 60, 400, 40): 1, (F64, 60, 400, 40): 1, (F32, 300, 300, 128): 1}
    rows = []
    for p, nx, ny, k in cases:
        tw, th = (58, 10) if p == F64 else (54, 22)
        rows.append((p, nx * ny * k, -(-nx * ny // 256) * k, -(-nx // tw) * -(-ny // th) * k))
    assert [g[0] for g in pick(rows, "b")] == list(cases.values())
