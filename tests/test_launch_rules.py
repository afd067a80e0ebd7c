"""The rules that choose a launch from its sizes, compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_20525_amd", "csrc")
SIMDS = 1024


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src = d / "rules.cpp"
    src.write_text('''
#include <stdio.h>
#include <string.h>
#include "launch_rules.h"
int main(int n, char **v) {
    int a[8] = {0};
    for (int i = 2; i < n; ++i) sscanf(v[i], "%d", &a[i - 2]);
    if (!strcmp(v[1], "est_share_rounds"))
        printf("%d", plan::est_share_rounds(a[0], a[1], a[2], a[3]));
    if (!strcmp(v[1], "costmap_small_tiles"))
        printf("%d", plan::costmap_small_tiles(a[0], a[1], a[2]));
    if (!strcmp(v[1], "softmin_entries"))
        printf("%d", plan::softmin_entries(a[0], a[1]));
    return 0;
}
''')
    exe = d / "rules"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    return lambda name, *a: int(subprocess.run([str(exe), name, *map(str, a)], check=True,
                                               capture_output=True, text=True).stdout)


@pytest.mark.parametrize("K,N,S,rounds", [
    # long horizons of several substeps, by the remainder
    (65536, 16, 50, 0), (65537, 16, 50, 1), (66000, 16, 50, 1), (80000, 16, 50, 1),
    (90000, 16, 50, 0), (137000, 16, 50, 2), (170000, 16, 50, 2), (185000, 16, 50, 0),
    (204288, 16, 50, 3), (240000, 16, 50, 3), (270000, 16, 50, 4), (300000, 16, 50, 0),
    (350000, 16, 50, 5), (400000, 16, 50, 6), (7 * 65536 + 64, 16, 50, 0),
    # one substep: smaller remainders only
    (66000, 100, 1, 1), (80000, 100, 1, 0), (147000, 100, 1, 2), (170000, 100, 1, 0),
    (204288, 100, 1, 3), (240000, 100, 1, 0),
    # a few steps are never shared
    (66000, 5, 1, 0), (66000, 24, 1, 0), (66000, 25, 1, 1), (204288, 1, 24, 0),
    (204288, 1, 25, 3), (400000, 4, 5, 0), (400000, 2, 2**30, 6)])
def test_est_shares_its_steps_where_that_is_faster(rule, K, N, S, rounds):
    assert rule("est_share_rounds", (K + 63) // 64, SIMDS, N, S) == rounds


@pytest.mark.parametrize("W,H,small", [
    (2, 2, 1), (64, 64, 1), (600, 600, 1), (700, 700, 0), (2048, 2048, 0), (1537, 1025, 0),
    (32 * 447, 1, 1), (32 * 447 + 1, 1, 0), (1, 32 * 448, 0), (67108863, 1, 0)])
def test_costmap_tiles_by_the_size_of_the_map(rule, W, H, small):
    assert rule("costmap_small_tiles", W, H, SIMDS // 4) == small


@pytest.mark.parametrize("K,N,entries", [
    (1, 1, 1), (200000, 128, 1), (1, 129, 2), (4096, 256, 2), (6144, 256, 2), (6145, 256, 4),
    (8192, 170, 2), (8192, 171, 4), (14335, 170, 2), (14336, 170, 4), (19999, 256, 4),
    (20000, 256, 2), (20000, 257, 4), (1, 2**30, 4)])
def test_softmin_entries_a_workgroup(rule, K, N, entries):
    assert rule("softmin_entries", K, N) == entries
