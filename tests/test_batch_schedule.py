"""Team sizes of the batched engine (batch_schedule.hpp, host code): the tuning that
names the default values is the default, and what the rule gives."""

import os
import shutil
import subprocess

import pytest

from paper_1607_06886_amd import build

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "batch_schedule.hpp"
// scale (-1: no tuning), grid, cap, then per query: its nodes
int main(int argc, char** argv) {
    const int scale = atoi(argv[1]), grid = atoi(argv[2]), cap = atoi(argv[3]);
    const pump_batch_tuning given{256, 2, 1, 1, scale};
    const pump_batch_tuning t = pump::tuning_or_default(scale < 0 ? nullptr : &given);
    double sum = 0.0;
    for (int i = 4; i < argc; ++i) sum += atof(argv[i]) * atof(argv[i]);
    printf("%d %d %d %d\n", t.explore_threads, t.blocks_per_cu, t.order, t.use_graph);
    for (int i = 4; i < argc; ++i) {
        const double n = atof(argv[i]);
        printf("%d ", pump::team_size(t.team_scale, grid, cap, n * n, sum, n));
    }
}
"""


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("schedule")
    src, exe = os.path.join(d, "s.cpp"), os.path.join(d, "s")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I" + os.path.join(build.ROOT, "include"),
                    "-I" + os.path.join(build.HERE, "csrc"), src, "-o", exe], check=True)

    def run(scale, nodes, grid=512, cap=64):
        out = subprocess.run([exe, str(scale), str(grid), str(cap), *map(str, nodes)], check=True,
                             capture_output=True, text=True).stdout.split()
        return [int(v) for v in out[:4]], [int(v) for v in out[4:]]

    return run


BATCHES = [[500], [2000] * 96, [8000, 4000, 2000, 1000] * 8, [300] * 512, [65535, 2, 2], list(range(1000, 8000, 111))]


@pytest.mark.parametrize("nodes", BATCHES)
def test_the_default_by_name_is_the_default(sizes, nodes):
    assert sizes(64, nodes) == sizes(-1, nodes)


@pytest.mark.parametrize("nodes", BATCHES)
@pytest.mark.parametrize("scale", [0, 1, 16, 63, 64, 65, 256])
def test_team_sizes(sizes, scale, nodes):
    _, got = sizes(scale, nodes)
    total = float(sum(n * n for n in nodes))
    for n, size in zip(nodes, got):
        share = 512.0 * n * n / total
        want = 1 if scale == 0 else int(min(max(1.0, (0.25 * scale * share + 0.5) // 1), 64.0))
        if scale == 64:
            want = min(want, int(max(1.0, 3.0 * share, n * n / 2.5e5)))
        assert size == want and 1 <= size <= 64
