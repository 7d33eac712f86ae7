"""Layouts that the device code relies on, checked by the compiler (no GPU)."""

import os
import subprocess

import pytest

from paper_1607_06886_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _holds(tmp_path, header, *checks):
    src = os.path.join(str(tmp_path), "check.hip")
    with open(src, "w") as f:
        f.write(f'#include "{header}"\n' + "".join(f"static_assert({c}, {c!r});\n".replace("'", '"') for c in checks))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only",
                        "-Wno-unused-command-line-argument",
                        "-I" + os.path.join(build.ROOT, "include"), "-I" + os.path.join(build.HERE, "csrc"), src],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


needs_hipcc = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


@needs_hipcc
def test_rank_table_lds_is_read_16_bytes_at_a_time(tmp_path):
    _holds(tmp_path, "rank_tables.hpp", "alignof(pump::RankLds) >= 16",
           "offsetof(pump::RankLds, key) % 16 == 0", "offsetof(pump::RankLds, rank) % 16 == 0")


@needs_hipcc
def test_expansion_counters_are_64_bits_wide(tmp_path):
    """One workgroup may carry a whole query (pump_batch_tuning.team_scale 0)."""
    _holds(tmp_path, "explore_lane.hpp",
           *[f"sizeof(pump::PairTotals::{k}) == 8" for k in ("sim", "pre", "drop", "wp", "bt", "flag")])
