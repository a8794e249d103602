"""The attention's split plan (csrc/attn_plan.h, plain C++) over the shapes the entry points take: every unit in
exactly one split, partials that fit the reported workspace, and in a pipelined step no workgroup that has to wait
for a CU which the staging kernel holds when fewer splits would have shortened the chain."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "attn_plan.h"
extern "C" void plan(int R, int Hq, int Hkv, int T, int B, int k, int busy, long long* o) {
  const oasis::AttnPlan p = oasis::attn_plan(R, Hq, Hkv, T, B, k, busy);
  o[0] = p.rows; o[1] = p.n_units; o[2] = p.nsplit; o[3] = p.units_per_split; o[4] = p.part_o_floats; o[5] = p.bytes;
}
"""
CUS = 256


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = os.environ.get("CXX") or shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2608_08097_amd", "csrc"), str(d / "shim.cpp"), "-o", str(d / "shim.so")],
                   check=True)
    f = ctypes.CDLL(str(d / "shim.so")).plan

    def call(R, Hq, Hkv, T, B, k, busy=0):
        o = (ctypes.c_longlong * 6)()
        f(R, Hq, Hkv, T, B, k, busy, o)
        return dict(zip(("rows", "units", "nsplit", "per", "part_o", "bytes"), o))

    return call


SHAPES = [(R, G * H, H, T, B, k) for R in (1, 2, 3, 6, 8, 12, 16, 17, 24, 31, 33, 64, 90) for H in (1, 2, 4, 8)
          for G, T in ((1, 1), (4, 5), (8, 4), (5, 7), (4, 9), (8, 9), (16, 5)) for B in (16, 32)
          for k in (0, 1, 5, 31, 64, 128, 257, 1024)]


def _staging(B, pairs):
    grid = 32 if B == 16 else min(64, max(32, pairs // 2))
    return min(grid, pairs)


def test_plans_cover_the_units_and_fit_the_workspace(plan):
    for s in SHAPES:
        R, _, H, _, B, k = s
        base = plan(*s)
        for busy in (0, _staging(B, R * H), 255, 300):
            p = plan(*s, busy)
            assert (p["nsplit"] - 1) * p["per"] < p["units"] <= p["nsplit"] * p["per"] and 1 <= p["nsplit"] <= 16, s
            assert p["bytes"] == base["bytes"], s  # the workspace serves the single call and the step alike
            if p["nsplit"] > 1:
                assert p["part_o"] == R * H * p["nsplit"] * p["rows"] * 128, s
                assert p["part_o"] * 4 + R * H * p["nsplit"] * p["rows"] * 8 <= p["bytes"], s
            else:
                assert p["part_o"] == 0, s


def test_a_step_with_many_rows_leaves_the_staging_workgroups_their_cus(plan):
    for s in SHAPES:
        R, _, H, _, B, _ = s
        busy = _staging(B, R * H)
        alone, p = plan(*s), plan(*s, busy)
        if p["rows"] <= 32:  # two such workgroups and a staging one fit a CU's LDS: planned as alone
            assert p == alone, s
            continue

        def chain(x):
            return -(-R * H * x["nsplit"] // (CUS - busy)) * x["per"]

        assert p["nsplit"] <= alone["nsplit"] and chain(p) <= chain(alone), s
    # 48 pairs of 35 rows: 5 splits (240 workgroups) would not fit beside 32 staging workgroups
    assert plan(12, 20, 4, 7, 16, 128)["nsplit"] == 5
    assert plan(12, 20, 4, 7, 16, 128, 32)["nsplit"] * 48 <= CUS - 32
