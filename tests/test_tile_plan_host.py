"""GEMM tile plans on the host: the rules of csrc/ffn_plan.h, compiled for the
host alone, at the shapes that stand for each side of a line."""
import os
import subprocess

import pytest

from paper_2608_01891_amd import build
from tests import test_gpu_ffn, test_gpu_gemm_ring, test_gpu_moe, test_gpu_tile_plan

MAIN = r"""
#include <stdio.h>
#include <string.h>
#include "ffn_plan.h"
int main() {
  char op[16];
  int a, b, c, d, e;
  while (scanf("%15s %d %d %d %d %d", op, &a, &b, &c, &d, &e) == 6) {
    if (!strcmp(op, "moe")) {  // T H I E k
      const aflex::MoePlan p = aflex::plan_moe((long long)a * e, b, c, d, e);
      printf("%d %d 0 0\n", p.bm, p.nt);
    } else {  // T N K gate_cols 0
      const aflex::FfnPlan p = aflex::plan_dense(a, b, c, d);
      printf("%d %d %d %d\n", p.bm, p.nt, p.down_splits, p.down_kps);
    }
  }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """Plans of many calls at once: [(rows per tile, non-temporal, K splits, k per split)]."""
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "main.hip", d / "main"
    src.write_text(MAIN)
    cmd = [build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", f"-I{build.CSRC}",
           f"-I{build.INCLUDE}", str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def ask(calls):
        text = "".join(" ".join(map(str, c)) + "\n" for c in calls)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return ask


def linear(T, K, N):
    return ("dense", T, N, K, 0, 0)


def swiglu(T, H, I):
    return ("dense", T, H, I, I, 0)


def moe(T, H, I, E, k):
    return ("moe", T, H, I, E, k)


# calls whose weights come from memory each time (a deep model's) must not lose to keeping them cached
@pytest.mark.parametrize("call,nt", [
    (linear(8, 5120, 5120), 1), (linear(8, 5120, 4096), 0), (linear(16, 8192, 5120), 1), (linear(17, 8192, 5120), 0),
    (linear(64, 8192, 5120), 0), (linear(32, 8192, 10304), 1), (linear(64, 8192, 10304), 1),
    (swiglu(16, 2048, 4096), 0), (swiglu(16, 2048, 5632), 1), (swiglu(32, 2048, 5632), 0), (swiglu(32, 4096, 14336), 1),
    (moe(24, 2048, 512, 8, 2), 0), (moe(24, 2048, 768, 8, 2), 1), (moe(128, 1024, 2816, 8, 2), 1),
    (moe(24, 512, 768, 64, 8), 1), (moe(2048, 1024, 2816, 8, 2), 0)])
def test_non_temporal_weights(plans, call, nt):
    assert plans([call])[0][1] == nt


# 33 ... 128 tokens: one 64-row tile, or two that read the weights twice, against one of 128 rows
@pytest.mark.parametrize("call,bm", [
    (linear(33, 8192, 5120), 64), (linear(64, 8192, 5120), 64), (linear(128, 8192, 5120), 64),
    (linear(64, 5120, 10240), 128), (linear(96, 7168, 9216), 128), (linear(128, 4096, 11264), 128),
    (linear(80, 4096, 9216), 128),
    (linear(40, 4096, 5120), 64), (linear(72, 4096, 5120), 64), (linear(40, 4096, 4096), 64), (linear(40, 5120, 5120), 64), (linear(128, 2048, 16384), 64), (linear(128, 2048, 1024), 64),
    (linear(64, 8192, 10304), 128), (linear(128, 8192, 10304), 128),
    (swiglu(64, 1024, 25600), 64), (swiglu(65, 1024, 25600), 128), (swiglu(128, 2048, 8192), 64),
    (swiglu(64, 4096, 14336), 64), (swiglu(65, 4096, 14336), 128), (swiglu(33, 5120, 25600), 128)])
def test_rows_up_to_128_tokens(plans, call, bm):
    assert plans([call])[0][0] == bm


# more than 128 tokens: 256-row tiles of few k-steps per split against 128-row ones that fill a round
@pytest.mark.parametrize("call,bm", [
    (linear(512, 4096, 4096), 128), (linear(768, 4096, 4096), 256), (linear(1024, 4096, 4096), 128),
    (linear(256, 5120, 5120), 128), (linear(640, 5120, 5120), 256), (linear(256, 8192, 5120), 128),
    (linear(320, 8192, 5120), 256), (linear(768, 2048, 4096), 128), (linear(1536, 2048, 4096), 256), (linear(4096, 4096, 4096), 256),
    (swiglu(512, 4096, 14336), 256)])
def test_few_k_steps(plans, call, bm):
    assert plans([call])[0][0] == bm


# 320-row tiles: a second round of 256-row ones, or not; too many rows for them; rounds to spare
@pytest.mark.parametrize("call,bm", [
    (moe(1000, 1024, 3584, 8, 2), 320), (moe(940, 1024, 3584, 8, 2), 256), (moe(1240, 1024, 3584, 8, 2), 256),
    (moe(1060, 4096, 3584, 8, 2), 320), (moe(1000, 512, 4096, 8, 2), 320), (moe(860, 512, 4096, 8, 2), 256),
    (moe(1120, 3072, 4096, 4, 2), 320), (moe(960, 3072, 4096, 4, 2), 256), (moe(1220, 3072, 4096, 4, 2), 256),
    (moe(1000, 4096, 14336, 8, 2), 256), (moe(2048, 4096, 14336, 8, 2), 256), (moe(1120, 2048, 2048, 8, 2), 256)]
    + [(moe(*c), 320) for c in test_gpu_tile_plan.MOE_ONE_ROUND])
def test_moe_one_round(plans, call, bm):
    assert plans([call])[0][0] == bm


def test_the_ring_tests_take_256_row_tiles(plans):
    r = test_gpu_gemm_ring
    one = plans([linear(*c) for c in r.RING_LINEAR + r.RING_RESIDUAL])
    assert [(p[0], p[2]) for p in one] == [(256, 1)] * len(one)
    split = plans([linear(*c) for c in r.RING_LINEAR_SPLIT])
    assert all(p[0] == 256 and p[2] > 1 for p in split)
    assert {p[0] for p in plans([swiglu(*c) for c in r.RING_SWIGLU] + [moe(*c) for c in r.RING_MOE])} == {256}


def test_the_boundary_tests_take_the_tiles_they_name(plans):
    f, m, t = test_gpu_ffn, test_gpu_moe, test_gpu_tile_plan
    assert [p[0] for p in plans([swiglu(T, f.EDGE_H, f.EDGE_I) for T, _ in f.TILE_EDGES])] == [b for _, b in f.TILE_EDGES]
    assert [p[0] for p in plans([moe(T, m.EDGE_H, m.EDGE_I, 8, 2) for T, _ in m.TILE_EDGES])] == \
        [b for _, b in m.TILE_EDGES]
    for shape, rows in t.LINEAR_ROWS.items():
        assert [p[0] for p in plans([linear(T, *shape) for T in t.LINEAR_T])] == rows, shape
    for shape, rows in t.SWIGLU_ROWS.items():
        assert [p[0] for p in plans([swiglu(T, *shape) for T in t.SWIGLU_T])] == rows, shape
    for shape, rows in t.MOE_ROWS.items():
        assert [p[0] for p in plans([moe(T, *shape, 4, 2) for T in t.MOE_T])] == rows, shape


# splits of linear layers: one work-group per CU instead of a few more, one round instead of several short ones
@pytest.mark.parametrize("call,splits", [
    (linear(40, 4096, 5120), 6), (linear(64, 2560, 8192), 4), (linear(40, 4096, 4096), 8), (linear(64, 8192, 5120), 12),
    (linear(40, 1024, 36864), 1), (linear(1400, 3072, 6144), 1), (linear(1400, 6144, 3072), 3), (linear(3000, 6144, 3072), 1),
    (linear(3000, 3072, 6144), 1), (linear(448, 7168, 9216), 3), (linear(256, 7168, 9216), 7), (linear(2048, 5120, 5120), 3)])
def test_linear_splits(plans, call, splits):
    assert plans([call])[0][2] == splits
