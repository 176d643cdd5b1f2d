"""The attention plans' arithmetic, the library's own (csrc/attn.hpp) compiled for the CPU, over
random ragged batches: every key tile in one work item, partial slots distinct, within the workspace and
where the merge looks for them, splits no more than the workgroups launched."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_31315_amd", "csrc")
MIN_TILES = int(re.search(r"constexpr int kBalMinTiles = (\d+);", open(os.path.join(CSRC, "sd_block.hip")).read()).group(1))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                    os.path.join(HERE, "attn_plan_check.cpp")], check=True)
    return ctypes.CDLL(so)


def _i32(x):
    return np.ascontiguousarray(x, np.int32).ctypes.data_as(ctypes.c_void_p)


def _batch(rng, S, G, hi):
    ctx = rng.integers(0, hi, S).astype(np.int32)
    top = min(64, 256 // G)
    B = np.where(rng.random(S) < 0.1, 0, rng.integers(1, int(rng.integers(1, top + 1)) + 1, S)).astype(np.int32)
    return ctx, B


@pytest.mark.parametrize("seed", range(8))
def test_balanced(plan, seed):
    rng = np.random.default_rng(seed)
    for _ in range(10):
        S, Hkv, G = int(rng.integers(1, 90)), int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 4, 5, 8, 32]))
        ctx, B = _batch(rng, S, G, int(rng.choice([300, 3000, 33000])))
        line = plan.check_bal(S, Hkv, G, _i32(ctx), _i32(B), 64, MIN_TILES)
        assert line == 0, f"attn_plan_check.cpp:{line}"


@pytest.mark.parametrize("grid", [256, 255, 100, 17, 1])
@pytest.mark.parametrize("S,Hkv", [(1, 1), (1, 8), (4, 8), (15, 8), (16, 8), (62, 2), (63, 2), (40, 8), (130, 1), (200, 2)])
def test_fp32(plan, S, Hkv, grid):
    """Pairs on both sides of 15/31 of the grid (124 of 256), one group and several, whole and reduced workspaces."""
    rng = np.random.default_rng(S * 1000 + Hkv * 10 + grid)
    n = ctypes.c_int(0)
    for G in (1, 4, 8, 12):
        for hi in (1, 200, 3000, 33000):
            ctx, B = _batch(rng, S, G, hi)
            line = plan.check_f32(S, Hkv, G, max(1, int(B.max())), _i32(ctx), _i32(B), grid, ctypes.byref(n))
            assert line == 0, f"attn_plan_check.cpp:{line}"


def test_fp32_uniform_batch_fills_the_grid(plan):
    """4 sequences x 8 kv heads of 2048 keys: the splits are most of the grid, so the plan is not trivially small."""
    ctx, B, n = np.full(4, 2048), np.full(4, 16), ctypes.c_int(0)
    assert plan.check_f32(4, 8, 4, 16, _i32(ctx), _i32(B), 256, ctypes.byref(n)) == 0
    assert 200 <= n.value <= 256
