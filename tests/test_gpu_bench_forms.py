"""The launches that the benchmark's forms report are those of the timed lbm_step call."""
import os
import sys

import pytest

from gpu_helpers import gpu_solver, smooth_random_2d

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,steps,fuse", [(1024, 40, 0), (1024, 2, 0), (300, 40, 0), (1024, 7, 1)])
def test_forward_form(n, steps, fuse):
    import torch

    out = bench.time_forward(torch, n, "f64", steps, 2, 256, 1, 0, fuse=fuse)
    plan = gpu_solver(smooth_random_2d(n, n, lam=6.0, s=1.7), fuse_steps=fuse).run_plan(steps)
    pieces = [l["steps"] for l in plan]
    assert out["launches"] == len(plan) and out["steps_per_launch"] == max(pieces)
    assert out["launch_steps"] == {str(k): pieces.count(k) for k in sorted(set(pieces), reverse=True)}
    top = next(l for l in plan if l["steps"] == out["dominant_steps"])
    assert (out["kernel"], out["segment_rows"]) == (top["kernel"], top["rows"])
    kind = {"step": "one_step", "lds2": "lds_two_step", "strip": "wave_strip", "tile": "tile"}[top["kernel"]]
    assert bench.kernel_kind(out) == kind


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_rest_form_is_one_call(storage):
    import torch

    from paper_1401_0427_amd.lbm import Solver

    out = bench.time_rest_2d(torch, 512, storage, steps=31, warmup=2)
    c = smooth_random_2d(512, 512, lam=6.0, s=1.7)
    S = Solver(2, 512, 512, lam=c.lam, s=c.s, h0=c.h0, rest=True, a=bench.REST_A,
               rates=list(bench.REST_RATES_2D), storage=storage)
    assert out["launches"] == len(S.run_plan(31))
    assert out["steps_per_launch"] == max(l["steps"] for l in S.run_plan(31))
