"""What hartree_plan_tune chooses among in FP32: per axis and length one radix
plan, and only tiles that give the same values bit for bit, so that the values
of a tuned plan do not depend on timings."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1209_4506_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1209_4506_amd", "csrc")
CELL = np.array([[20.2, 0.0, 0.0], [3.0, 25.2, 0.0], [-2.0, 1.0, 28.3]])
LENGTHS = [32, 48, 60, 64, 72, 90, 96, 120, 128, 150, 160, 180, 192, 200, 210, 240, 256, 288, 300, 320, 360, 384, 400, 420,
           480, 512, 576, 600, 640, 720, 768, 800, 840, 960, 1024, 2048]
SEVERAL = {48: 2, 128: 2, 160: 2, 180: 3, 360: 6}  # compiled radix plans of a length, where not one


@pytest.fixture(scope="module")
def choices(tmp_path_factory):
    """The host functions that select what is timed, compiled by themselves."""
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("tune")
    src, out = str(d / "t.cpp"), str(d / "t.so")
    with open(src, "w") as fh:
        fh.write('#include "tune.hpp"\n'
                 'extern "C" int times(int f, int x, int n, int plan, int lp, int pad)\n'
                 "{ return hartree::tune_times(f, x, n, plan, lp, pad); }\n"
                 'extern "C" int sized(int x, int n) { return hartree::multi_sized_only(x, n); }\n')
    r = subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(out)


def set_axis(LIB, h, base, x, choice):
    cfg = (ctypes.c_int32 * 9)(*base)
    cfg[3 * x:3 * x + 3] = choice
    return LIB.hartree_plan_set_config(h, cfg) == 0


def axis_choices(x):
    return [(i, lp, pad) for i in range(-1, 64) for lp in range(7) for pad in ((0,) if x == 2 else (0, 1, 2))]


@pytest.mark.parametrize("prec", [0, 1])
def test_one_radix_plan_per_length(choices, prec):
    """Of the compiled choices that a plan accepts the tuner times one radix
    plan in FP32, with at least one tile, and every one in FP64 (host checks)."""
    from paper_1209_4506_amd.hartree import LIB

    vp, i32, d = ctypes.c_void_p, ctypes.c_int32, ctypes.c_double
    # (without a device 64 KiB of LDS are assumed: 2,048 in FP64 has no tile)
    for n in LENGTHS if prec == 1 else LENGTHS[:-1]:
        for x in range(3):
            dims = [12, 10, 14]
            dims[x] = n
            h = vp()
            assert LIB.hartree_plan_create(ctypes.byref(h), (d * 9)(*CELL.reshape(9)), (i32 * 3)(*dims), prec, None) == 0
            base = (ctypes.c_int32 * 9)()
            assert LIB.hartree_plan_get_config(h, base) == 0
            accepted = [c for c in axis_choices(x) if c[0] >= 0 and set_axis(LIB, h, list(base), x, c)]
            timed = [c for c in accepted if choices.times(1 - prec, x, n, *c)]
            LIB.hartree_plan_destroy(h)
            assert len({c[0] for c in accepted}) == SEVERAL.get(n, 1), (n, x)
            assert len({c[0] for c in timed}) == (1 if prec == 1 else SEVERAL.get(n, 1)), (n, x, timed)
            assert prec == 1 or timed == accepted


def values(torch, plan, rho, ge):
    V, E = plan.solve(rho)
    G = plan.backward(grad_v=rho * 0.3, grad_e=ge, rho=rho)
    F = plan.backward(grad_e=ge, rho=rho)
    torch.cuda.synchronize()
    return [t.clone() for t in (V, G, F)], E.clone()


def same(torch, got, want, what):
    assert all(torch.equal(a, b) for a, b in zip(got[0], want[0])), what
    # (E_H sums its tiles' parts in double)
    assert torch.allclose(got[1], want[1], rtol=1e-13, atol=0.0), what


@pytest.mark.gpu
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_timed_choices_agree(choices, axis):
    """Every choice that the tuner times for a length gives the same potential
    and gradients, bit for bit."""
    import torch

    from paper_1209_4506_amd.hartree import HartreeError, Plan

    for n in LENGTHS:
        print("case timed choices", axis, n, flush=True)
        dims = [24, 20, 18]
        dims[axis] = n
        plan = Plan(CELL, dims, precision="fp32", max_atoms=1)
        base = plan.get_config()
        rho = torch.as_tensor(inputs.random_grid(tuple(dims), 71).astype(np.float32), device="cuda")
        ge = torch.tensor([0.3], dtype=torch.float64, device="cuda")
        want = None
        for c in axis_choices(axis):
            if c[0] < 0 or not choices.times(0, axis, n, *c):
                continue
            cfg = base.copy()
            cfg[0, axis] = c
            try:
                plan.set_config(cfg)
            except HartreeError:
                continue
            got = values(torch, plan, rho, ge)
            want = want or got
            same(torch, got, want, (axis, n, c))
        assert want is not None


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(48, 128, 160), (160, 48, 128), (128, 160, 180), (180, 360, 48), (360, 180, 96), (96, 64, 360),
                                  "several", "one", "listed"])
def test_tuning_again(dims):
    """Plans of one workload tuned apart give the same potential and gradients:
    lengths with several radix plans, and batches (of several lengths on an
    axis, of one, and of lengths outside the multi-plan list)."""
    import torch

    from paper_1209_4506_amd.hartree import Plan

    print("case tuning again", dims, flush=True)
    shapes = {"several": [(48, 60, 64), (64, 96, 60), (96, 48, 128), (60, 180, 72)], "one": [(48, 180, 64)] * 3,
              "listed": [(48, 300, 135), (180, 60, 128)]}.get(dims)
    want = None
    for _ in range(4):
        if shapes is None:
            plan = Plan(CELL, dims, precision="fp32", max_atoms=1)
        else:
            plan = Plan(np.stack([CELL] * len(shapes)), np.array(shapes), precision="fp32", max_atoms=1)
        plan.tune(reps=1)
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        rho = plan.empty_grid().normal_(generator=g)
        got = values(torch, plan, rho, torch.full((plan.nprob,), 0.3, dtype=torch.float64, device="cuda"))
        want = want or got
        same(torch, got, want, dims)
