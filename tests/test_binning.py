"""The rule between the two forms of the binning, and grids whose columns of
bricks are long."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1209_4506_amd", "csrc")


@pytest.fixture(scope="module")
def by_columns(tmp_path_factory):
    """bin_by_columns for problems on a grid of spacing 0.2 and widths up to
    0.7, compiled by itself."""
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("bin")
    src, out = str(d / "b.cpp"), str(d / "b.so")
    with open(src, "w") as fh:
        fh.write('#include "bin_rule.hpp"\n'
                 'extern "C" int columns(int n, const hartree::BinShape *s) { return hartree::bin_by_columns(n, s); }\n')
    r = subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(out)

    class Shape(ctypes.Structure):
        _fields_ = [("nb", ctypes.c_int * 3), ("touch", ctypes.c_double * 3), ("atoms", ctypes.c_int)]

    def call(brick, cutoff, *problems):
        shapes = (Shape * len(problems))()
        for s, (dims, atoms) in zip(shapes, problems):
            s.atoms = atoms
            for x in range(3):
                s.nb[x] = -(-dims[x] // brick[x])
                s.touch[x] = min(s.nb[x], int(2 * cutoff * 0.7 / 0.2) / brick[x] + 1)
        return bool(lib.columns(len(problems), shapes))

    return call


def test_rule(by_columns):
    """The form that measured faster by more than a quarter (us, columns /
    visits), FP32 and diagonal cells but where it says otherwise; more than
    4,096 atoms in a problem never fit the columns."""
    large, small = (16, 16, 32), (8, 8, 32)
    for dims, atoms, columns in (((16, 16, 16), 1, True),           # 15 / 20
                                 ((16, 16, 16), 4096, True),        # 84 / 221
                                 ((64, 64, 64), 4096, True),        # 71 / 200
                                 ((96, 100, 90), 1500, True),       # 20 / 60
                                 ((256, 256, 256), 4096, True),     # 21 / 31
                                 ((512, 512, 512), 4096, True),     # 29 / 40
                                 ((1024, 1024, 1024), 4096, True),  # 72 / 140
                                 ((1024, 1024, 1024), 1, True),     # 15 / 99
                                 ((40, 2048, 64), 4096, True),      # 21 / 35
                                 ((1024, 1024, 8), 16, True),       # 14 / 20
                                 ((1024, 1024, 8), 256, False),     # 32 / 21
                                 ((1024, 1024, 8), 4096, False),    # 64 / 26
                                 ((2048, 2048, 8), 4096, False),    # 189 / 38
                                 ((8, 8, 4096), 256, False),        # 45 / 20
                                 ((8, 8, 4096), 4096, False)):      # 553 / 42
        assert by_columns(large, 6.0, (dims, atoms)) == columns, (dims, atoms)
        assert not by_columns(large, 6.0, (dims, 4097))
        assert not by_columns(large, 6.0, ((48, 60, 72), 100), (dims, 4097))
    for dims, atoms, columns in (((96, 100, 90), 4096, True),       # 37 / 174
                                 ((512, 512, 512), 4096, True),     # 69 / 113
                                 ((1024, 1024, 8), 256, False),     # 122 / 29
                                 ((2048, 2048, 8), 1500, False)):   # 570 / 76
        assert by_columns(small, 9.0, (dims, atoms)) == columns, ("8 x 8", dims, atoms)
    # 24 problems of the sizes of the batched workload: 36 / 68
    batch = [((a, b, c), 300) for a in (48, 90, 240) for b in (60, 180) for c in (48, 72, 120, 240)]
    assert by_columns(large, 6.0, *batch)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("natoms", [3, 300])
@pytest.mark.parametrize("kind", ["diagonal", "skew"])
def test_long_columns(oracle_mod, prec, natoms, kind):
    """70 bricks along c (3 atoms: by columns, 300: by visits): density and
    forces against the oracle at the bounds of the other parity tests."""
    import torch

    from paper_1209_4506_amd import hartree as H

    print("case long columns", prec, natoms, kind, flush=True)
    dims, cell = (16, 10, 2240), np.diag([4.0, 2.5, 560.0])
    if kind == "skew":
        cell[2, 0] = -30.0
    rng = np.random.default_rng(natoms)
    pos, Z, sig = rng.uniform(0.0, 1.0, (natoms, 3)) @ cell, rng.uniform(0.5, 2.0, natoms), rng.uniform(0.4, 0.7, natoms)
    plan = H.Plan(cell, dims, precision=prec, max_atoms=natoms, max_sigma=0.7)
    R, q, w = (torch.as_tensor(x, dtype=torch.float64, device="cuda") for x in (pos, Z, sig))
    rho = plan.splat(R, q, w, subtract_background=False).double().cpu().numpy()
    ref = oracle_mod.splat(cell.reshape(9), dims, pos, Z, sig, subtract_background=False)
    assert np.abs(rho - ref).max() <= (1e-13 if prec == "fp64" else 1e-6) * np.abs(ref).max()
    g = np.cos(0.37 * np.arange(ref.size)).reshape(dims).astype(np.float64 if prec == "fp64" else np.float32)
    f = plan.splat_adjoint(R, q, w, torch.as_tensor(g, device="cuda")).cpu().numpy()
    want = oracle_mod.splat_adjoint(cell.reshape(9), pos, Z, sig, g.astype(np.float64))
    assert np.abs(f - want).max() <= (1e-10 if prec == "fp64" else 1e-5) * np.abs(want).max()
    assert plan.device_status() == 0
