"""The tiles that plans are created with."""
import numpy as np
import pytest

from paper_1209_4506_amd import inputs

# FP32 batches (grids): axes whose lengths all have a plan of the multi-plan list
# and ones where some have not, lengths whose shared kernels round otherwise
# than their own (32 and 48 along a, 32 along b, 64 and 72 along c)
BATCHES = [[(48, 48, 48)] * 3, [(32, 32, 32)] * 2, [(240, 200, 64), (210, 200, 210), (200, 240, 64)],
           [(72, 180, 180), (180, 72, 72), (64, 64, 180)], [(32, 48, 32), (48, 64, 60), (48, 64, 48)],
           [(64, 60, 72), (60, 60, 64)], [(27, 45, 72), (75, 32, 180)], [(210, 240, 200), (64, 64, 210), (64, 240, 200)],
           [(72, 150, 60), (240, 180, 72), (150, 60, 120), (90, 90, 240)]]


def default_widths(dims, precision):
    """Pencils per tile along a, b and c of a plan as created (host only)."""
    import ctypes

    from paper_1209_4506_amd.hartree import LIB

    d, i32 = ctypes.c_double, ctypes.c_int32
    h, cfg = ctypes.c_void_p(), (i32 * 9)()
    assert LIB.hartree_plan_create(ctypes.byref(h), (d * 9)(9, 0, 0, 0, 9, 0, 0, 0, 9), (i32 * 3)(*dims), precision, None) == 0
    assert LIB.hartree_plan_get_config(h, cfg) == 0
    LIB.hartree_plan_destroy(h)
    return [1 << cfg[3 * x + 1] for x in range(3)]


def test_short_lengths_take_wide_tiles():
    """Widths that measured faster by an eighth and more than half and a quarter
    of them, or than twice (short strided lengths, many and few tiles)."""
    fp64, fp32 = 0, 1
    for prec, axis, dims, widths in ((fp32, 0, (16, 64, 2048), {64}), (fp32, 1, (64, 16, 2048), {32, 64}),
                                     (fp32, 1, (16, 16, 4096), {32, 64}), (fp32, 0, (8, 360, 360), {64}),
                                     (fp64, 0, (4, 360, 360), {64}), (fp64, 0, (16, 16, 4096), {32, 64}),
                                     (fp64, 0, (144, 360, 360), {16, 32}), (fp64, 1, (360, 9, 360), {32, 64}),
                                     (fp32, 0, (16, 10, 12), {1, 2, 4, 8, 16, 32}), (fp32, 0, (32, 360, 360), {64}),
                                     (fp32, 0, (64, 64, 2048), {32, 64}), (fp32, 1, (64, 32, 2048), {32, 64}),
                                     (fp32, 1, (400, 48, 20), {8, 16}), (fp64, 0, (64, 100, 300), {32}),
                                     (fp64, 0, (64, 400, 20), {8, 16, 32}), (fp64, 0, (72, 360, 360), {32}),
                                     (fp64, 0, (160, 16, 4096), {16}), (fp64, 0, (60, 192, 192), {8}),
                                     (fp64, 0, (96, 192, 192), {8}), (fp64, 2, (12, 10, 200), {1, 2, 4}),
                                     (fp64, 2, (192, 192, 200), {4, 8}), (fp32, 0, (135, 168, 189), {16}),
                                     (fp32, 0, (35, 192, 192), {16, 32}), (fp32, 1, (2000, 24, 20), {8, 16})):
        assert default_widths(dims, prec)[axis] in widths, (prec, axis, dims, default_widths(dims, prec))


@pytest.mark.gpu
@pytest.mark.parametrize("dims", BATCHES)
def test_batches_as_created(dims):
    """An FP32 batch as created gives the values of the widest tiles along a and
    b and four pencils along c, bit for bit (E_H but for the order of its sum
    over tiles)."""
    import torch

    from paper_1209_4506_amd import hartree as H

    print("case batch as created", dims, flush=True)
    cells = np.stack([np.array([[9.0 + q, 0.0, 0.0], [1.0, 10.0, 0.0], [0.0, -2.0, 11.0]]) for q in range(len(dims))])
    plan = H.Plan(cells, np.array(dims), precision="fp32", max_atoms=1)
    rho = torch.as_tensor(np.concatenate([inputs.random_grid(d, 80 + q).reshape(-1) for q, d in enumerate(dims)]).astype(np.float32),
                          device="cuda")
    ge = torch.full((len(dims),), 0.3, dtype=torch.float64, device="cuda")
    out = []
    for wide in (False, True):
        if wide:
            cfg = plan.get_config()
            for q in range(len(dims)):
                for x in range(3):
                    for lp in range(2 if x == 2 else 6, -1, -1):
                        one = H.Plan(cells[q], dims[q], precision="fp32", max_atoms=1, bind=False)
                        c = one.get_config()
                        c[0, x, 1:] = (lp, 0)
                        try:
                            one.set_config(c)
                        except H.HartreeError:
                            continue
                        cfg[q, x, 1:] = (lp, 0)
                        break
            plan.set_config(cfg)
        V, E = plan.solve(rho)
        G = plan.backward(grad_v=rho, grad_e=ge, rho=rho)
        torch.cuda.synchronize()
        out.append((V.clone(), G.clone(), E.clone()))
    (V, G, E), (V2, G2, E2) = out
    assert torch.equal(V, V2) and torch.equal(G, G2)
    assert torch.allclose(E, E2, rtol=1e-13, atol=0.0)
