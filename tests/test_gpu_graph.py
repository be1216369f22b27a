"""One-launch replay of a whole fwd+bwd step (hartree_graph_begin / end / launch).

Every replay is checked bit for bit against the same sequence run eagerly on
the same plan (the kernels and their reduction orders are identical), with
the program's own eager work and synchronisations between replays, and after
the atoms move in place (the binning is inside the captured sequence).
"""
import numpy as np
import pytest
import torch

from paper_1209_4506_amd import inputs

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def H():
    import paper_1209_4506_amd.hartree as h

    return h


class Step:
    """Preallocated buffers and the calls of one step on a (batched) plan."""

    def __init__(self, H, probs, prec, fused=False):
        dev = torch.device("cuda")
        self.fused = fused
        cells = np.stack([q.cell for q in probs])
        dims = np.array([q.dims for q in probs])
        self.counts = [q.natoms for q in probs]
        self.plan = H.Plan(cells if len(probs) > 1 else cells[0], dims if len(probs) > 1 else dims[0],
                           precision=prec, max_atoms=int(sum(self.counts)))
        p = self.plan
        self.pos = torch.tensor(np.concatenate([q.pos for q in probs]), device=dev)
        self.Z = torch.tensor(np.concatenate([q.Z for q in probs]), device=dev)
        self.sig = torch.tensor(np.concatenate([q.sigma for q in probs]), device=dev)
        c = np.concatenate([inputs.random_grid(q.dims, 40 + i).reshape(-1) for i, q in enumerate(probs)])
        dvs = np.repeat(p.dv(), [q.npoints for q in probs])
        self.gv = torch.tensor(c * dvs, device=dev).to(p.dtype).reshape(p.grid_shape()).contiguous()
        self.ge = torch.ones(p.nprob, dtype=torch.float64, device=dev)
        self.rho = p.empty_grid()
        self.V = p.empty_grid()
        self.E = torch.empty(p.nprob, dtype=torch.float64, device=dev)
        self.grho = p.empty_grid()
        self.gpos = torch.empty((self.pos.shape[0], 3), dtype=torch.float64, device=dev)
        self.token = None

    def run(self, rebind=True):
        p = self.plan
        counts = self.counts if p.batched else None
        if rebind:
            self.token = p.bind_atoms(self.pos, self.Z, self.sig, atom_counts=counts)
        p.splat_bound(self.token, out=self.rho)
        if self.fused:
            # the backward chain beside the solve's (hartree_solve_backward)
            p.solve_backward(self.rho, grad_v=self.gv, grad_e=self.ge, v=self.V, e_h=self.E, out=self.grho)
        else:
            p.solve(self.rho, v=self.V, e_h=self.E)
            p.backward(grad_v=self.gv, grad_e=self.ge, rho=self.rho, out=self.grho)
        p.splat_adjoint_bound(self.token, self.grho, out=self.gpos)

    def outputs(self):
        return [t.clone() for t in (self.rho, self.V, self.E, self.grho, self.gpos)]

    def scribble(self):
        """Eager work between replays: overwrite every output."""
        for t in (self.rho, self.V, self.grho):
            t.fill_(123.0)
        self.E.fill_(-1.0)
        self.gpos.fill_(float("nan"))


def assert_same(got, ref, what):
    names = ["rho", "V", "E_H", "grad_rho", "grad_pos"]
    for n, g, r in zip(names, got, ref):
        assert torch.equal(g, r), "%s: %s differs from the eager run" % (what, n)


def check_graph(step, rebind):
    step.run(rebind=True)
    torch.cuda.synchronize()
    assert step.plan.device_status() == 0
    ref = step.outputs()
    step.plan.capture(lambda: step.run(rebind=rebind))
    torch.cuda.synchronize()
    assert_same(step.outputs(), ref, "capture run")
    for rep in range(3):
        step.scribble()
        torch.cuda.synchronize()
        step.plan.replay()
        torch.cuda.synchronize()
        assert_same(step.outputs(), ref, "replay %d" % rep)
    return ref


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_graph_batched_replays_and_moved_atoms(H, prec):
    probs = [inputs.small_problem((30, 36, 40), 25, seed=61, L=(8.0, 8.5, 9.0)),
             inputs.small_problem((21, 16, 27), 12, seed=62, L=(7.0, 9.0, 8.0)),
             inputs.small_problem((48, 20, 35), 40, seed=63, L=(12.0, 6.0, 10.0))]
    say("case graph batched", prec, [q.dims for q in probs])
    step = Step(H, probs, prec)
    check_graph(step, rebind=True)
    # move the atoms in place: the replay re-bins them
    step.pos.add_(torch.tensor(np.random.default_rng(5).normal(0.0, 0.3, tuple(step.pos.shape)), device="cuda"))
    torch.cuda.synchronize()
    step.plan.replay()
    torch.cuda.synchronize()
    got = step.outputs()
    step.run(rebind=True)
    torch.cuda.synchronize()
    assert_same(got, step.outputs(), "replay after moving the atoms")
    assert step.plan.device_status() == 0


def test_graph_single_plan_bound_outside(H):
    p = inputs.cubic32()
    say("case graph cubic32 fp32, binding outside the graph")
    step = Step(H, [p], "fp32")
    check_graph(step, rebind=False)


def test_graph_errors(H):
    say("case graph argument errors")
    p = inputs.cubic32()
    plan = H.Plan(p.cell, p.dims, precision="fp32", max_atoms=p.natoms)
    with pytest.raises(H.HartreeError):
        plan.replay()  # nothing captured yet
    assert H.LIB.hartree_graph_begin(plan._h, None) != 0  # the default stream cannot be captured
    s = torch.cuda.Stream()
    import ctypes

    assert H.LIB.hartree_graph_end(plan._h, ctypes.c_void_p(s.cuda_stream)) != 0  # no capture open


BATCHED = [((30, 36, 40), 25, 61, (8.0, 8.5, 9.0)), ((21, 16, 27), 12, 62, (7.0, 9.0, 8.0)),
           ((48, 20, 35), 40, 63, (12.0, 6.0, 10.0))]
# compiled plan lengths <= 240 in table order (entries 0 .. 15); along c the
# entries 41, 42, 43 stand for 48, 128 and 160
SMALL_LENGTHS = [32, 48, 60, 64, 72, 90, 96, 120, 128, 150, 160, 180, 192, 200, 210, 240]


def multi_plan_config(plan, probs):
    """Every problem on its length's listed plan at the size-adapted tile
    width, no pad: each pass one multi-plan launch."""
    entry = {n: i for i, n in enumerate(SMALL_LENGTHS)}
    entry_c = {**entry, 48: 41, 128: 42, 160: 43}
    cfg = plan.get_config()
    for q, pr in enumerate(probs):
        for x in range(3):
            n = pr.dims[x]
            p, lo, target = (32, 4, 2048) if x == 2 else (64, 8, 4096 if x == 0 else 2048)
            while p > lo and p * n > target:
                p //= 2
            cfg[q, x] = ((entry_c if x == 2 else entry)[n], p.bit_length() - 1, 0)
    return cfg


BATCHED_MULTI = [((48, 60, 32), 25, 65, (8.0, 9.5, 6.0)), ((64, 48, 60), 30, 66, (10.0, 8.0, 9.0)),
                 ((32, 32, 48), 12, 67, (6.0, 6.0, 8.0))]


SKIP_GROUPED = pytest.mark.skip(reason=(
    "the capture of hartree_solve_backward on a batched plan with several launch groups per pass, when its "
    "backward chain forked side streams of its own, ended in a segmentation fault inside hipStreamEndCapture / "
    "hipGraphInstantiate with no cause found in the library; that path is switched off (such plans now run the "
    "chains in order), and this case stays off the GPU until a cause is shown"))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["single", pytest.param("batched", marks=SKIP_GROUPED), "batched_multi"])
def test_solve_backward_concurrent_chains(H, prec, kind):
    """hartree_solve_backward runs the backward chain on its own stream and
    spectrum beside the solve's: V, E_H, grad_rho (and the forces after it)
    are identical bit for bit to hartree_solve then hartree_backward, eagerly
    and in every graph replay (the two chains as parallel branches)."""
    if kind == "single":
        probs = [inputs.small_problem((48, 40, 36), 30, seed=64, L=(9.0, 8.0, 7.5))]
    elif kind == "batched_multi":
        # lengths of the multi-plan list only (FP32): every pass one launch
        # group, so the two chains run side by side (FP64: in order)
        probs = [inputs.small_problem(d, n, seed=sd, L=L) for d, n, sd, L in BATCHED_MULTI]
    else:
        probs = [inputs.small_problem(d, n, seed=sd, L=L) for d, n, sd, L in BATCHED]
    say("case solve_backward", kind, prec, [q.dims for q in probs])
    ref_step = Step(H, probs, prec)
    step = Step(H, probs, prec, fused=True)
    if kind == "batched_multi" and prec == "fp32":
        for st in (ref_step, step):
            st.plan.set_config(multi_plan_config(st.plan, probs))
    ref_step.run()
    torch.cuda.synchronize()
    ref = ref_step.outputs()
    step.run()
    torch.cuda.synchronize()
    assert step.plan.device_status() == 0
    assert_same(step.outputs(), ref, "eager solve_backward")
    step.plan.capture(lambda: step.run(rebind=True))
    torch.cuda.synchronize()
    for rep in range(3):
        step.scribble()
        torch.cuda.synchronize()
        step.plan.replay()
        torch.cuda.synchronize()
        assert_same(step.outputs(), ref, "solve_backward replay %d" % rep)


# (hartree_solve_backward records the chains of such plans in order too)
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_captured_groups_in_order(H, prec):
    """A batched plan whose passes have several launch groups: under capture
    the groups are recorded in order and hartree_solve_backward's chains as two
    branches; every replay equals the eager solve and backward bit for bit."""
    probs = [inputs.small_problem(d, n, seed=sd, L=L) for d, n, sd, L in BATCHED]
    say("case captured groups", prec, [q.dims for q in probs])
    ref_step, step = Step(H, probs, prec), Step(H, probs, prec, fused=True)
    ref_step.run()
    torch.cuda.synchronize()
    ref = ref_step.outputs()
    step.plan.capture(lambda: step.run(rebind=True))
    torch.cuda.synchronize()
    for rep in range(3):
        step.scribble()
        torch.cuda.synchronize()
        step.plan.replay()
        torch.cuda.synchronize()
        assert_same(step.outputs(), ref, "replay %d" % rep)


def test_solve_backward_zero_gradient_and_errors(H):
    """No upstream gradient: grad_rho is zero and V, E_H are the solve's;
    v aliasing grad_v or grad_rho is rejected."""
    say("case solve_backward zero gradient and argument errors")
    p = inputs.cubic32()
    plan = H.Plan(p.cell, p.dims, precision="fp32", max_atoms=p.natoms)
    rho = torch.tensor(inputs.random_grid(p.dims, 7), dtype=torch.float32, device="cuda").contiguous()
    V, E = plan.solve(rho)
    V2, E2, G = plan.solve_backward(rho)
    torch.cuda.synchronize()
    assert torch.equal(V, V2) and torch.equal(E, E2)
    assert torch.count_nonzero(G).item() == 0
    gv = torch.ones_like(rho)
    with pytest.raises(H.HartreeError):
        plan.solve_backward(rho, grad_v=gv, v=gv)
    out = plan.empty_grid()
    with pytest.raises(H.HartreeError):
        plan.solve_backward(rho, grad_v=gv, v=out, out=out)


@pytest.mark.parametrize("which", ["grad_v only", "grad_e only"])
def test_solve_backward_partial_gradients(H, which):
    """One upstream gradient only, on the concurrent path (a small single
    plan): V, E_H and grad_rho equal the two calls in order bit for bit."""
    say("case solve_backward", which)
    p = inputs.cubic32()
    plan = H.Plan(p.cell, p.dims, precision="fp32", max_atoms=p.natoms)
    rho = torch.tensor(inputs.random_grid(p.dims, 8), dtype=torch.float32, device="cuda").contiguous()
    gv = torch.tensor(inputs.random_grid(p.dims, 9), dtype=torch.float32, device="cuda").contiguous()
    ge = torch.tensor([0.7], dtype=torch.float64, device="cuda")
    kw = {"grad_v": gv} if which == "grad_v only" else {"grad_e": ge}
    V, E = plan.solve(rho)
    G = plan.backward(rho=rho, **kw)
    V2, E2, G2 = plan.solve_backward(rho, **kw)
    torch.cuda.synchronize()
    assert torch.equal(V, V2) and torch.equal(E, E2)
    assert torch.equal(G, G2)
    assert torch.count_nonzero(G2).item() > 0
