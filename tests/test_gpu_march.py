"""Passes that hand over moments (omega = 1) against the marching kernel at one
step per pass, which stores populations after every step: the same bits in the
state (padding included), the readout and the captures, for calls that split
into every kind of pass."""
import os

import pytest
import torch

from gpu_common import banner, captured_moments, random_case

pytestmark = pytest.mark.gpu

# ragged, degenerate and narrower than a strip; whole records (108 FP32, 46
# FP64 columns: the loop for aligned strips) and one column more
LATTICES = [(1, 1), (7, 3), (23, 37), (130, 97), (6, 300), (40, 216), (40, 217), (33, 92), (70, 150)]


def make(prec, ny, nx, field, env, p):
    from paper_1810_07642_amd import Sim
    os.environ.update(env)
    try:
        sim = Sim(nx, ny, prec, **p)
        h0, th = random_case(ny, nx, 71)
        return sim.init(h0, th if field else None)
    finally:
        for k in env:
            del os.environ[k]


def outcome(sim, steps):
    out = []
    for n in steps:
        sim.step(n)
        out += [sim.state_save().cpu()] + [t.cpu() for t in sim.read()]
    cap = torch.zeros(9 * sim.capture_bytes(), dtype=torch.uint8, device=sim.device)
    sim.step_capture(9, cap)
    sim.check()
    return out + [cap.cpu(), sim.state_save().cpu()]


@pytest.mark.parametrize("g", [1e-3, 0.0])
@pytest.mark.parametrize("field", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_passes_of_moments_equal_single_steps_bitwise(prec, field, g):
    p = dict(tau=1.0, gamma=0.01, g=g, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, href=0.4)
    steps = (4, 5, 10, 7, 23)
    for (ny, nx) in LATTICES:
        banner(f"passes of moments: {prec} {ny}x{nx} field={field} g={g}")
        ref = outcome(make(prec, ny, nx, field, {"TFLBM_FUSE": "1"}, p), steps)
        for ns, rows in (("2", None), ("3", None), ("3", "1"), ("2", "7")):
            env = {"TFLBM_BLOCK": "0", "TFLBM_MARCH": ns}
            if rows:
                env["TFLBM_MARCH_ROWS"] = rows
            sim = make(prec, ny, nx, field, env, p)
            assert sim.steps_per_pass == 3
            for a, b in zip(outcome(sim, steps), ref):
                assert torch.equal(a, b), (ny, nx, ns, rows)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_passes_of_moments_in_a_callers_graph(prec):
    """A caller's own graph of 20 steps ends on the buffer it started from,
    as with one step per pass, so that each replay advances the state like the
    eager call."""
    p = dict(tau=1.0, gamma=0.01, g=1e-3, hstar=0.1, delta=1.0, ax=1e-5)
    env = {"TFLBM_BLOCK": "0", "TFLBM_MARCH": "3"}
    a, b = (make(prec, 70, 150, True, env, p) for _ in range(2))
    a.step(20)
    b.step(20)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            a.step(20)
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
        b.step(20)
        torch.cuda.synchronize()
        assert torch.equal(a.state_save(), b.state_save())
    a.check()


# steps of a call with captures: 10 and 23 split into passes of moments, with
# middle passes of two and of three steps and either kind of last pass; 9 does not
CAPTURE_STEPS = (10, 23, 9)
# three records and more (108 FP32, 46 FP64 columns): whole ones, and one column
# more or less; narrower than a strip
CAPTURE_LATTICES = [(40, 330), (33, 432), (20, 433), (50, 691), (70, 150), (23, 37)]


@pytest.mark.parametrize("g", [1e-3, 0.0])
@pytest.mark.parametrize("field", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_captures_of_passes_of_moments_equal_single_steps_bitwise(prec, field, g):
    """The captured moments, on buffers that held something else."""
    p = dict(tau=1.0, gamma=0.01, g=g, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, href=0.4)

    def captures(sim):
        out = []
        for n in CAPTURE_STEPS:
            cap = torch.full((n * sim.capture_bytes(),), 0xA5, dtype=torch.uint8, device=sim.device)
            sim.step_capture(n, cap)
            out += [captured_moments(cap, prec, sim.ny, sim.nx, n).cpu(), sim.state_save().cpu()]
        sim.check()
        return out

    for (ny, nx) in CAPTURE_LATTICES:
        banner(f"captures of passes of moments: {prec} {ny}x{nx} field={field} g={g}")
        ref = captures(make(prec, ny, nx, field, {"TFLBM_FUSE": "1"}, p))
        for ns, rows in (("2", None), ("3", None), ("3", "9"), ("2", "7")):
            env = {"TFLBM_BLOCK": "0", "TFLBM_MARCH": ns}
            if rows:
                env["TFLBM_MARCH_ROWS"] = rows
            for a, b in zip(captures(make(prec, ny, nx, field, env, p)), ref):
                assert torch.equal(a, b), (ny, nx, ns, rows)


@pytest.mark.parametrize("field", [True, False])
def test_fp64_two_step_passes_by_the_general_stages_bitwise(field):
    """FP64 at tau = 1 on a lattice of three steps per pass: a call of two
    steps, and the last pass of 5 and 8 without passes of moments, run the general
    stages' two-step kernel.  The same bits as single steps, and as the general
    stages throughout."""
    p = dict(tau=1.0, gamma=0.01, g=1e-3, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5)
    for steps, env in ((2, {"TFLBM_BLOCK": "0"}), (5, {"TFLBM_BLOCK": "0", "TFLBM_MARCH": "0"}),
                       (8, {"TFLBM_BLOCK": "0", "TFLBM_MARCH": "0"})):
        banner(f"two-step passes by the general stages: field={field} {steps} steps")
        got = [state(make("fp64", 1024, 1024, field, e, p), steps)
               for e in (env, {"TFLBM_FUSE": "1"}, {"TFLBM_OMEGA1": "0"})]
        for other in got[1:]:
            for a, b in zip(got[0], other):
                assert torch.equal(a, b), steps


def state(sim, steps):
    sim.step(steps)
    sim.check()
    return [sim.state_save().cpu()] + [t.cpu() for t in sim.read()]
