"""The block kernel (several steps of a tile per launch, its state in
registers) against the marching kernel at one step per pass: the same bits in
the state (padding included), the readout and the captures, for every shape at
its smallest, a middle and its largest number of steps per pass."""
import os

import pytest
import torch

from gpu_common import banner, captured_moments, random_case
from test_gpu_gamma import gamma_field

pytestmark = pytest.mark.gpu

# lattices smaller than a tile in one or both directions (periodic images
# inside a tile), ragged ones, and whole multiples of no tile
LATTICES = [(1, 1), (5, 3), (23, 37), (130, 97), (6, 300), (300, 6), (70, 150)]
# rows of a tile per shape (rows per wavefront x wavefronts)
SHAPES = {("fp32", 1.0): (32, 48, 80), ("fp32", 0.9): (32, 24), ("fp16s", 1.0): (32, 48, 80), ("fp16s", 0.9): (32, 24),
           ("fp64", 1.0): (32, 48), ("fp64", 0.9): (16, 24)}
CASES = [(prec, tau, shape) for (prec, tau), rows in SHAPES.items() for shape in range(len(rows))]


def run(prec, ny, nx, field, steps, env, p):
    from paper_1810_07642_amd import Sim
    os.environ.update(env)
    try:
        sim = Sim(nx, ny, prec, gamma_field=field == "gamma", **p)
        h0, th = random_case(ny, nx, 61)
        sim.init(h0, None if field == "uniform" else th, gamma_field(ny, nx, 62) if field == "gamma" else None)
    finally:
        for k in env:
            del os.environ[k]
    sim.step(steps)
    cap = torch.zeros(5 * sim.capture_bytes(), dtype=torch.uint8, device=sim.device)
    mid = tuple(t.cpu() for t in sim.read())
    sim.step_capture(5, cap)
    sim.check()
    return (sim.state_save().cpu(), cap.cpu()) + mid + tuple(t.cpu() for t in sim.read()), sim.steps_per_pass


@pytest.mark.parametrize("g", [1e-3, 0.0])
@pytest.mark.parametrize("prec,tau,shape", CASES)
def test_block_kernel_equals_marching_kernel_bitwise(prec, tau, shape, g):
    rows = SHAPES[(prec, tau)][shape]
    most = min((rows - 2) // 6, 9)  # two output rows, eight output columns of 64
    for (ny, nx) in LATTICES:
        for n, m in ((9, 3), (3, 9)):
            p = dict(tau=tau, gamma=0.01, g=g, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, n=n, m=m, href=0.4)
            for field in ("theta", "uniform", "gamma") if n == 9 else ("theta",):
                banner(f"block kernel: {prec} tau={tau} shape {shape} g={g} {ny}x{nx} {field} n={n}")
                ref, _ = run(prec, ny, nx, field, 11, {"TFLBM_FUSE": "1"}, p)
                for ns in sorted({1, 2, most}):
                    got, spp = run(prec, ny, nx, field, 11,
                                   {"TFLBM_BLOCK": str(ns), "TFLBM_BLOCK_SHAPE": str(shape)}, p)
                    assert spp == ns
                    for a, b in zip(got, ref):
                        assert torch.equal(a, b), (ny, nx, field, ns)


def test_block_kernel_flags_bad_heights():
    """h <= 0 and NaN at one site are reported whichever tile holds it."""
    from paper_1810_07642_amd import Sim
    from paper_1810_07642_amd._lib import TFLBM_ENONFINITE, TFLBM_OK
    os.environ["TFLBM_BLOCK"] = "3"
    try:
        for bad in (-0.1, float("nan")):
            for at in ((0, 0), (40, 99), (69, 149)):
                sim = Sim(150, 70, "fp32", hstar=0.1)
                h0 = torch.full((70, 150), 0.3, dtype=torch.float64)
                sim.init(h0)
                sim.step(3)
                assert sim.status() == TFLBM_OK
                # a bad site that enters through a checkpoint, not through init's own check
                h0[at] = bad
                other = Sim(150, 70, "fp32", hstar=0.1).init(h0)
                sim.state_load(other.state_save(), 0)
                sim.step(3)
                assert sim.status() == TFLBM_ENONFINITE, (bad, at)
    finally:
        del os.environ["TFLBM_BLOCK"]


@pytest.mark.parametrize("prec,tau", list(SHAPES))
def test_short_calls_equal_marching_kernel_bitwise(prec, tau):
    """Calls of a few steps, which the default plan gives to one kernel or the
    other, in a row on one handle."""
    for (ny, nx) in ((67, 90), (137, 553), (256, 256), (320, 704), (151, 1001)):
        p = dict(tau=tau, gamma=0.01, g=0.0, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, n=9, m=3, href=0.4)
        for steps in (1, 2, 3, 4):
            banner(f"short calls: {prec} tau={tau} {ny}x{nx} {steps} steps")
            ref, _ = run(prec, ny, nx, "theta", steps, {"TFLBM_BLOCK": "0"}, p)
            got, _ = run(prec, ny, nx, "theta", steps, {}, p)
            for a, b in zip(got, ref):
                assert torch.equal(a, b), (ny, nx, steps)


@pytest.mark.parametrize("prec,nx,ny", [("fp64", 480, 1301), ("fp32", 840, 1070)])
def test_calls_that_leave_the_plan_equal_single_steps_bitwise(prec, nx, ny):
    """Lattices whose calls go to the block kernel, the passes of moments or the
    marching kernel by their length, in a row on one handle."""
    p = dict(tau=1.0, gamma=0.01, g=0.0, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, n=9, m=3, href=0.4)
    for steps in (4, 7, 24):
        banner(f"calls that leave the plan: {prec} {ny}x{nx} {steps} steps")
        ref, _ = run(prec, ny, nx, "theta", steps, {"TFLBM_FUSE": "1"}, p)
        got, _ = run(prec, ny, nx, "theta", steps, {}, p)
        for a, b in zip(got, ref):
            assert torch.equal(a, b), steps


def test_odd_fp16s_calls_in_a_callers_graph():
    """FP16S of odd width: a caller's own graph of three steps ends on the
    buffer it started from, as with the marching kernel's two passes, so that
    each replay advances the state like the eager call."""
    p = dict(tau=0.9, gamma=0.01, g=1e-3, hstar=0.1, delta=1.0, ax=1e-5, href=0.4)
    from paper_1810_07642_amd import Sim
    h0, th = random_case(2622, 279, 63)
    a, b = (Sim(279, 2622, "fp16s", **p).init(h0, th) for _ in range(2))
    a.step(3)
    b.step(3)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            a.step(3)
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
        b.step(3)
        torch.cuda.synchronize()
        assert torch.equal(a.state_save(), b.state_save())
    a.check()


@pytest.mark.parametrize("block", [True, False])
def test_fp32_calls_of_two_steps_in_a_callers_graph(block):
    """2560 strip rows: two steps are two passes, of either kernel, so that a
    caller's own graph of them ends on the buffer it started from."""
    from paper_1810_07642_amd import Sim
    p = dict(tau=1.0, gamma=0.01, hstar=0.1, delta=1.0, ax=1e-5, href=0.4, **({} if block else dict(n=10, m=4)))
    h0, th = random_case(512, 512, 64)
    a, b = (Sim(512, 512, "fp32", **p).init(h0, th) for _ in range(2))
    a.step(2)
    b.step(2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            a.step(2)
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
        b.step(2)
        torch.cuda.synchronize()
        assert torch.equal(a.state_save(), b.state_save())
    a.check()


@pytest.mark.parametrize("prec,tau,shape", CASES)
def test_captures_equal_marching_kernel_bitwise(prec, tau, shape):
    """The captured moments, on buffers that held something else; whole
    records (108, 46, 116 columns) and one column less."""
    from paper_1810_07642_amd import Sim
    p = dict(tau=tau, gamma=0.01, g=1e-3, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, href=0.4)
    for (ny, nx) in ((23, 37), (40, 216), (40, 232), (33, 92), (50, 231), (70, 340)):
        banner(f"captures by the block kernel: {prec} tau={tau} shape {shape} {ny}x{nx}")
        h0, th = random_case(ny, nx, 65)

        def capture(env):
            os.environ.update(env)
            try:
                sim = Sim(nx, ny, prec, **p).init(h0, th)
            finally:
                for k in env:
                    del os.environ[k]
            cap = torch.full((5 * sim.capture_bytes(),), 0xA5, dtype=torch.uint8, device=sim.device)
            sim.step_capture(5, cap)
            sim.check()
            return captured_moments(cap, prec, ny, nx, 5).cpu()

        ref = capture({"TFLBM_FUSE": "1"})
        assert torch.equal(capture({"TFLBM_BLOCK": "2", "TFLBM_BLOCK_SHAPE": str(shape)}), ref), (ny, nx)
