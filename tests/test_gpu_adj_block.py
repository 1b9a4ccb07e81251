"""The reverse block kernel (several reverse steps of a tile per launch)
against the marching kernel at one step per pass: the same bits in both
gradients, for every shape at its smallest, a middle and its largest number of
steps per pass."""
import os

import pytest
import torch

from gpu_common import banner, random_case

pytestmark = pytest.mark.gpu

# smaller than a tile in one or both directions, ragged, one strip and one column more
LATTICES = [(1, 1), (5, 3), (23, 37), (6, 300), (300, 6), (70, 150), (97, 108), (54, 55)]
# rows of a tile per shape (rows per wavefront x wavefronts); FP16S adjoints are FP32
SHAPES = {("fp32", 1.0): (32, 36), ("fp16s", 1.0): (32, 36), ("fp32", 0.9): (16, 32), ("fp64", 1.0): (12, 16),
          ("fp64", 0.9): (12, 16)}
CASES = [(prec, tau, shape) for (prec, tau), rows in SHAPES.items() for shape in range(len(rows))]


@pytest.mark.parametrize("prec,tau,shape", CASES)
def test_reverse_block_kernel_equals_marching_kernel_bitwise(prec, tau, shape):
    from paper_1810_07642_amd import Sim
    rows = SHAPES[(prec, tau)][shape]
    most = min((rows - 2) // 6, 9)
    for (ny, nx) in LATTICES:
        for n, m in ((9, 3), (3, 9)):
            p = dict(tau=tau, gamma=0.01, g=1e-3, hstar=0.1, delta=1.0, ax=1e-5, ay=-1e-5, n=n, m=m, href=0.4)
            h0, th = random_case(ny, nx, 81)
            grad_h = torch.randn((ny, nx), generator=torch.Generator().manual_seed(82), dtype=torch.float64)
            for field in (True, False) if n == 9 else (True,):
                banner(f"reverse block kernel: {prec} tau={tau} shape {shape} {ny}x{nx} field={field} n={n}")

                def grads(env, segments):
                    os.environ.update(env)
                    try:
                        sim = Sim(nx, ny, prec, **p).init(h0, th if field else None)
                    finally:
                        for k in env:
                            del os.environ[k]
                    total = sum(segments)
                    cb = sim.capture_bytes()
                    cap = torch.empty(total * cb, dtype=torch.uint8, device=sim.device)
                    sim.step_capture(total, cap)
                    adj = torch.empty(sim.adj_bytes(), dtype=torch.uint8, device=sim.device)
                    sim.adj_seed(adj, grad_h)
                    for k in segments:
                        total -= k
                        sim.adj_steps(adj, cap[total * cb:], k)
                    return [t.cpu() for t in sim.adj_finish(adj)]

                ref = grads({"TFLBM_ADJ_FUSE": "1"}, (12,))
                assert all(bool(torch.isfinite(t).all()) for t in ref)
                for ns in sorted({1, 2, most}):
                    env = {"TFLBM_ADJ_BLOCK": str(ns), "TFLBM_ADJ_BLOCK_SHAPE": str(shape)}
                    for segments in ((12,), (7, 1, 4)):
                        for a, b in zip(grads(env, segments), ref):
                            assert torch.equal(a, b), (ny, nx, field, ns, segments)
