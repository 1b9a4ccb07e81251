"""Which kernels a call launches, and in which buffer it leaves the state: the
host side of the library on the CPU (launch_host.py)."""
import pytest

import launch_host as lh

pytestmark = pytest.mark.skipif(lh.compiler() is None, reason="needs a C compiler")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return lh.build_driver(tmp_path_factory.mktemp("launch"))


def kernels(exe, case, call):
    """The mangled names of the kernels that a call on the lattice launches."""
    res = lh.drive(exe, [lh.sim(**case), "capture 1", "seed", call])
    assert all(r.rc == 0 for r in res)
    return [l.kernel for l in res[3].launches]


@pytest.mark.parametrize("case,steps,block", [
    # measured, us per step marching / block: 15.9 / 20.6, 13.7 / 15.2, 8.6 / 9.6, 11.0 / 9.0, 6.9 / 3.7
    (dict(nx=675, ny=1181, prec="fp32", tau=0.9), 8, False), (dict(nx=509, ny=1530, prec="fp32"), 8, False),
    (dict(nx=606, ny=508, prec="fp32"), 4, False),
    (dict(nx=399, ny=1186, prec="fp32"), 24, True), (dict(nx=297, ny=315, prec="fp32"), 8, True)])
def test_reverse_calls_take_the_faster_kernel(exe, case, steps, block):
    names = kernels(exe, case, f"adj {steps}")
    assert all(("adj_block_kernel" in n) == block for n in names), names
