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


@pytest.mark.parametrize("case,call,block", [
    # measured, us per step marching / block
    (dict(nx=744, ny=922, prec="fp32"), "capture 2", False),              # 13.0 / 13.6
    (dict(nx=744, ny=922, prec="fp32"), "step 24", True),                 # 10.6 / 6.8
    (dict(nx=1165, ny=1007, prec="fp32"), "step 4", False),               # 15.9 / 18.6
    (dict(nx=784, ny=597, prec="fp64"), "step 2", False),                 # 13.0 / 12.9
    (dict(nx=784, ny=597, prec="fp64"), "step 7", True),                  # odd: 1 / 0.7
    (dict(nx=723, ny=817, prec="fp64"), "step 4", False),                 # 13.3 / 15.2
    (dict(nx=1232, ny=911, prec="fp32", tau=0.9), "capture 4", False),    # 19.1 / 25.0
    (dict(nx=1232, ny=911, prec="fp32", tau=0.9), "step 4", True),        # 17.9 / 16.4
    (dict(nx=1157, ny=327, prec="fp32", tau=0.9), "capture 4", True),     # 12.1 / 9.2
    (dict(nx=568, ny=1446, prec="fp16s"), "capture 2", False),            # 13.3 / 14.0
    (dict(nx=161, ny=1164, prec="fp32", tau=0.9), "step 2", True),        # 11.4 / 7.0, two passes
    (dict(nx=421, ny=590, prec="fp32", tau=0.9), "capture 3", True),      # 11.7 / 7.5
    (dict(nx=128, ny=128, prec="fp32"), "capture 3", True),
    (dict(nx=128, ny=128, prec="fp32"), "step 2", False)])
def test_forward_calls_take_the_faster_kernel(exe, case, call, block):
    names = kernels(exe, case, call)
    assert all(("12block_kernel" in n) == block for n in names), names


def test_calls_that_leave_a_block_plan_launch_whole_grids(exe):
    """Passes of moments on a handle with a block plan, which serves its longer calls."""
    seen = 0
    for case in (dict(nx=480, ny=1301, prec="fp64"), dict(nx=840, ny=1070, prec="fp32")):
        cmd = [lh.sim(**case)] + [f"{op} {n}" for n in range(1, 24) for op in ("step", "capture")]
        res = lh.drive(exe, cmd)
        assert all(l.grid > 0 for r in res for l in r.launches)
        assert any("12block_kernel" in l.kernel for r in res for l in r.launches)
        seen += sum("march_kernel" in l.kernel for r in res for l in r.launches)
    assert seen > 0


NO_BLOCK = ["env TFLBM_BLOCK 0", "env TFLBM_MARCH 0", "env TFLBM_ADJ_BLOCK 0"]
DEFAULT = ["env TFLBM_BLOCK", "env TFLBM_MARCH", "env TFLBM_ADJ_BLOCK"]


def ends(exe, case, env, counts):
    """The buffers that calls of `counts` steps, captures and reverse steps end on."""
    cmd, at = list(env), []
    for n in counts:
        calls = [[f"step {n}", "read"], [f"capture {n}", "read"]]
        if case.get("field") != "gamma":
            calls.append(["capture 1", "seed", f"adj {n}", "finish"])
        for c in calls:
            cmd += [lh.sim(**case)] + c
            at.append(len(cmd) - 1)
    res = lh.drive(exe, cmd)
    assert all(r.rc == 0 for r in res)
    return [res[i].launches[0].src for i in at]


# FP16S of odd width (one step per pass models best on the first three), and
# lattices of every form that the block kernels, the passes of moments and the
# marching kernels step
PARITY = [dict(nx=279, ny=2622, prec="fp16s", tau=0.9), dict(nx=357, ny=2623, prec="fp16s", tau=0.9),
          dict(nx=277, ny=2676, prec="fp16s", tau=0.9), dict(nx=901, ny=641, prec="fp16s"),
          dict(nx=450, ny=450, prec="fp64", tau=0.9), dict(nx=64, ny=64, prec="fp64"),
          dict(nx=1024, ny=1024, prec="fp64"), dict(nx=512, ny=512, prec="fp32"),
          dict(nx=901, ny=641, prec="fp32", tau=1.2, field="gamma"), dict(nx=2048, ny=2048, prec="fp32"),
          dict(nx=480, ny=1301, prec="fp64"), dict(nx=840, ny=1070, prec="fp32"),
          dict(nx=512, ny=512, prec="fp32", n=10, m=4), dict(nx=4096, ny=4096, prec="fp64")]


@pytest.mark.parametrize("case", PARITY, ids=lambda c: "_".join(str(v) for v in c.values()))
def test_calls_end_on_the_marching_kernels_buffer(exe, case):
    """A caller's own graph of a call can be replayed where the call ends on
    the buffer it started from: every plan ends on the marching kernel's."""
    counts = range(1, 13)
    assert ends(exe, case, DEFAULT, counts) == ends(exe, case, NO_BLOCK, counts)


@pytest.mark.parametrize("case", [dict(nx=450, ny=450, prec="fp64", tau=0.9), dict(nx=500, ny=500, prec="fp64", tau=0.9),
                                  dict(nx=138, ny=1335, prec="fp64", tau=0.9), dict(nx=212, ny=1089, prec="fp16s", tau=0.9),
                                  dict(nx=1359, ny=228, prec="fp16s", tau=0.9)],
                         ids=lambda c: "_".join(str(v) for v in c.values()))
def test_one_step_per_pass_drops_no_block_plan(exe, case):
    """Where a pass of one step models best, the block kernel still takes the
    best plan of several steps that beats the marching kernel."""
    res = lh.drive(exe, [lh.sim(**case), "spp", "step 12"])
    assert res[1].rc >= 2
    assert all("block_kernel" in l.kernel for l in res[2].launches) and len(res[2].launches) <= 6


def test_one_step_per_pass_drops_no_reverse_block_plan(exe):
    for case in (dict(nx=64, ny=1007, prec="fp64"), dict(nx=434, ny=925, prec="fp32"), dict(nx=804, ny=515, prec="fp32")):
        res = lh.drive(exe, [lh.sim(**case), "capture 12", "seed", "adj 12"])
        assert all("adj_block_kernel" in l.kernel for l in res[3].launches) and len(res[3].launches) <= 6, case


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_passes_of_moments_stay_off_small_lattices(exe, prec):
    """Exponents that the block kernel does not serve, at tau = 1: lattices
    whose tiles are a chain of rows run the passes of the plan without moments."""
    def names(nx, ny, env):
        res = lh.drive(exe, list(env) + [lh.sim(nx, ny, prec, n=10, m=4), "step 10", "capture 16", "spp"])
        return [l.kernel for r in res for l in r.launches], res[-1].rc
    for nx, ny in ((64, 64), (128, 128), (256, 256), (90, 2500), (900, 200)):
        plain, spp = names(nx, ny, NO_BLOCK)
        got, got_spp = names(nx, ny, DEFAULT)
        assert got == plain and got_spp == spp and not any("march_kernel" in n for n in got), (nx, ny)
    assert any("march_kernel" in n for n in names(1024, 1024, DEFAULT)[0])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_fused_passes_begin_at_a_lattice_size_of_their_own(exe, prec):
    """The steps per pass, and with them the buffer a call ends on, do not
    change with the registers of the one-step kernel (its resident workgroups)."""
    for occupancy in (8, 12, 16):
        for rows, spp in ((2560, 1), (3072, 1), (3073, 2)):
            res = lh.drive(exe, NO_BLOCK + [f"occupancy {occupancy}", lh.sim(40, rows, prec, tau=0.9), "spp", "step 2"])
            assert res[-2].rc == spp and len(res[-1].launches) == 2 // spp, (occupancy, rows)


ESTATE, EHIP = -5, -3
READERS = ["read", "mass", "mass_noalloc", "terms", "save", "step 1", "capture 1"]


@pytest.mark.parametrize("case", [dict(nx=512, ny=512, prec="fp32"), dict(nx=128, ny=128, prec="fp16s"),
                                  dict(nx=1024, ny=1024, prec="fp64"), dict(nx=4096, ny=4096, prec="fp32")],
                         ids=lambda c: "_".join(str(v) for v in c.values()))
@pytest.mark.parametrize("call", ["step 20", "capture 20"])
def test_state_is_lost_where_a_launch_fails_between_passes_of_moments(exe, case, call):
    """The current buffer holds moments then: no call takes them for
    populations, until a new state comes."""
    first = lh.sim(**case)
    cmd = [first, "fail 1", call] + READERS + ["check", "load", "read", "step 20", "read"]
    rc = [r.rc for r in lh.drive(exe, cmd)]
    assert rc[2] == EHIP and rc[3:3 + len(READERS)] == [ESTATE] * len(READERS)
    assert rc[3 + len(READERS):] == [0] * 5
    # after a failing first launch the state is the one before the call; a new init brings one
    assert [r.rc for r in lh.drive(exe, [first, "fail 0", call] + READERS)] == [0, 0, EHIP] + [0] * len(READERS)
    assert [r.rc for r in lh.drive(exe, [first, "fail 1", call, "init", "read"])] == [0, 0, EHIP, 0, 0]


def test_state_stays_where_passes_hand_over_populations(exe):
    for case in (dict(nx=512, ny=512, prec="fp32", tau=0.9), dict(nx=1024, ny=1024, prec="fp64", tau=0.9)):
        rc = [r.rc for r in lh.drive(exe, [lh.sim(**case), "fail 1", "step 20", "read", "step 3", "read"])]
        assert rc == [0, 0, EHIP, 0, 0, 0]


def test_a_capture_that_fails_loses_no_state(exe):
    """The library's own step graphs: nothing has run, the steps are launched."""
    res = lh.drive(exe, [lh.sim(128, 128, "fp64"), "step 256", "fail 1", "step 64", "read"])
    assert [r.rc for r in res] == [0] * 5 and len(res[3].launches) > 1


@pytest.mark.parametrize("march,middle", [(2, "ELi2ELb1ELb1"), (3, "ELi3ELb1ELb1")])
def test_captured_calls_split_into_passes_of_moments(exe, march, middle):
    """The step counts whose captures are compared bit for bit on the GPU:
    10 and 23 steps split, with a middle pass of either kind, 9 do not."""
    for prec in ("fp64", "fp32"):
        for nx, ny in ((330, 40), (433, 20), (37, 23)):
            env = ["env TFLBM_BLOCK 0", f"env TFLBM_MARCH {march}"]
            res = lh.drive(exe, env + [lh.sim(nx, ny, prec), "capture 10", "capture 23", "capture 9"])
            for r in res[-3:-1]:
                assert all("march_kernel" in l.kernel for l in r.launches) and len(r.launches) >= 4
            assert any(middle in l.kernel for r in res[-3:-1] for l in r.launches)
            assert not any("march_kernel" in l.kernel for l in res[-1].launches)


def test_fp64_two_step_passes_take_the_general_stages(exe):
    """On lattices of three steps per pass: calls of two steps, and without
    passes of moments the last pass of a call of 5."""
    sim = lh.sim(1024, 1024, "fp64")
    res = lh.drive(exe, ["env TFLBM_BLOCK 0", sim, "step 2", "env TFLBM_MARCH 0", sim, "step 5"])
    general, three = "11step_kernelILi0ELi1ELb0ELi2ELb0ELb0E", "11step_kernelILi0ELi1ELb0ELi3ELb0ELb1E"
    assert [general in l.kernel for l in res[2].launches] == [True]
    assert len(res[5].launches) == 2 and three in res[5].launches[0].kernel and general in res[5].launches[1].kernel
