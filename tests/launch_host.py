"""The library's host side on the CPU: tests/launch_driver.c stands in for the
HIP runtime, records the launches of each call and lets a chosen one fail."""
import collections
import os
import shutil
import subprocess

from paper_1810_07642_amd import _lib

HERE = os.path.dirname(os.path.abspath(__file__))
PREC = {"fp64": 0, "fp32": 1, "fp16s": 2}
FIELD = {"uniform": 0, "theta": 1, "gamma": 2}

# a launch: its kernel (mangled name), grid, and the buffers it reads and writes
Launch = collections.namedtuple("Launch", "kernel grid src dst")
Result = collections.namedtuple("Result", "rc launches")


def compiler():
    return shutil.which("gcc") or shutil.which("cc")


def build_driver(out_dir):
    exe = os.path.join(str(out_dir), "launch_driver")
    lib = os.path.dirname(_lib.LIB_PATH)
    subprocess.run([compiler(), "-O1", "-rdynamic", "-I" + os.path.dirname(_lib.HEADER), "-o", exe,
                    os.path.join(HERE, "launch_driver.c"), "-L" + lib, "-l:" + os.path.basename(_lib.LIB_PATH),
                    "-Wl,-rpath," + lib, "-Wl,--allow-shlib-undefined"], check=True, capture_output=True, timeout=120)
    return exe


def sim(nx, ny, prec, tau=1.0, n=9, m=3, field="theta", g=0.0):
    """The command that creates, binds and initialises a handle (in place of an earlier one)."""
    return f"sim {nx} {ny} {PREC[prec]} {tau} {n} {m} {FIELD[field]} {g}"


def drive(exe, commands):
    """The Result of each command (see launch_driver.c), in one process."""
    env = {k: v for k, v in os.environ.items() if not k.startswith("TFLBM_")}
    r = subprocess.run([exe], input="\n".join(commands) + "\n", capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, r.stderr
    out, launches = [], []
    for line in r.stdout.splitlines():
        w = line.split()
        if w[0] == "launch":
            launches.append(Launch(w[1], int(w[2]), int(w[3], 16), int(w[4], 16)))
        else:
            out.append(Result(int(w[1]), launches))
            launches = []
    assert len(out) == len(commands)
    return out
