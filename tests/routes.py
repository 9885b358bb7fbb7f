"""The library's routing rules (csrc/routes.hpp, compiled by a small harness):
which boxes take launches of several steps.  The GPU tests of those launches
assert with it that their boxes do take them."""
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256  # compute units of the MI355X
BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2, "e4m11": 2}


@functools.lru_cache(maxsize=None)
def _harness():
    d = tempfile.mkdtemp(prefix="lbm_routes_")
    exe = os.path.join(d, "routes_harness")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror",
                    os.path.join(HERE, "routes_harness.cpp"), "-o", exe], check=True)
    return exe


def ask(lines):
    out = subprocess.run([_harness()], input="\n".join(lines) + "\n", capture_output=True, text=True,
                         check=True)
    return [[int(v) for v in line.split()] for line in out.stdout.splitlines()]


def march(lattice, dims, storage, bc=(0, 0, 0), mask=False, comp=False):
    """Planes per segment of the two-step launches of a 3D two-lattice box,
    None where it takes one-step launches."""
    if storage not in ("f64", "f32"):
        return None
    q = "march %d %d %d %d %d %d %d %d %d %d %d" % ((lattice, BYTES[storage]) + tuple(dims) + tuple(bc)
                                                    + (bool(mask), bool(comp), CUS))
    planes = ask([q])[0][0]
    return planes if planes > 0 else None
