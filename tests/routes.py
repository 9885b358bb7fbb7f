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


STORAGE = {"f64": 0, "f32": 1, "f16": 2, "bf16": 3, "e4m11": 4}
REGIONS = ("24x8", "32x8", "32x6", "32x4")  # edge x most steps


def boxes_2d(questions):
    """Launches of D2Q9 two-lattice boxes, one per question (dims, storage, walls,
    mask, comp, steps): a list of (steps, "strips" | "24x8" | ... | "one")."""
    lines = ["2d %d %d %d %d %d %d %d" % (dims[0], dims[1], STORAGE[storage], bool(walls or mask), bool(mask),
                                          bool(comp), steps)
             for dims, storage, walls, mask, comp, steps in questions]
    out = []
    for row in ask(lines):
        launches = list(zip(row[4::2], row[5::2]))
        out.append([(k, "one" if k == 1 else "strips" if r < 0 else REGIONS[r]) for k, r in launches])
    return out


def box_2d(dims, storage, walls=False, mask=False, comp=False, steps=48):
    return boxes_2d([(dims, storage, walls, mask, comp, steps)])[0]
