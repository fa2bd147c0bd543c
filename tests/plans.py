"""The library's GEMM plans for given sizes, from a small host program (tests/host/plan_driver.cpp) that includes the
planner's own header."""
import os
import subprocess
import tempfile
from collections import namedtuple

from paper_2306_15799_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256

SplitPlan = namedtuple("SplitPlan", "tm tn splits tilesM tilesN steps")
GradPlan = namedtuple("GradPlan", "fine splits tilesM tilesN starters")


_dir = None


def _driver():
    """The program, built once per test session."""
    global _dir
    if _dir is None:
        _dir = tempfile.TemporaryDirectory()
        subprocess.run([build.find_hipcc(), "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-I",
                        os.path.join(build.ROOT, "include"), "-I", build.CSRC, os.path.join(HERE, "host", "plan_driver.cpp"),
                        "-o", os.path.join(_dir.name, "plans")], check=True, capture_output=True, text=True)
    return os.path.join(_dir.name, "plans")


def _ask(lines):
    res = subprocess.run([_driver()], input="\n".join(lines), check=True, capture_output=True, text=True, timeout=300)
    return [[int(x) for x in line.split()] for line in res.stdout.splitlines()]


def proj(shapes):
    """Plans of the projection for (B, H, n, d, k, ...)."""
    return [SplitPlan(*r) for r in _ask(["proj %d %d %d %d %d" % tuple(s[:5]) for s in shapes])]


def fused(shapes):
    """Plans of the two paper-order products for (B, H, n, d, k, dm)."""
    return [(SplitPlan(*r[:6]), SplitPlan(*r[6:])) for r in _ask(["fused %d %d %d %d %d %d" % tuple(s) for s in shapes])]


def grad(shapes):
    """Plans of the gradient products for (B, H, n, d, k, ...)."""
    return [GradPlan(bool(r[0]), *r[1:]) for r in _ask(["grad %d %d %d %d %d" % tuple(s[:5]) for s in shapes])]


def ids(p):
    """Work item ids of the tile GEMM: (split, column tile, operand) padded to a multiple of 8, times the row tiles."""
    return 8 * p.tilesM * -(-p.splits * p.tilesN * 2 // 8)
