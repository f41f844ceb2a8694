"""The rules of the term sums' plan, read from the kernels' source: what the cuts of
the series may add up to."""
import math
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = open(os.path.join(ROOT, "paper_2605_29097_amd", "csrc", "cheb.hip")).read()


def _const(name):
    return float(re.search(rf"\b{name} = (-?[\d.]+);", SRC).group(1))


def test_cuts_add_up_to_the_stated_bound():
    """1e-6 of the sum of the term magnitudes (include/rfvr.h).  Interpolation at K nodes is within twice the cut's bound,
    and with cells the box's own cut comes on top."""
    tol = 1e-6 * (1 + 1e-9)
    assert math.exp(_const("kChebLogTol")) <= tol
    box = math.exp(_const("kChebCellsLogTol"))
    assert box + 2 * math.exp(_const("kCellLogTol")) <= tol
