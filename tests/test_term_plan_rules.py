"""The rules of the term sums' plan, read from the kernels' source: what the cuts of
the series may add up to, and that the benchmark's count of their work follows the
same rules."""
import math
import os
import re
from types import SimpleNamespace

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = open(os.path.join(ROOT, "paper_2605_29097_amd", "csrc", "cheb.hip")).read()


def _const(name):
    return float(re.search(rf"\b{name} = (-?[\d.]+);", SRC).group(1))


def _list(name):
    return [int(v) for v in re.search(rf"\b{name}\[\] = \{{([\d, ]+)\}}", SRC).group(1).split(",")]


def test_cuts_add_up_to_the_stated_bound():
    """1e-6 of the sum of the term magnitudes (include/rfvr.h).  Interpolation at K nodes is within twice the cut's bound,
    and with cells the box's own cut comes on top."""
    tol = 1e-6 * (1 + 1e-9)
    assert math.exp(_const("kChebLogTol")) <= tol
    box = math.exp(_const("kChebCellsLogTol"))
    assert box + 2 * math.exp(_const("kCellLogTol")) <= tol


@pytest.mark.parametrize("n_pts,n_meas,n_freq,side", [(1 << 20, 1024, 128, 0.2), (1 << 19, 1024, 64, 0.35), (1 << 19, 576, 100, 0.5),
                                                      (1 << 16, 2049, 64, 0.25), (1 << 20, 700, 101, 0.05),
                                                      (1 << 18, 1023, 64, 0.2), ((1 << 17) - 1, 1024, 64, 0.2), (1 << 20, 511, 64, 0.2)])
def test_benchmark_counts_the_plan_s_cells(n_pts, n_meas, n_freq, side):
    """bench.cell_order against the rule of k_cheb_plan and cell_count, with their constants as the source has them."""
    import bench
    corners = torch.tensor([[x, y, z] for x in (0.0, side) for y in (0.0, side) for z in (0.0, side)])
    xyz = torch.zeros(n_pts, 3)
    xyz[:8] = corners
    df = 4e9 / (n_freq - 1)
    got = bench.cell_order(24, xyz, SimpleNamespace(n_meas=n_meas, n_freq=n_freq, df=df))
    pays = re.search(r"over_points \? pairs >= \(n_meas < (\d+) \? ([\d.]+) : ([\d.]+)\) && n_meas >= (\d+) && n_pts >= \(1L << (\d+)\)", SRC)
    few, least_few, least, meas, pts = (float(v) for v in pays.groups())
    if n_pts * n_meas < (least_few if n_meas < few else least) or n_meas < meas or n_pts < 1 << int(pts):
        assert got == 0
        return
    most = min(int(re.search(r"kMaxCells = (\d+);", open(os.path.join(ROOT, "paper_2605_29097_amd", "csrc", "rfvr_impl.hpp")).read()).group(1)),
               n_pts // 256, (1 << 21) // n_meas)
    edge = max(t for t in range(1, 65) if t ** 3 <= most)
    h = 0.5 * math.sqrt(3) * float(torch.tensor(side)) / edge * (1 + 1e-5) + 1e-6
    z = 2 * math.pi * 0.5 * (n_freq - 1) * 2 * df / 299792458.0 * h
    log_bound = lambda k: (-math.inf if z <= 0 else math.inf if z / 2 >= k + 1 else
                           k * math.log(z / 2) - math.lgamma(k + 1) + math.log(2) - math.log1p(-z / 2 / (k + 1)))
    want = [k for k in _list("kCellKs") if log_bound(k) <= _const("kCellLogTol")]
    assert got == (want[0] if want else 0)


def test_benchmark_counts_no_cells_for_coinciding_points():
    import bench
    assert bench.cell_order(24, torch.ones(1 << 18, 3), SimpleNamespace(n_meas=1024, n_freq=64, df=6e7)) == 0
