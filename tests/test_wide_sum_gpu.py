"""The blocked bf16 forwards that sum their directions in LDS, against the fp64
oracle: sides of one block of 8 lines, of odd block counts (two opposite scans
meet in the middle block) both ways, one way and neither way, scans of unequal
length, lines of 1 to 4 positions per lane, direction subsets without
opposite or crossing scans, and the largest sums LDS holds next to the first
that it does not.  Two runs give the same bits, and no workspace is taken.  With
one or two directions, whose sum has no order, the pixel-major call gives the same
bits too: both layouts round u * h and then add."""
import numpy as np
import pytest

import gspn_inputs as gi
import paper_2606_00746_amd as gspn
from gpu_util import ignored_taps, require_gpu, upload
from test_parity_gpu import case, check_against_oracle, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    case("sum-8x16", 2, 6, 3, 8, 16),
    case("sum-16x8-dirs14", 2, 6, 6, 16, 8, dirs=14),
    case("sum-24x40", 3, 8, 2, 24, 40),
    case("sum-40x24-dirs3", 2, 8, 8, 40, 24, dirs=3),
    case("sum-64x56-dirs12", 1, 8, 2, 64, 56, dirs=12),
    case("sum-72x72", 1, 6, 2, 72, 72),
    case("sum-80x72-dirs5", 2, 4, 4, 80, 72, dirs=5),
    case("sum-128x128", 1, 4, 1, 128, 128),
    case("sum-8x136-dirs10", 1, 4, 2, 8, 136, dirs=10),
    case("sum-136x120", 1, 4, 2, 136, 120),
    case("sum-256x72-dirs11", 1, 2, 1, 256, 72, dirs=11),
    case("sum-160x160-dirs8", 1, 2, 1, 160, 160, dirs=8),
    case("planes-168x168", 1, 2, 1, 168, 168),
]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_sum_in_lds(wl):
    torch = require_gpu()
    inputs = gi.make_inputs(wl)
    got = run_gpu(inputs, wl, False, layout="blocked")
    check_against_oracle(inputs, got, wl, False, wl.name)
    t = upload(inputs, wl.dtype, wl.dirs, layout="blocked")
    a, b = (gspn.scan_fwd(t["x"], t["w"], t["lam"], t["u"], wl.dirs, layout="blocked")
            for _ in range(2))
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    if bin(wl.dirs).count("1") <= 2:
        pm = upload(inputs, wl.dtype, wl.dirs)
        c = gspn.scan_fwd(pm["x"], pm["w"], pm["lam"], pm["u"], wl.dirs)
        assert torch.equal(a.view(torch.int16), c.view(torch.int16))
    n = gspn.workspace_size(gspn.OP_FWD_BLOCKED, t["x"], t["w"], wl.dirs)
    assert (n == 0) == wl.name.startswith("sum")


# pixel-major, enough planes (D B C > 512) on lines above 128 for the wide family:
# 3 and 4 positions per lane, vertical directions read in place alone (lanes that
# own the line's last columns, W = 136, 200, 8) and beside copied horizontal ones
WIDE = [
    case("wide-pm-160x136-c136", 1, 136, 8, 160, 136),
    case("wide-pm-136x200-dirs3", 2, 132, 4, 136, 200, dirs=3),
    case("wide-pm-256x64-dirs12", 2, 130, 26, 256, 64, dirs=12),
    case("wide-pm-8x200-T2B-G=C", 1, 516, 516, 8, 200, dirs=1),
    case("wide-pm-200x8-dirs9", 4, 66, 11, 200, 8, dirs=9),
    case("wide-pm-248x192-dirs7-peaky", 1, 174, 6, 248, 192, dirs=7, sigma=2.0),
]


def _is_wide(t, wl):
    """The query is the wide forward's: the directions' fp32 planes and the copies
    of the horizontal ones."""
    up = lambda n: (n + 255) // 256 * 256                          # noqa: E731
    n, nh = wl.B * wl.C * wl.H * wl.W, bin(wl.dirs & 12).count("1")
    need = up(4 * bin(wl.dirs).count("1") * n) + 2 * up(2 * nh * n) + \
        up(6 * nh * wl.B * wl.G * wl.H * wl.W)
    return gspn.workspace_size(gspn.OP_FWD, t["x"], t["w"], wl.dirs) == need


@pytest.mark.parametrize("wl", WIDE, ids=lambda w: w.name)
def test_wide_pixel_major(wl):
    """... against the oracle; taps that the scan ignores may hold NaN."""
    inputs = gi.make_inputs(wl)
    t = upload(inputs, wl.dtype, wl.dirs)
    assert _is_wide(t, wl)
    got = run_gpu(inputs, wl, False)
    check_against_oracle(inputs, got, wl, False, wl.name)
    w = inputs["w"].copy()
    w[np.broadcast_to(ignored_taps(wl.dirs, wl.H, wl.W)[:, None, None], w.shape)] = np.nan
    dirty = run_gpu({**inputs, "w": w}, wl, False)
    assert np.array_equal(dirty["y"], got["y"])
