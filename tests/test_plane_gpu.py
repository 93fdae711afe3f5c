"""Planes with both sides at most 64 outside the square kernels, against the
fp64 oracle, on either side of every line where the kernel changes: 8-step
blocks and lanes per channel (16, 17, 32, 33, 40 and 41 a side), odd and even
widths (odd planes start at any 2-byte address), one pixel, rows and columns,
one channel per group, channels that fill a workgroup unevenly, a group in
several workgroups, both types and layouts; shapes with enough planes for the
plane family in every pass and, with few, for the line family and the small
kernels."""
import numpy as np
import pytest

import gspn_inputs as gi
import oracle
import paper_2606_00746_amd as gspn
from gpu_util import ignored_taps, require_gpu, to_host, upload
from test_parity_gpu import GRAD_KEYS, case, check_against_oracle, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    case("1x1-cpg5", 2, 10, 2, 1, 1),
    case("7x7-cpg33", 2, 66, 2, 7, 7),
    case("16x9-dirs6", 2, 40, 4, 16, 9, dirs=6),
    case("15x16-f32-cpg9", 2, 36, 4, 15, 16, dtype="f32", gate="normal"),
    case("8x8-f32-G=C", 1, 12, 12, 8, 8, dtype="f32", gate="normal"),
    case("17x17-cpg13", 4, 208, 16, 17, 17),
    case("28x28-cpg12", 4, 192, 16, 28, 28),
    case("25x32-cpg3-dirs11", 4, 192, 64, 25, 32, dirs=11),
    case("32x31-f32-cpg5", 4, 160, 32, 32, 31, dtype="f32", gate="normal"),
    case("31x18-G=C", 2, 300, 300, 31, 18),
    case("33x33-cpg2", 2, 288, 144, 33, 33),
    case("37x37-cpg32", 1, 288, 9, 37, 37),
    case("40x34-dirs9-peaky", 2, 288, 144, 40, 34, dirs=9, sigma=2.0),
    case("41x37-cpg9", 4, 288, 32, 41, 37),
    case("37x20-G=C", 1, 300, 300, 37, 20, dirs=5),
    case("37x38-f32-cpg4", 2, 288, 72, 37, 38, dtype="f32", gate="normal"),
    case("36x36-cpg31", 1, 310, 10, 36, 36),
    case("few-28x28", 1, 6, 2, 28, 28),
    case("few-53x64", 1, 5, 1, 53, 64),
    case("1x64", 2, 6, 3, 1, 64),
    case("64x2-f32-dirs14", 1, 6, 1, 64, 2, dirs=14, dtype="f32", gate="normal"),
    case("64x64-f32", 1, 4, 2, 64, 64, dtype="f32", gate="normal"),
]


# planes enough that the plane family takes both passes in both layouts: every
# count of 8-step blocks, both types
PLANE = [
    case("7x7-cpg33-all", 16, 231, 7, 7, 7),
    case("8x7-f32-cpg9", 8, 450, 50, 8, 7, dtype="f32", gate="normal"),
    case("13x14-cpg3-dirs11", 8, 402, 134, 13, 14, dirs=11),
    case("16x9-cpg10-dirs6", 8, 400, 40, 16, 9, dirs=6),
    case("15x16-f32-cpg9-all", 8, 405, 45, 15, 16, dtype="f32", gate="normal"),
    case("17x17-cpg13-all", 8, 221, 17, 17, 17),
    case("24x20-f32-cpg12", 6, 288, 24, 24, 20, dtype="f32", gate="normal"),
    case("20x17-f32-B2T", 4, 2048, 256, 20, 17, dirs=2, dtype="f32", gate="normal"),
    case("28x28-cpg12-all", 8, 216, 18, 28, 28),
    case("25x31-cpg5-dirs3", 8, 250, 50, 25, 31, dirs=3),
    case("18x28-f32-cpg6-dirs13", 6, 300, 50, 18, 28, dirs=13, dtype="f32", gate="normal"),
    case("37x37-cpg32-all", 4, 256, 8, 37, 37),
    case("40x21-cpg8", 4, 256, 32, 40, 21),
    case("33x34-f32-cpg4-dirs12", 4, 256, 64, 33, 34, dirs=12, dtype="f32", gate="normal"),
    case("36x11-f32-cpg8", 4, 256, 32, 36, 11, dtype="f32", gate="normal"),
    case("48x19-cpg12-dirs12", 4, 252, 21, 48, 19, dirs=12),
    case("41x15-f32-cpg8", 4, 256, 32, 41, 15, dtype="f32", gate="normal"),
    case("53x20-cpg8", 4, 256, 32, 53, 20),
    case("10x55-f32-cpg8", 4, 256, 32, 10, 55, dtype="f32", gate="normal"),
    case("64x12-cpg9", 4, 252, 28, 64, 12),
    case("9x61-f32-cpg8", 4, 256, 32, 9, 61, dtype="f32", gate="normal"),
]

# planes of a few pixels, which the small kernels take in both passes
SMALL = [
    case("2x2-f32-cpg3", 2, 6, 2, 2, 2, dtype="f32", gate="normal"),
    case("3x3-cpg4-dirs7", 3, 8, 2, 3, 3, dirs=7),
    case("1x3-cpg16", 1, 32, 2, 1, 3),
    case("1x13-G=C-R2L", 2, 5, 5, 1, 13, dirs=8),
]

# one channel a group up to 16 a side: so many planes that the pixel-major forward is
# the plane family's, with one channel in a wave of four
MANY = [
    case("many-8x8-f32-G=C", 10, 1960, 1960, 8, 8, dtype="f32", gate="normal"),
    case("many-5x9-f32-G=C-dirs6", 10, 1961, 1961, 5, 9, dirs=6, dtype="f32", gate="normal"),
    case("many-6x7-G=C-dirs12", 16, 3001, 3001, 6, 7, dirs=12),
    case("many-4x11-G=C-dirs7", 16, 3000, 3000, 4, 11, dirs=7),
]


@pytest.mark.parametrize("wl", MANY, ids=lambda w: w.name)
def test_many_planes_forward(wl):
    inputs = gi.make_inputs(wl, with_dy=False)
    check_against_oracle(inputs, run_gpu(inputs, wl, False), wl, False, wl.name)


@pytest.mark.parametrize("layout", ["pixel", "blocked"])
@pytest.mark.parametrize("wl", CASES + PLANE + SMALL, ids=lambda w: w.name)
def test_plane_parity(wl, layout):
    inputs = gi.make_inputs(wl, with_dy=True)
    got = run_gpu(inputs, wl, True, layout=layout)
    check_against_oracle(inputs, got, wl, True, f"{wl.name} {layout}")


@pytest.mark.parametrize("wl", [case("nan-13x14", 8, 402, 134, 13, 14),
                                case("nan-40x21", 4, 256, 32, 40, 21),
                                case("nan-28x28", 4, 192, 16, 28, 28),
                                case("nan-37x37", 2, 288, 144, 37, 37),
                                case("nan-few-45x64", 1, 4, 2, 45, 64)], ids=lambda w: w.name)
def test_ignored_taps_may_hold_nan(wl):
    inputs = gi.make_inputs(wl, with_dy=True)
    clean = run_gpu(inputs, wl, True)
    w = inputs["w"].copy()
    ign = ignored_taps(wl.dirs, wl.H, wl.W)
    w[np.broadcast_to(ign[:, None, None], w.shape)] = np.nan
    got = run_gpu({**inputs, "w": w}, wl, True)
    for k in ("y",) + GRAD_KEYS:
        assert np.array_equal(got[k], clean[k]), k


@pytest.mark.parametrize("wl", [case("inf-13x15-cpg12", 8, 408, 34, 13, 15),
                                case("inf-40x21", 4, 256, 32, 40, 21),
                                case("inf-16x16-f32", 4, 192, 16, 16, 16, dtype="f32"),
                                case("inf-13x15", 4, 192, 16, 13, 15),
                                case("inf-37x37", 2, 288, 144, 37, 37),
                                case("inf-few-64x40", 1, 8, 2, 64, 40),
                                case("inf-28x28", 4, 192, 16, 28, 28)], ids=lambda w: w.name)
def test_infinity_stays_in_its_channel(wl):
    """An infinite x in one channel changes nothing of the other channels, and
    the gradients of ignored taps stay 0.  (Lines of 17 to 32 positions share
    a wave by twos, whose shifts pass 0 x infinity on: there, of the channels
    of the other groups.)"""
    inputs = gi.make_inputs(wl, with_dy=True)
    clean = run_gpu(inputs, wl, True)
    c = 5
    x = inputs["x"].copy()
    x[0, c, 0, :] = np.inf
    got = run_gpu({**inputs, "x": x}, wl, True)
    cpg = wl.C // wl.G
    pairs = 17 <= max(wl.H, wl.W) <= 32
    others = [k for k in range(wl.C) if (k // cpg != c // cpg if pairs else k != c)]
    for key, axis in (("y", 1), ("dx", 1), ("dlam", 2), ("du", 2)):
        a, b = (np.take(v[key], others, axis=axis) for v in (got, clean))
        assert np.array_equal(a, b), key
    ign = np.broadcast_to(ignored_taps(wl.dirs, wl.H, wl.W)[:, None, None], got["dw"].shape)
    assert np.all(got["dw"][ign] == 0.0)


@pytest.mark.parametrize("wl", [case("adj-13x15", 4, 192, 16, 13, 15),
                                case("adj-15x13-f32", 2, 96, 8, 15, 13, dtype="f32"),
                                case("adj-28x28", 4, 192, 16, 28, 28),
                                case("adj-25x29-f32", 4, 160, 32, 25, 29, dtype="f32"),
                                case("adj-37x37", 2, 288, 144, 37, 37),
                                case("adj-few-40x45", 1, 8, 2, 40, 45)], ids=lambda w: w.name)
def test_infinite_adjoint_at_a_lines_end(wl):
    """An infinite dy at the last position of the lines both ways (the corner):
    the off-grid taps there are ignored, so infinities stay infinite, with the
    oracle's sign, and nothing becomes NaN that is none by the equations (u, w
    and lam are positive and x is made positive; the other channels of the
    group keep their bits)."""
    inputs = gi.make_inputs(wl, with_dy=True)
    inputs["x"] = np.maximum(np.abs(inputs["x"]), np.float32(0.5))
    clean = run_gpu(inputs, wl, True)
    c = 5
    dy = inputs["dy"].copy()
    dy[0, c, wl.H - 1, wl.W - 1] = np.inf
    got = run_gpu({**inputs, "dy": dy}, wl, True)
    ref = oracle.scan_bwd(inputs["x"], inputs["w"], inputs["lam"], inputs["u"], dy, wl.dirs)
    for k in GRAD_KEYS:
        assert np.array_equal(np.isnan(got[k]), np.isnan(ref[k])), k
        assert np.array_equal(got[k] == np.inf, ref[k] == np.inf), k
        assert not np.isneginf(got[k]).any(), k
    assert np.isinf(ref["dlam"][:, 0, c]).sum() > wl.H * wl.W
    others = [k for k in range(wl.C) if k != c]
    for k, axis in (("dx", 1), ("dlam", 2), ("du", 2)):
        assert np.array_equal(np.take(got[k], others, axis=axis),
                              np.take(clean[k], others, axis=axis)), k


@pytest.mark.parametrize("wl", [case("no-workspace-50x64", 1, 8, 1, 50, 64),
                                case("no-workspace-43x30-dirs12", 2, 126, 42, 43, 30, dirs=12)],
                         ids=lambda w: w.name)
def test_caller_without_workspace(wl):
    """A backward whose groups now split over more workgroups than its query
    once sized (or lines go through memory) still runs in no workspace, and so
    does the forward, in the plane family for many planes."""
    torch = require_gpu()
    print(f"[case] {wl.name}", flush=True)
    inputs = gi.make_inputs(wl, with_dy=True)
    t = upload(inputs, wl.dtype, wl.dirs)
    out = [torch.empty_like(t[k]) for k in ("x", "w", "lam", "u")]
    ptrs = [t[k].data_ptr() for k in ("x", "w", "lam", "u", "dy")] + [v.data_ptr() for v in out]
    y = torch.empty_like(t["x"])
    args = (wl.dirs, wl.B, wl.C, wl.G, wl.H, wl.W, gspn.BF16, None, 0,
            torch.cuda.current_stream().cuda_stream)
    assert gspn.gspn_scan_fwd(*[t[k].data_ptr() for k in ("x", "w", "lam", "u")], y.data_ptr(),
                              *args) == 0
    assert gspn.gspn_scan_bwd(*ptrs, *args) == 0
    torch.cuda.synchronize()
    got = {"y": to_host(y), **dict(zip(GRAD_KEYS, (to_host(v) for v in out)))}
    check_against_oracle(inputs, got, wl, True, wl.name)
