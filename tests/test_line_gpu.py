"""The line family (planes with a side of 65 to 256 that no other family takes)
against the fp64 oracle, at the sizes where it changes its plan: lines of 64,
65, 128, 129, 256 positions (1, 2 and 4 positions per lane) and 257 (the
general family), lengths that are no multiple of a lane's positions, lines
shorter than them, tiles of 32 x 64 pixels with remainders, groups in one and
several channel chunks, both layouts and types; and gspn_scan_bwd_static, whose
fixed workspace makes it take smaller rounds or the general family."""
import numpy as np
import pytest

import gspn_inputs as gi
import oracle
import paper_2606_00746_amd as gspn
from gpu_util import normwise_err, require_gpu, to_host, tolerance, upload
from test_parity_gpu import case, check_against_oracle, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    case("line-65x64", 2, 6, 3, 65, 64),
    case("line-64x65-dirs6", 4, 40, 8, 64, 65, dirs=6),
    case("line-33x128-cpg9", 4, 36, 4, 33, 128),
    case("line-129x31-G=C", 4, 24, 24, 129, 31, dirs=13),
    case("line-127x67-f32", 2, 16, 4, 127, 67, dtype="f32", gate="normal"),
    case("line-131x150-f32", 1, 16, 4, 131, 150, dtype="f32", gate="normal"),
    case("line-256x254-cpg8", 1, 8, 1, 256, 254, dirs=9),
    case("line-1x66", 4, 200, 50, 1, 66),
    case("line-100x1", 4, 128, 32, 100, 1),
    case("line-201x1", 2, 128, 32, 201, 1),
    case("line-2x200-G=C", 2, 70, 70, 2, 200),
    case("line-3x131-f32-dirs5", 2, 128, 32, 3, 131, dirs=5, dtype="f32", gate="normal"),
    case("general-257x10", 1, 2, 1, 257, 10),
]


def query(wl, op):
    require_gpu()               # (torch first: the library then shares its HIP runtime)
    dt = gspn.BF16 if wl.dtype == "bf16" else gspn.F32
    st, need = gspn.gspn_workspace_size(op, wl.dirs, wl.B, wl.C, wl.G, wl.H, wl.W, dt)
    assert st == 0
    return need


def general_need(wl, backward):
    """What the general family takes: the line family's query differs from it."""
    D, HW = bin(wl.dirs).count("1"), wl.H * wl.W
    return 4 * D * HW * wl.B * (wl.C + (4 * wl.G if backward else 0))


@pytest.mark.parametrize("layout", ["pixel", "blocked"])
@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_line_parity(wl, layout):
    for op, backward in (((gspn.OP_FWD, False), (gspn.OP_BWD, True)) if layout == "pixel" else
                         ((gspn.OP_FWD_BLOCKED, False), (gspn.OP_BWD_BLOCKED, True))):
        if backward and wl.G == wl.C:
            continue              # (the general family takes more than a round there)
        general = query(wl, op) == general_need(wl, backward)
        assert general == wl.name.startswith("general"), (wl.name, op)
    inputs = gi.make_inputs(wl, with_dy=True)
    got = run_gpu(inputs, wl, True, layout=layout)
    check_against_oracle(inputs, got, wl, True, f"{wl.name} {layout}")


@pytest.mark.parametrize("wl,same", [
    (case("static-rounds", 8, 24, 6, 100, 101), True),      # two rounds instead of one
    (case("static-general", 1, 24, 1, 256, 250), False),    # one group does not fit
], ids=lambda v: getattr(v, "name", ""))
def test_static_backward_limits(wl, same):
    """gspn_scan_bwd_static works in 64 MiB: smaller rounds than gspn_scan_bwd
    give the same bits; where one group's lines do not fit it runs the general
    family, whose need decides what it refuses."""
    torch = require_gpu()
    print(f"[case] {wl.name}", flush=True)
    assert query(wl, gspn.OP_BWD) > 64 << 20
    inputs = gi.make_inputs(wl, with_dy=True)
    t = upload(inputs, wl.dtype, wl.dirs)
    ref = gspn.scan_bwd(t["x"], t["w"], t["lam"], t["u"], t["dy"], wl.dirs)
    out = [torch.empty_like(v) for v in ref]
    args = [t[k].data_ptr() for k in ("x", "w", "lam", "u", "dy")] + [v.data_ptr() for v in out]
    st = gspn.gspn_scan_bwd_static(*args, wl.dirs, wl.B, wl.C, wl.G, wl.H, wl.W, gspn.BF16,
                                   torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    for k, a, b in zip(("dx", "dw", "dlam", "du"), out, ref):
        if same:
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), k
        else:
            assert normwise_err(to_host(a), to_host(b)) <= tolerance(wl.dtype), k


@pytest.mark.parametrize("wl,layout,part", [
    (case("less-workspace", 2, 32, 8, 90, 101), "pixel", None),
    # half of the need: two rounds of groups that are split into chunks (and, with
    # an odd count of groups, of unequal length)
    (case("less-split-f32", 3, 72, 2, 90, 101, dtype="f32", gate="normal"), "blocked", 0.55),
    (case("less-split-cpg36", 5, 36, 1, 130, 70), "pixel", 0.65),
    (case("less-blocked", 2, 32, 8, 70, 134, dirs=11), "blocked", 0.55),
], ids=lambda v: getattr(v, "name", ""))
def test_caller_with_less_workspace(wl, layout, part):
    """A workspace below the query's size but of what the general family takes
    is accepted: the line family in smaller rounds (the same bits)."""
    torch = require_gpu()
    print(f"[case] {wl.name}", flush=True)
    inputs = gi.make_inputs(wl, with_dy=True)
    t = upload(inputs, wl.dtype, wl.dirs, layout)
    ref = gspn.scan_bwd(t["x"], t["w"], t["lam"], t["u"], t["dy"], wl.dirs, layout=layout)
    blocked = layout == "blocked"
    need = query(wl, gspn.OP_BWD_BLOCKED if blocked else gspn.OP_BWD)
    less = int(part * need) if part else general_need(wl, True)
    assert general_need(wl, True) <= less < need
    out = [torch.full_like(v, float("nan")) for v in ref]
    ws = torch.empty(less, dtype=torch.uint8, device="cuda")
    ptrs = [t[k].data_ptr() for k in ("x", "w", "lam", "u", "dy")] + [v.data_ptr() for v in out]
    args = (wl.dirs, wl.B, wl.C, wl.G, wl.H, wl.W,
            gspn.BF16 if wl.dtype == "bf16" else gspn.F32, ws.data_ptr())
    stream = torch.cuda.current_stream().cuda_stream
    bwd = gspn.gspn_scan_bwd_blocked if blocked else gspn.gspn_scan_bwd
    assert bwd(*ptrs, *args, general_need(wl, True) - 1, stream) == -9
    assert bwd(*ptrs, *args, less, stream) == 0
    torch.cuda.synchronize()
    for k, a, b in zip(("dx", "dw", "dlam", "du"), out, ref):
        assert torch.equal(a, b), k


@pytest.mark.parametrize("wl,same", [
    (case("less-forward-wide", 1, 8, 8, 128, 128), False),   # rounds of a plane: general
    (case("less-forward-cpg64", 3, 64, 1, 72, 80), True),    # rounds of a group
    (case("less-forward-odd", 1, 8, 4, 77, 101), False),
], ids=lambda v: getattr(v, "name", ""))
def test_forward_with_less_workspace(wl, same):
    """A forward whose caller has what the general family takes (and no less) is
    accepted, whichever family the query sizes."""
    torch = require_gpu()
    print(f"[case] {wl.name}", flush=True)
    inputs = gi.make_inputs(wl)
    t = upload(inputs, wl.dtype, wl.dirs)
    ref = gspn.scan_fwd(t["x"], t["w"], t["lam"], t["u"], wl.dirs)
    less = 4 * 4 * wl.B * wl.C * wl.H * wl.W
    assert gspn.workspace_size(gspn.OP_FWD, t["x"], t["w"], wl.dirs) > less
    y = torch.full_like(t["x"], float("nan"))
    ws = torch.empty(less, dtype=torch.uint8, device="cuda")
    args = [t[k].data_ptr() for k in ("x", "w", "lam", "u")] + [y.data_ptr(), wl.dirs, wl.B, wl.C,
                                                              wl.G, wl.H, wl.W, gspn.BF16,
                                                              ws.data_ptr()]
    stream = torch.cuda.current_stream().cuda_stream
    assert gspn.gspn_scan_fwd(*args, less - 1, stream) == -9
    assert gspn.gspn_scan_fwd(*args, less, stream) == 0
    torch.cuda.synchronize()
    if same:
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
    check_against_oracle(inputs, {"y": to_host(y)}, wl, False, wl.name)


def test_line_rounds():
    """More planes than one round's workspace (512 MB) holds: units of the
    first and the last round against the oracle."""
    wl = case("line-rounds", 6, 192, 12, 130, 129)
    lines = 2 * 4 * 4 * wl.B * wl.C * wl.H * wl.W        # h and a of four directions
    assert query(wl, gspn.OP_BWD) < lines
    inputs = gi.make_inputs(wl, with_dy=True)
    got = run_gpu(inputs, wl, True)
    cpg = wl.C // wl.G
    for b, g in [(0, 0), (3, 7), (5, 11)]:
        sl = oracle.slice_group(inputs, b, g, wl.G)
        cs = slice(g * cpg, (g + 1) * cpg)
        part = {"y": got["y"][b:b + 1, cs], "dx": got["dx"][b:b + 1, cs],
                "dw": got["dw"][:, b:b + 1, g:g + 1], "dlam": got["dlam"][:, b:b + 1, cs],
                "du": got["du"][:, b:b + 1, cs]}
        check_against_oracle(sl, part, wl.with_(B=1, C=cpg, G=1), True, f"{wl.name} b={b} g={g}")
    assert all(np.all(np.isfinite(v)) for v in got.values())
