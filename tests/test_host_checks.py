"""Host-side code of libgspn, built and run on the CPU: the index functions that
the kernels share with the host, over every size they take, and the choice of the
kernel family."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2606_00746_amd", "csrc")


LIB = os.path.join(ROOT, "paper_2606_00746_amd", "libgspn.so")
LINK = (LIB, "-Wl,-rpath," + os.path.dirname(LIB))


def _build_and_run(tmp_path, name, *link, stdin=""):
    from paper_2606_00746_amd import build as lib_build
    exe = str(tmp_path / name)
    cmd = [lib_build.hipcc(), "--offload-arch=" + lib_build.ARCH, "--offload-host-only", "-O2",
           "-std=c++17", "-Wall", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-x", "hip",
           os.path.join(HERE, name + ".cpp"), "-x", "none", *link, "-o", exe]
    for c in (cmd, [exe]):
        r = subprocess.run(c, input=stdin, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, f"{' '.join(c)}\n{r.stdout[-4000:]}\n{r.stderr[-4000:]}"
    return r.stdout


def test_plane_records_stay_inside_lds(tmp_path):
    assert "all plans clean" in _build_and_run(tmp_path, "plane_lds")


def test_routes_follow_the_measured_times(tmp_path):
    assert "all routes clean" in _build_and_run(tmp_path, "routes", *LINK)


def test_gpu_cases_take_the_family_they_name(tmp_path):
    """The cases of the GPU tests that stand for one kernel family are that
    family's, pass by pass and layout by layout."""
    import test_line_gpu
    import test_plane_gpu
    import test_wide_sum_gpu
    both = ("fwd", "bwd", "fwd_blocked", "bwd_blocked")
    want = {}
    for cases, family, ops in ((test_plane_gpu.PLANE, "plane", both),
                               (test_plane_gpu.SMALL, "small", both),
                               (test_plane_gpu.MANY, "plane", ("fwd",)),
                               (test_line_gpu.CASES, "line", both),
                               (test_wide_sum_gpu.WIDE, "wide", ("fwd",)),
                               (test_wide_sum_gpu.CASES, "sum", ("fwd_blocked",))):
        for wl in cases:
            head = wl.name.split("-")[0]
            for op in ops:
                want[wl, op] = {"general": "general", "planes": "wide"}.get(head, family)
    lines = [f"{wl.name} {wl.B} {wl.C} {wl.G} {wl.H} {wl.W} {int(wl.dtype == 'bf16')} {wl.dirs} {op}"
             for wl, op in want]
    out = _build_and_run(tmp_path, "family", *LINK, stdin="\n".join(lines) + "\n")
    got = [tuple(ln.split()) for ln in out.splitlines()]
    assert got == [(wl.name, op, family) for (wl, op), family in want.items()]


def test_line_family_sizes_its_own_workspace():
    """From the held sizes on, the query gives what one round of the line family
    takes, not what the general family would (backwards of one large group,
    whose general kernels take its channels in turn)."""
    import paper_2606_00746_amd as g
    for dirs, C, G, H, W in ((15, 8, 1, 70, 70), (1, 32, 1, 80, 80), (3, 16, 1, 101, 67)):
        D = bin(dirs).count("1")
        st, n = g.gspn_workspace_size(g.OP_BWD, dirs, 1, C, G, H, W, g.BF16)
        assert st == 0 and n > 4 * D * (C + 4 * G) * H * W


def test_sizes_are_kept_per_current_device(monkeypatch):
    """The binding asks the library for a call's workspace (and reserve) once per
    sizes and device: the current device, on which the plan is made."""
    import torch

    from paper_2606_00746_amd import _native as n
    device = [0]
    monkeypatch.setattr(n, "_get_device", lambda: device[0], raising=False)
    monkeypatch.setattr(n, "gspn_workspace_size", lambda *a: (0, 1000 + device[0]))
    monkeypatch.setattr(n, "gspn_reserve_size", lambda *a: (0, 2000 + device[0]))
    x, w = torch.empty(1, 4, 99, 98), torch.empty(1, 1, 2, 3, 99, 98)
    on = torch.device("cpu")
    n._workspace_bytes.cache_clear()
    n._reserve_bytes.cache_clear()
    try:
        for device[0] in (0, 1, 0):
            assert n._workspace(0, 1, 1, 4, 2, 99, 98, 0, on)[1] == 1000 + device[0]
            assert n.reserve_size(x, w, 1) == 2000 + device[0]
    finally:
        n._workspace_bytes.cache_clear()
        n._reserve_bytes.cache_clear()
