"""Host-side code of libgspn, built and run on the CPU: the index functions that
the kernels share with the host, over every size they take, and the choice of the
kernel family."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2606_00746_amd", "csrc")


def _build_and_run(tmp_path, name, *link):
    from paper_2606_00746_amd import build as lib_build
    exe = str(tmp_path / name)
    cmd = [lib_build.hipcc(), "--offload-arch=" + lib_build.ARCH, "--offload-host-only", "-O2",
           "-std=c++17", "-Wall", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-x", "hip",
           os.path.join(HERE, name + ".cpp"), "-x", "none", *link, "-o", exe]
    for c in (cmd, [exe]):
        r = subprocess.run(c, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, f"{' '.join(c)}\n{r.stdout[-4000:]}\n{r.stderr[-4000:]}"
    return r.stdout


def test_plane_records_stay_inside_lds(tmp_path):
    assert "all plans clean" in _build_and_run(tmp_path, "plane_lds")


def test_routes_follow_the_measured_times(tmp_path):
    assert "all routes clean" in _build_and_run(tmp_path, "routes", os.path.join(
        ROOT, "paper_2606_00746_amd", "libgspn.so"),
        "-Wl,-rpath," + os.path.join(ROOT, "paper_2606_00746_amd"))


def test_line_family_sizes_its_own_workspace():
    """From the held sizes on, the query gives what one round of the line family
    takes, not what the general family would (backwards of one large group,
    whose general kernels take its channels in turn)."""
    import paper_2606_00746_amd as g
    for dirs, C, G, H, W in ((15, 8, 1, 70, 70), (1, 32, 1, 80, 80), (3, 16, 1, 101, 67)):
        D = bin(dirs).count("1")
        st, n = g.gspn_workspace_size(g.OP_BWD, dirs, 1, C, G, H, W, g.BF16)
        assert st == 0 and n > 4 * D * (C + 4 * G) * H * W
