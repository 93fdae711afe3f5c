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
