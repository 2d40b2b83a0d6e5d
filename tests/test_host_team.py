"""Host check of the planning threads where a process gets no more of them
(tests/host_team_check.cpp).  Compiled like the planner check; no
device call."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2103_07512_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_host_team(tmp_path):
    from paper_2103_07512_amd import tgp
    assert os.path.exists(tgp.LIBRARY), "build the library first (__graft_entry__.build())"
    exe = str(tmp_path / "host_team_check")
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "-w", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(PKG, "csrc"), os.path.join(HERE, "host_team_check.cpp"), "-o", exe,
                        "-L", PKG, "-ltgp", f"-Wl,-rpath,{PKG}", "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-4000:] + r.stderr[-2000:]
