"""The listing of steps that the kernels over steps run, checked on the host: tests/native/list_steps_check.cpp includes host.cpp and links the built library."""
import os
import subprocess

from paper_2311_09549_amd import binding as sc

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_leaf_is_listed_once(tmp_path):
    exe, where = str(tmp_path / "list_steps_check"), os.path.dirname(sc.LIB_PATH)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "-w", "-x", "hip", "--offload-host-only", os.path.join(HERE, "native", "list_steps_check.cpp"), "-o", exe,
                           "-L" + where, "-lsparsecontract", "-Wl,-rpath," + where, "-pthread"], timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)   # (a piece that fits no chunk was once tried for ever)
    assert r.returncode == 0, r.stdout + r.stderr
