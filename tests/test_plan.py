"""The workspace plan's shared regions (tests/sanitize/plan_checks.cpp), on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_36835_amd")
BUILD = os.path.join(PKG, "_build")


def test_plan_regions(tmp_path):
    from paper_2609_36835_amd import build as B
    objs = sorted(os.path.join(BUILD, f) for f in os.listdir(BUILD) if f.endswith(".hip.o")) if os.path.isdir(BUILD) else []
    if not objs:
        pytest.skip("kernel objects not built (run paper_2609_36835_amd.build first)")
    obj, exe = str(tmp_path / "plan.o"), str(tmp_path / "plan")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]
    for cmd in ([B._hipcc(), "-std=c++17", "-O1", *inc, "-c", os.path.join(ROOT, "tests", "sanitize", "plan_checks.cpp"),
                 "-o", obj], [B._hipcc(), f"--offload-arch={B.ARCH}", obj, *objs, "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, (" ".join(cmd), r.stderr[-4000:])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60, env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    print(r.stdout[-2000:])
    assert r.returncode == 0, r.stdout[-4000:]
