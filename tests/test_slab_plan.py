"""Host checks of the plans behind launches in slab order (csrc/hop_common.h)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2001_07557_amd", "csrc")


def run(tmp_path, name):
    hipcc = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) and shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    exe = str(tmp_path / name)
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", name + ".hip"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.strip().splitlines()


def test_most_tiles_of_a_slab(tmp_path):
    last = run(tmp_path, "slab_plan_check")[-1].split()
    assert last[0] == "cases" and int(last[1]) >= 10000 and last[2:] == ["bad", "0"]
