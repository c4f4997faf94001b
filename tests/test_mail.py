"""Host check of the slots through which kernels hand numbers to the host
(``csrc/mail.hip``): the driver plays the stream by hand, so a post can come
late, never, or after its call has given up.  No GPU call is made."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2001_07557_amd", "csrc")


def test_slots_are_given_out_again_only_when_their_posts_have_landed(tmp_path):
    hipcc = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) and shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    exe = str(tmp_path / "mail_check")
    subprocess.run([hipcc, "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "mail_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    last = r.stdout.strip().splitlines()[-1].split()
    assert last[0] == "checks" and int(last[1]) >= 9 and last[2:] == ["bad", "0"], r.stdout
