"""The pinned result slots (csrc/host_slot.h) on the CPU, with stand-ins for HIP."""
import os
import subprocess

import pytest

from conftest import ROOT

ROCM = "/opt/rocm/include"


@pytest.mark.skipif(not os.path.isdir(os.path.join(ROCM, "hip")), reason="needs the HIP headers")
def test_slots_are_waited_for_and_given_back(tmp_path):
    """A slot lent to a kernel is given back only after a wait for its stream, on
    early returns too; one that cannot be waited for stays taken; a call that finds
    none free copies."""
    exe = str(tmp_path / "host_slot_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", ROCM,
                    "-I", os.path.join(ROOT, "paper_2608_23144_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host_slot_check.cpp"), "-o", exe, "-pthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
