"""CPU check of the single-box C entries: no exception can leave them for want of
memory, so their host code holds no throwing operator new (std::nothrow and HIP
allocations report a status instead)."""
import os
import subprocess

import pytest

from paper_2507_08820_amd import build


def test_single_box_entries_allocate_without_throwing(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not here")
    obj = tmp_path / "api.o"
    subprocess.run([build.HIPCC, f"--offload-arch={build.ARCH}", "--offload-host-only", "-O3", "-std=c++17", "-fPIC", "-c",
                    os.path.join(build.CSRC, "api.cpp"), "-o", str(obj)], check=True, capture_output=True)
    symbols = subprocess.run(["nm", str(obj)], check=True, capture_output=True, text=True).stdout.split()
    assert "rflbm_sk_sample" in symbols
    assert "_Znwm" not in symbols and "_Znam" not in symbols
