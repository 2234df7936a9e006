"""CPU check of the built step kernels: vector registers of the batch kernels.  A
persistent block of 256 threads keeps eight waves a SIMD with 64 registers a lane;
statistics, which hold a block to fewer waves by their LDS, may use 72."""
import os
import re
import subprocess

import pytest

from paper_2507_08820_amd import build

LLVM = "/opt/rocm/llvm/bin"


def kernels(obj, tmp):
    """(name, vector registers, scratch bytes) of every kernel of a built object."""
    fat, code = os.path.join(tmp, "fatbin"), os.path.join(tmp, "code")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, os.path.join(tmp, "copy.o")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={code}",
                    f"--targets=hipv4-amdgcn-amd-amdhsa--{build.ARCH}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    out = []
    for block in notes.split("  - .agpr_count")[1:]:
        get = lambda key: re.search(rf"\.{key}:\s+(\S+)", block).group(1)
        out.append((get("name"), int(get("vgpr_count")), int(get("private_segment_fixed_size"))))
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _, _ in out), check=True, capture_output=True,
                           text=True).stdout.split("\n")
    return [(name, v, s) for name, (_, v, s) in zip(names, out)]


def test_batch_kernels_keep_their_waves(tmp_path):
    obj = os.path.join(build.BUILD, "step.o")
    if not os.path.exists(obj) or not os.path.exists(f"{LLVM}/llvm-readelf"):
        pytest.skip("the built object or the LLVM tools are not here")
    seen = 0
    for name, vgprs, scratch in kernels(obj, str(tmp_path)):
        m = re.search(r"batch_kernel<(\d), (\w+), (\d+), (\d), (\w+), (\w+)>", name)
        if not m:
            continue
        assert scratch == 0, name
        if m.group(1) != "0" and m.group(4) == "1":  # 16-bit storage, every omega_g = 1
            seen += 1
            assert vgprs <= (72 if m.group(5) == "true" else 64), (name, vgprs)
    assert seen > 0
