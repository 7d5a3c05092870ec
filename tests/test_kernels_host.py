"""What the built library says about its kernels, and the host's share of what they compute with (nothing is launched)."""
import os
import re
import subprocess

import pytest


@pytest.fixture(scope="module")
def library():
    from paper_2412_20501_amd.build import ensure_built
    with open(ensure_built(), "rb") as f:
        return f.read()


def test_no_kernel_has_scratch(library):
    """A kernel with scratch starts about 1 us later.  The code objects' metadata (MessagePack) name each kernel's bytes a lane."""
    found = re.findall(rb"\.name\xd9.(_ZN2tr\w+)\xbb\.private_segment_fixed_size(.)", library, re.S)
    kernels = {name.decode(): size[0] for name, size in found}
    assert sum("block_attn_kernel" in name for name in kernels) == 56 and sum("merge" in name for name in kernels) > 4
    assert {name: size for name, size in kernels.items() if size} == {}


def test_divisions_by_multiplication(tmp_path):
    """csrc/divisor.h, which the kernels divide with, compiled for the host."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path / "divisor_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(root, "paper_2412_20501_amd", "csrc"),
                    os.path.join(root, "tests", "c_abi", "divisor_check.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "divisor ok" in res.stdout, res.stdout + res.stderr
