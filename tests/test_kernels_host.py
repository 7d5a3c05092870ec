"""What the built library says about its kernels, and the host's share of what they compute with (nothing is launched)."""
import os
import re
import struct
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
    assert sum("segments_attn_kernel" in name for name in kernels) == 28 and sum("trio_attn_kernel" in name for name in kernels) == 6
    assert {name: size for name, size in kernels.items() if size} == {}


OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _code_objects(library):
    """The gfx950 code objects in the library's offload bundles."""
    at = library.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entries, place = struct.unpack_from("<Q", library, at + 24)[0], at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", library, place)
            if b"gfx950" in library[place + 24:place + 24 + length] and size:
                yield library[at + offset:at + offset + size]
            place += 24 + length
        at = library.find(b"__CLANG_OFFLOAD_BUNDLE__", place)


@pytest.fixture(scope="module")
def waits_in_steps(library, tmp_path_factory):
    """{kernel: waits for loads in the middle of a step, between its first and last product with V read from LDS}.  Steps run while the loads of later tiles
    are on their way, and every wait for those stands in front of a barrier: one that the compiler put into the stream itself drains them."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    found = {}
    for n, code in enumerate(_code_objects(library)):
        path = str(tmp_path_factory.mktemp("code") / f"{n}.co")
        with open(path, "wb") as f:
            f.write(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", path], capture_output=True, text=True, check=True).stdout
        name, run = None, []
        for line in text.splitlines() + ["<end>:"]:
            line = line.split("//")[0].strip()
            label = re.match(r"<(\w+)>:$", line)
            if label or "branch" in line or line.startswith(("s_barrier", "s_endpgm")):   # the end of a straight run
                work = [i for i, x in enumerate(run) if x.startswith(("v_mfma", "ds_read_b64_tr"))]
                if name and any(run[i].startswith("ds_read_b64_tr") for i in work):
                    found.setdefault(name, []).extend(x for x in run[work[0]:work[-1]] if x.startswith("s_waitcnt") and "vmcnt" in x)
                run = []
                if label and label[1].startswith("_Z"):
                    name = label[1]
            elif line:
                run.append(line)
    return found


@pytest.mark.parametrize("family,kernels", [("segments_attn_kernel", 28), ("trio_attn_kernel", 6)])
def test_steps_do_not_wait_for_loads(waits_in_steps, family, kernels):
    mine = {name: waits for name, waits in waits_in_steps.items() if family in name}
    assert len(mine) == kernels
    assert {name: waits for name, waits in mine.items() if waits} == {}


def test_divisions_by_multiplication(tmp_path):
    """csrc/divisor.h, which the kernels divide with, compiled for the host."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path / "divisor_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(root, "paper_2412_20501_amd", "csrc"),
                    os.path.join(root, "tests", "c_abi", "divisor_check.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "divisor ok" in res.stdout, res.stdout + res.stderr
