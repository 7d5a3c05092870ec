"""What the built library says about its kernels, and the host's share of what they compute with (nothing is launched)."""
import re

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
