"""What the compiler's own notes in the built library say of the kernels: none spills to memory."""
import os
import re

import pytest

from paper_2504_08838_amd import build

# .name and .private_segment_fixed_size are neighbours in a kernel's msgpack map (the keys are sorted)
NOTE = re.compile(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)(_Z\w+?)\xbb\.private_segment_fixed_size(.)", re.S)


@pytest.fixture(scope="module")
def scratch():
    """First byte of the scratch size by kernel: 0 is none, anything else is some."""
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        notes = f.read()
    found = {m.group(1).decode(): m.group(2)[0] for m in NOTE.finditer(notes)}
    assert len(found) == notes.count(b".private_segment_fixed_size")
    return found


def test_every_kernel_keeps_everything_in_registers(scratch):
    """In the persistent forward -- thirteen variants: traced, probed, 2:4, query heads a group of the attention step -- a reload would
    wait behind the stream in flight, in every phase."""
    assert len(scratch) > 50 and sum("mega_forward_kernel" in name for name in scratch) == 13
    assert not [name for name, size in scratch.items() if size]
