"""What the compiler's own notes in the built library say of the kernels: none spills to memory, and which arguments share a cache line."""
import os
import re

import pytest

from paper_2504_08838_amd import build

# .name and .private_segment_fixed_size are neighbours in a kernel's msgpack map (the keys are sorted)
NOTE = re.compile(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)(_Z\w+?)\xbb\.private_segment_fixed_size(.)", re.S)
# an argument's .offset (a small number, or a byte or two behind their mark), .size and .value_kind; the arguments stand in front of the name
GRID = re.compile(rb"\.offset([\x00-\x7f]|\xcc.|\xcd..)\xa5\.size\x04\xab\.value_kind\xb4hidden_block_count_x", re.S)


@pytest.fixture(scope="module")
def notes():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        return f.read()


@pytest.fixture(scope="module")
def scratch(notes):
    """First byte of the scratch size by kernel: 0 is none, anything else is some."""
    found = {m.group(1).decode(): m.group(2)[0] for m in NOTE.finditer(notes)}
    assert len(found) == notes.count(b".private_segment_fixed_size")
    return found


def test_every_kernel_keeps_everything_in_registers(scratch):
    """In the persistent forward -- thirteen variants: traced, probed, 2:4, query heads a group of the attention step -- a reload would
    wait behind the stream in flight, in every phase."""
    assert len(scratch) > 50 and sum("mega_forward_kernel" in name for name in scratch) == 13
    assert not [name for name, size in scratch.items() if size]


def test_the_dense_stream_has_its_arguments_and_the_grid_in_one_cache_line(notes):
    """The launches of a dense layer take a few microseconds each: a second line of 64 bytes is a trip that all of them wait for."""
    at = {}
    for m in NOTE.finditer(notes):
        if b"lm_head_kernel" in m.group(1):
            offset = list(GRID.finditer(notes, max(0, m.start() - 4096), m.start()))[-1].group(1)
            at[m.group(1)] = int.from_bytes(offset[len(offset) > 1:], "big")
    assert len(at) > 50 and max(at.values()) + 4 <= 64
