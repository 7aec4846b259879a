"""Buffer requests straight into LDS, as the built library has them: what keeps them inside their buffer is the range check, and that
looks at the request's vector and immediate offsets alone -- the scalar offset is not part of it.  So none may have one."""
import collections
import os
import re
import struct
import subprocess

import pytest

from paper_2504_08838_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
REQUEST = re.compile(r"buffer_load_dword\w* (?:v\d+|off), s\[\d+:\d+\], (\S+)(?: .*)? lds\b")


def _code_objects(lib):
    """The GPU code of every source file: a bundle is its magic, a count, then (offset, size, length of the name, name) per target."""
    at = lib.find(BUNDLE)
    while at >= 0:
        pos = at + len(BUNDLE) + 8
        for _ in range(struct.unpack_from("<Q", lib, at + len(BUNDLE))[0]):
            off, size, n = struct.unpack_from("<QQQ", lib, pos)
            if b"gfx950" in lib[pos + 24:pos + 24 + n]:
                yield lib[at + off:at + off + size]
            pos += 24 + n
        at = lib.find(BUNDLE, at + 1)


@pytest.fixture(scope="module")
def scalar_offsets(tmp_path_factory):
    """Scalar offset operands of all such requests, by kernel family."""
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        lib = f.read()
    found = collections.defaultdict(collections.Counter)
    for i, code in enumerate(_code_objects(lib)):
        path = tmp_path_factory.mktemp("code") / f"{i}.co"
        path.write_bytes(code)
        kernel = None
        asm = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True)
        for line in asm.stdout:
            if line.endswith(">:\n"):
                kernel = re.search(r"sd2\d+([a-z]\w*?_kernel)", line)
            elif " lds" in line and "buffer_load" in line:
                found[kernel.group(1)][REQUEST.search(line).group(1)] += 1
        assert asm.wait() == 0
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
@pytest.mark.parametrize("kernel", ["mega_forward_kernel", "lm_head_kernel"])
def test_no_scalar_offset(scalar_offsets, kernel):
    assert list(scalar_offsets[kernel]) == ["0"]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_other_kernel_has_such_requests(scalar_offsets):
    assert set(scalar_offsets) == {"mega_forward_kernel", "lm_head_kernel"}
