"""CPU-only checks of the machine code that the built library holds, where the kernels rely on an order that the compiler is free to change."""
import functools
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2605_09825_amd as mx

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(library):
    """The gfx950 code objects inside a HIP library: bundles of (offset, size, target) entries."""
    data = open(library, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if target.endswith(b"gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


@functools.lru_cache(maxsize=None)
def kernels():
    """Instructions of every kernel of the built library, by mangled name."""
    objdump = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(mx.LIB_PATH):
        from paper_2605_09825_amd.build import build
        build()
    found = {}
    for code in code_objects(mx.LIB_PATH):
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--no-leading-addr", "/dev/stdin"], input=code,
                              capture_output=True, check=True).stdout.decode()
        lines = None
        for line in text.splitlines():
            name = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:", line)
            if name:
                lines = found.setdefault(name.group(1), [])
            elif lines is not None and line.startswith("\t"):
                lines.append(line.split("//")[0].strip())
    assert found
    return found


def named(pattern):
    got = {n: code for n, code in kernels().items() if re.search(pattern, n)}
    assert got, pattern
    return got


# modes 1 and 2 (both axes, 32 x 32 regions) park a tile's rows in LDS two at a time, mode 0 (one axis) takes them from registers one by one
@pytest.mark.parametrize("pattern", ["quantize_cols_kernelILi.ELi.ELi%dE" % mode for mode in (0, 1, 2)] + ["quantize_backward_kernel"])
def test_column_wise_quantisers_use_the_rows_of_a_tile_in_the_order_they_are_loaded_in(pattern):
    """A wave's 32 loads, one per row, are waited for as their rows are used.  With a load of rows 0 .. 15 behind those of 16 .. 31 the wait for the
    first half of the rows, which are worked on while the second is on its way, is one for nearly all 32."""
    for name, code in named(pattern).items():
        tiles, loads, left = 0, 0, None  # left: the last wait's count, while a tile's are looked at
        for line in code:
            wait = re.match(r"s_waitcnt.*vmcnt\((\d+)\)", line)
            if line.startswith("global_load_dword "):
                loads = loads + 1 if left is None else 1
                left = None
            elif wait and (loads == 32 or left is not None):
                left, before, loads = int(wait.group(1)), 32 if left is None else left, 0
                assert 0 < before - left <= 2, (name, line)
                if left == 0:
                    tiles, left = tiles + 1, None
        assert tiles == (2 if "backward" in pattern else 1) and left is None, name
