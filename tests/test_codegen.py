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


class Line(str):
    """An instruction's text, with its address and that of the instruction it may branch to (None: no branch)."""


def instructions(listing):
    """Instructions of every function of an llvm-objdump listing, by mangled name."""
    found, lines, start = {}, None, 0
    for line in listing.splitlines():
        name = re.match(r"([0-9a-f]+) <(\w+)>:", line)
        if name:
            lines, start = found.setdefault(name.group(2), []), int(name.group(1), 16)
        elif lines is not None and line.startswith("\t") and "//" in line:
            text, _, rest = line.partition("//")
            ins = Line(text.strip())
            ins.address = int(rest.split(":")[0], 16)
            target = re.search(r"<\w+?(?:\+0x([0-9a-f]+))?>", rest) if "branch" in text else None
            ins.target = start + int(target.group(1) or "0", 16) if target else None
            lines.append(ins)
    return found


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
        found.update(instructions(subprocess.run([objdump, "-d", "--no-show-raw-insn", "/dev/stdin"], input=code,
                                                 capture_output=True, check=True).stdout.decode()))
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


# ---- the matrix instructions of the tiled GEMM kernels, which are inline assembly -----------------------------------------------

BEFORE = 2  # wait states between a vector instruction and the matrix instruction that reads its result
AFTER = 20  # ... between a matrix instruction and whatever touches its sums next (19, for one of 16 passes)


def registers(text):
    """Vector registers that an operand list names: ("v" or "a", number)."""
    got = set()
    for kind, one, first, last in re.findall(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        got |= {(kind, r) for r in (range(int(first), int(last) + 1) if last else [int(one)])}
    return got


def wait_states(line):
    return int(line.split()[1], 0) + 1 if line.startswith("s_nop") else 1


def unwaited(code):
    """Places of a kernel where the result of a vector instruction is read by a matrix instruction, or its sums by any other one, too early, on any path."""
    at = {line.address: i for i, line in enumerate(code)}
    follow = [([] if line.startswith(("s_branch", "s_endpgm", "s_setpc")) or i + 1 == len(code) else [i + 1]) +
              ([at[line.target]] if line.target is not None else []) for i, line in enumerate(code)]
    lead = [[] for _ in code]
    for i, to in enumerate(follow):
        for t in to:
            lead[t].append(i)
    wrong = []
    for i, line in enumerate(code):
        if not line.startswith("v_mfma"):
            continue
        ops = line.split(None, 1)[1].split(", ")
        sums, sources = registers(ops[0]), registers(ops[1]) | registers(ops[2]) | registers(" ".join(ops[4:]))
        todo = [(p, 0) for p in lead[i]]
        while todo:
            p, waited = todo.pop()
            if waited >= BEFORE:
                continue
            before = code[p]
            if before.startswith("v_") and not before.startswith("v_mfma"):
                written = before.split(None, 1)[1].split(", ")
                if sources & registers(" ".join(written[:2] if "swap" in before else written[:1])):
                    wrong.append((before, line))
            todo += [(q, waited + wait_states(before)) for q in lead[p]]
        todo = [(n, 0) for n in follow[i]]
        while todo:
            n, waited = todo.pop()
            if waited >= AFTER:
                continue
            after = code[n]
            if after.startswith(("v_", "ds_", "global_", "buffer_", "scratch_", "flat_")) and sums & registers(after):
                wrong.append((line, after))
            todo += [(q, waited + wait_states(after)) for q in follow[n]]
    return wrong


def listing(*lines):
    return instructions("0000 <k>:\n" + "".join("\t%s // %012X: 0\n" % (line, 4 * i) for i, line in enumerate(lines)))["k"]


MATRIX = "v_mfma_scale_f32_16x16x128_f8f6f4 a[4:7], v[8:11], v[12:15], a[4:7], v16, v17 op_sel:[1,0,0] cbsz:4 blgp:4"


@pytest.mark.parametrize("lines,sound", [
    (["v_mov_b32_e32 v16, v1", "s_nop 1", MATRIX], True),
    (["v_mov_b32_e32 v16, v1", "s_nop 0", MATRIX], False),
    (["v_permlane16_swap_b32_e32 v2, v12", "s_nop 0", MATRIX], False),
    (["v_mov_b32_e32 v1, v16", MATRIX], True),
    ([MATRIX, "s_nop 15", "s_nop 3", "v_accvgpr_read_b32 v0, a5"], True),
    ([MATRIX, "s_nop 15", "s_nop 2", "v_accvgpr_read_b32 v0, a5"], False),
    ([MATRIX, MATRIX], False),
])
def test_the_check_below_sees_a_missing_wait(lines, sound):
    assert (not unwaited(listing(*lines))) == sound


def test_tiled_gemm_matrix_instructions_stand_apart_from_what_they_depend_on():
    """In assembly the compiler does not keep the waits that the matrix unit needs: slots, and the copies a compiler may put at a change of stage body,
    decide.  Nothing is kept in scratch memory, whose loads would be such copies too."""
    for name, code in named("gemm_tile").items():
        assert sum(line.startswith("v_mfma_scale_f32_16x16x128") for line in code) >= 4 * 64, name
        assert not unwaited(code), name
        assert not any(line.startswith("scratch_") for line in code), name
