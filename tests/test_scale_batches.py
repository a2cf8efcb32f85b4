"""CPU-only check of the schedule (plain C++ constants) by which the ragged-shape kernel's 32 x 32 tiles refill their two scale buffers: no batch is
written while reads of the batch in its place may be on their way, and each is there before its first stage is read."""
import os
import shutil
import subprocess
import tempfile

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_09825_amd", "csrc")
BATCHES = 300


def barriers(per):
    """The barrier behind which each batch is written, as the kernel's header has it."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = '#include <stdio.h>\n#include "scale_batches.h"\nint main() { for (int b = 1; b < %d; ++b) printf("%%d %%d\\n", ' \
          'mxfp4::scale_batch_barrier(b, %d), mxfp4::scale_batch_drained(b, %d) && mxfp4::scale_batch_in_time(b, %d)); }\n'
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "a")
        subprocess.run([cxx, "-std=c++17", "-I", CSRC, "-x", "c++", "-", "-o", exe], input=src % (BATCHES, per, per, per),
                       text=True, check=True)
        return [tuple(map(int, l.split())) for l in subprocess.run([exe], capture_output=True, text=True).stdout.splitlines()]


@pytest.mark.parametrize("per", [8, 16])  # stages per batch: E2M1, E4M3
def test_no_batch_is_overwritten_while_it_is_read(per):
    written = barriers(per)
    assert len(written) == BATCHES - 1 and all(ok for _, ok in written)
    for b, (at, _) in enumerate(written, start=1):
        # behind barrier `at` and in front of barrier at + 1 the half b % 2 changes hands.  Stage t's reads are issued behind barrier t and
        # are known to have returned in front of barrier t + 2.
        for t in range((b - 2) * per, (b - 1) * per):
            assert t + 2 <= at
        for t in range(b * per, (b + 1) * per):
            assert at + 1 <= t
