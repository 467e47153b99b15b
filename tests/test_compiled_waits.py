"""The wait counts of the backward products, checked on their compiled code:
vector-memory operations complete in order, so a copy into LDS has landed only
once a wait leaves fewer operations in flight than were issued after it.  Which
loads the compiler puts between the copies is not fixed by the source."""
import re
import subprocess

import pytest

from paper_2601_14327_amd import build

DW_D_ON_LOAD = "gemm_bwd_kernelILi256ELi256ELi2ELi4ELi3ELb1ELb0ELb1E"  # dW_d, dY formed on load


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "gemm_bwd.s"
    subprocess.run([build._hipcc(), "-x", "hip", *build.COMMON, *build.HIP_FLAGS,
                    "--cuda-device-only", "-S", f"{build.CSRC}/gemm_bwd.hip", "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL, timeout=300)
    return out.read_text().splitlines()


def _body(asm, name):
    start = next(i for i, l in enumerate(asm) if l.startswith("_Z") and name in l)
    end = next(i for i in range(start, len(asm)) if asm[i].startswith(".Lfunc_end"))
    return [l.split(";")[0].strip() for l in asm[start:end]]


def test_on_load_chunks_are_read_after_their_copies(asm):
    """dW_d with dY formed on load: a thread scales its own copied chunks in
    place, ds_read_b128 (the fragments are read by ds_read_b64_tr).  Of the 16
    copies before the loop (A and B of step 0, A and B of step 1, four each) the
    first twelve have landed at the loop's first such read, all at its first
    barrier."""
    body = _body(asm, DW_D_ON_LOAD)
    flight, copies, reads, barriers = [], 0, 0, 0
    for l in body:
        wait = re.match(r"s_waitcnt .*?vmcnt\((\d+)\)", l)
        if wait:
            flight = flight[max(0, len(flight) - int(wait[1])):]
        elif re.match(r"(buffer|global|flat)_(load|store|atomic)", l):
            copy = l.startswith("buffer_load") and l.endswith("lds")
            flight.append(copies if copy else None)
            copies += copy
        elif l.startswith("ds_read_b128"):
            reads += 1
            landed = 4 if reads <= 4 else 12   # step 0's own chunks, then step 1's
            assert not [c for c in flight if c is not None and c < landed], (reads, flight)
        elif l == "s_barrier":
            barriers += 1
            assert not [c for c in flight if c is not None and c < (8 if barriers == 1 else 16)]
            if barriers == 2:
                break
    assert copies == 20 and reads == 8 and barriers == 2   # (A of step 2 in the loop)
