"""The wait counts of the backward products, checked on their compiled code:
vector-memory operations complete in order, so a copy into LDS has landed only
once a wait leaves fewer operations in flight than were issued after it.  Which
loads the compiler puts between the copies is not fixed by the source."""
import re
import subprocess

import pytest

from paper_2601_14327_amd import build

WGRAD = "gemm_bwd_kernelILi256ELi256ELi2ELi4ELi3ELb1E"
DW_GIVEN, DW_GATHERED, DW_D_ON_LOAD = WGRAD + "Lb0ELb0E", WGRAD + "Lb1ELb0E", WGRAD + "Lb0ELb1E"


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


@pytest.mark.parametrize("kernel", [DW_GIVEN, DW_GATHERED, DW_D_ON_LOAD])
def test_weight_gradient_halves_land_before_their_barrier(asm, kernel):
    """Of the 16 copies before the loop (A and B of step 0, A and B of step 1, four
    each) the first eight have landed at the barrier ahead of the loop, all at the
    loop's first.  dW_d with dY formed on load also scales each thread's own copied
    chunks in place, read by ds_read_b128 (fragments by ds_read_b64_tr): those of
    step 0 ahead of the loop, those of step 1 in its first iteration."""
    flight, copies, reads, barriers = [], 0, 0, 0
    for l in _body(asm, kernel):
        wait = re.match(r"s_waitcnt .*?vmcnt\((\d+)\)", l)
        if wait:
            flight = flight[max(0, len(flight) - int(wait[1])):]
        elif re.match(r"(buffer|global|flat)_(load|store|atomic)", l):
            copy = l.startswith("buffer_load") and l.endswith("lds")
            flight.append(copies if copy else None)
            copies += copy
        elif l.startswith("ds_read_b128"):
            reads += 1
            landed = 4 if reads <= 4 else 12
            assert not [c for c in flight if c is not None and c < landed], (reads, flight)
        elif l == "s_barrier":
            barriers += 1
            assert not [c for c in flight if c is not None and c < (8 if barriers == 1 else 16)]
            if barriers == 2:
                break
    assert copies == 20 and barriers == 2   # (A of step 2 in the loop)
    assert reads == (8 if kernel == DW_D_ON_LOAD else 0)
