"""Static check of the generated gfx950 code of the two-step kernel: its lanes
read LDS columns that other lanes of the wavefront wrote, so between the LDS
writes of a row and the reads that follow them, and between those and the next
row's writes, the code must hold a point that the compiler moves no LDS
operation across (a wavefront barrier, which the listing shows as a comment).
The hardware runs a wavefront's LDS operations in order."""
import os
import re
import shutil
import subprocess

import pytest

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def unordered(lines):
    """Per pair kernel: (LDS writes, reads, places where one follows the other
    with no wavefront barrier between them)."""
    found, name, last, counts = {}, None, None, None
    for line in lines:
        m = re.match(r"^(_Z\w*lbm_pair_kernel\w*):", line)
        if m:
            name, last, counts = m.group(1), None, [0, 0, 0]
        if name is None:
            continue
        if line.startswith(".Lfunc_end"):
            found[name], name = tuple(counts), None
        elif "wave barrier" in line:
            last = None
        else:
            m = re.match(r"^\s*ds_(write|read)", line)
            if m:
                counts[0 if m.group(1) == "write" else 1] += 1
                counts[2] += last not in (None, m.group(1))
                last = m.group(1)
    return found


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None,
                    reason="needs hipcc")
def test_lds_operations_of_the_two_step_kernel_are_ordered(tmp_path):
    from paper_2408_15654_amd import build

    out = tmp_path / "lbm.s"
    subprocess.check_call([HIPCC, *build.FLAGS, "--offload-device-only", "-S", "-o", str(out),
                           build.SOURCES[0]], stderr=subprocess.DEVNULL)
    found = unordered(out.read_text().splitlines())
    assert len(found) == 16  # four storages, r != 1 or not, rho_A != rho_B or not
    for name, (writes, reads, bad) in found.items():
        assert writes and reads, name
        assert bad == 0, (name, writes, reads, bad)


def test_the_check_sees_a_missing_barrier():
    head, tail = ["_Z15lbm_pair_kernelv:"], [".Lfunc_end0:"]
    w, r, b = "\tds_write_b64 v1, v[2:3]", "\tds_read_b64 v[4:5], v1 offset:8", "\t; wave barrier"
    assert unordered(head + [w, b, r, b, w] + tail) == {"_Z15lbm_pair_kernelv": (2, 1, 0)}
    assert unordered(head + [w, r, b, w] + tail) == {"_Z15lbm_pair_kernelv": (2, 1, 1)}
    assert unordered(head + [w, b, r, w] + tail) == {"_Z15lbm_pair_kernelv": (2, 1, 1)}
