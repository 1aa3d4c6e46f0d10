"""What waves and blocks agree on, from the compiled device code (CPU): the order of
the LDS exchanges within a wave, and one decision per block on a shared status.

The transforms inside a block (columns of at most 64 rows) pass data between the
lanes of one wave through LDS without a block barrier: staged rows to the fold,
the fold to the products, the products' reads to the unfolded results that take
their places, and, towards the grid, the results to the last sums. The hardware
keeps a wave's LDS accesses in order, but the compiler may swap a lane's write
and its read of another place unless a fence stands between them. Every such
transform has to state those fences, three one way and four the other.

The one-launch block solves of the lognormal path give up where another block has.
That status may be set at any time, so a block has to settle it between two barriers:
were every wave to read it at the start and leave, some would go and the rest would
run on without their rows."""

import os
import re
import shutil
import subprocess

import pytest


def _kernels(src, pattern):
    """(name, device code) of the kernels of a source whose names match."""
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not found")
    from paper_1205_1864_amd import build as bld
    cmd = [bld.hipcc(), *bld.COMMON, "-x", "hip", "--cuda-device-only", "-S", "-emit-llvm", "-o", "-",
           os.path.join(bld.CSRC, src)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    out = []
    for body in re.split(r"^define ", res.stdout, flags=re.M)[1:]:
        m = re.search(r"@(\S*" + pattern + r"\w*)\(", body.split("\n", 1)[0])
        if m:
            out.append((m.group(1), body.split("\n}", 1)[0]))
    return out


def test_transforms_inside_a_block_are_fenced():
    kernels = _kernels("k_sine.hip", r"sine_pcg_kernelI[df]Li\d+ELb0ELb1E")
    assert len(kernels) == 4, "one-launch kernels of two sizes in two precisions"
    for name, body in kernels:
        fences = len(re.findall(r'fence syncscope\("wavefront"\) acq_rel', body))
        barriers = len(re.findall(r"call void @llvm\.amdgcn\.wave\.barrier", body))
        # two directions of the right-hand side, the warm guess and the solution, rows and columns each
        assert fences >= 2 * 3 + 2 * 3 + 2 * 4 and barriers >= fences, (name, fences, barriers)


def test_block_solves_decide_once_per_block():
    kernels = _kernels("k_logn.hip", "logn_solve_kernelI")
    assert len(kernels) == 9
    for name, body in kernels:
        entry = body.split("{", 1)[1].split("\n\n", 1)[0]  # up to the first branch, which every lane runs
        loads = re.findall(r"(%\w+) = load atomic", entry)
        tests = [t for v in loads for t in re.findall(r"(%\w+) = icmp \w+ i64 " + re.escape(v) + r",", body)]
        assert len(loads) <= 1, (name, loads)
        for t in tests:
            assert not re.search(r"br i1 " + re.escape(t) + r"\b", body), f"{name}: waves leave by themselves"
