"""Order of the LDS exchanges within a wave, from the compiled device code (CPU).

The transforms inside a block (columns of at most 64 rows) pass data between the
lanes of one wave through LDS without a block barrier: staged rows to the fold,
the fold to the products, the products' reads to the unfolded results that take
their places, and, towards the grid, the results to the last sums. The hardware
keeps a wave's LDS accesses in order, but the compiler may swap a lane's write
and its read of another place unless a fence stands between them. Every such
transform has to state those fences, three one way and four the other."""

import os
import re
import shutil
import subprocess

import pytest


def test_transforms_inside_a_block_are_fenced():
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not found")
    from paper_1205_1864_amd import build as bld
    cmd = [bld.hipcc(), *bld.COMMON, "-x", "hip", "--cuda-device-only", "-S", "-emit-llvm", "-o", "-",
           os.path.join(bld.CSRC, "k_sine.hip")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    fused = 0
    for body in re.split(r"^define ", res.stdout, flags=re.M)[1:]:
        m = re.search(r"@(\S*sine_pcg_kernelI[df]Li\d+ELb0ELb1E\w*)\(", body.split("\n", 1)[0])
        if not m:
            continue
        fused += 1
        body = body.split("\n}", 1)[0]
        fences = len(re.findall(r'fence syncscope\("wavefront"\) acq_rel', body))
        barriers = len(re.findall(r"call void @llvm\.amdgcn\.wave\.barrier", body))
        # two directions of the right-hand side, the warm guess and the solution, rows and columns each
        assert fences >= 2 * 3 + 2 * 3 + 2 * 4 and barriers >= fences, (m.group(1), fences, barriers)
    assert fused == 4, "one-launch kernels of two sizes in two precisions"
