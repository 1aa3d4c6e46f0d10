"""Register budget of the inner solver in the sine basis and of the lognormal block
solves, from the compiler's resource report (CPU): both keep a column's state in
registers for the whole solve, and their comments say what spills."""

import os
import re
import shutil

import pytest

from test_kernel_resources import _report

# kernel name pattern -> (max VGPR spills, max scratch bytes per lane)
BUDGET = {
    "k_sine.hip": {
        r"sine_pcg_kernelI[df]Li(2|5|8|11|14|18|23)E": (0, 0),
        r"sine_pcg_kernelI[df]Li27E": (8, 32),
        r"sine_[xy]_kernel": (0, 0),
    },
    "k_logn.hip": {
        r"logn_solve_kernelILi64E": (0, 0),
        r"logn_solve_kernelILi512ELi(2|8|20)E": (0, 0),
        r"logn_solve_kernelILi512ELi38E": (300, 620),
    },
}


@pytest.mark.parametrize("src", sorted(BUDGET))
def test_solver_kernels_within_register_budget(src):
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not found")
    kernels = _report(src)
    for pat, (max_spill, max_scratch) in BUDGET[src].items():
        hits = [k for k in kernels if re.search(pat, k)]
        assert hits, f"no kernel matches {pat}"
        for k in hits:
            r = kernels[k]
            assert r.get("VGPRs Spill", 0) <= max_spill and r.get("ScratchSize", 0) <= max_scratch, (k, r)
