"""Shapes of the sine-basis solver's transform passes, on the CPU.

A pass deals the work items of a strip of lines to the threads of a block: each
holds at most four items, each wave one or two pairs of product tiles, and the
folded strip lies in LDS. The host rules (csrc/sg_internal.h, printed by
tests/host_tiling/sine_passes.cpp, built with g++) are checked for every transform
length of the solver, alone and beside every longer one in a ragged launch: every
item is dealt exactly once, every product tile has a wave, and the strip fits."""

import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = "/opt/rocm"
BATCH = 4            # items a thread holds
LDS = 160 * 1024
MAX_NX = 1024


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(f"{ROCM}/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are missing")
    exe = str(tmp_path_factory.mktemp("sine") / "sine_passes")
    src = os.path.join(HERE, "host_tiling", "sine_passes.cpp")
    res = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                          f"-I{os.path.join(ROOT, 'include')}", "-o", exe, src], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]

    def run(cases):
        text = "".join(" ".join(map(str, c)) + "\n" for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return np.array([line.split() for line in out.splitlines()], dtype=np.int64)
    return run


def lengths(nx, parts):
    """Entries of each product's operand: wave numbers by parity, and of n_e = 2 H four ways."""
    if parts == 2:
        return [(nx + 1) // 2, nx // 2]
    H = (nx + 1) // 2
    return [H - H // 2, H // 2, H // 2, H - H // 2 - 1]


def dealt_along_x(threads, lines, items, log):
    """(row, item) places that the threads' first BATCH turns meet, with how often."""
    t = np.arange(threads)[:, None]
    u = np.arange(BATCH)[None, :]
    rstep = threads >> log
    rper = max(1, lines // rstep)
    chunk = u // rper
    r = (t >> log) + (u - chunk * rper) * rstep
    i = (t & ((1 << log) - 1)) + (chunk << log)
    ok = (r < lines) & (i < items)
    return np.bincount((r * items + i)[ok], minlength=lines * items)


def dealt_along_y(threads, lines, items):
    t = np.arange(threads)[:, None]
    u = np.arange(BATCH)[None, :]
    c, i = t % lines + 0 * u, t // lines + u * (threads // lines)
    ok = i < items
    return np.bincount((c * items + i)[ok], minlength=lines * items)


def check(case, row):
    nx, member, ragged, lines = case
    parts, nq, items, threads, per_wave, lds64, lds32, steps, served, mparts, mnq, fwd, inv, flog, ilog = row
    assert served == 1 and steps <= BATCH, case
    # the member's products: every entry of every part in a tile, every pair of tiles on a wave
    assert 16 * mnq >= max(lengths(member, mparts)) and sum(lengths(member, mparts)) == member, case
    assert mnq * mparts // 2 <= per_wave * (threads // 64), case
    # its folded strip, rows padded by 16 bytes and parts 128 bytes apart, in what the launch asks for
    for elem, lds in ((8, lds64), (4, lds32)):
        assert mparts * (lines * (16 * mnq + 16 // elem) * elem + 128) <= lds <= LDS, case
    return threads, lines, ((fwd, flog), (inv, ilog))


def test_every_length_alone_and_beside_longer_ones(shapes):
    cases = [(nx, nx, 0, lines) for nx in range(1, MAX_NX + 1) for lines in (16, 32)]
    cases += [(nx, m, 1, lines) for nx in range(1, MAX_NX + 1) for m in range(1, nx + 1, 1 if nx % 64 in (0, 1, 63) else 7)
              for lines in (16, 32)]
    rows = shapes(cases)
    assert len(rows) == len(cases)
    seen = set()
    for case, row in zip(cases, rows):
        if case[3] == 32 and row[2] > 16:
            continue  # longer transforms take strips of 16
        threads, lines, dealt = check(case, row)
        for items, log in dealt:
            if (threads, lines, items, log) in seen:
                continue
            seen.add((threads, lines, items, log))
            assert np.all(dealt_along_x(threads, lines, items, log) == 1), case
            assert np.all(dealt_along_y(threads, lines, items) == 1), case


def test_shapes_past_the_kernels_are_refused(shapes):
    """Strips of 32 lines of the longest transforms (LDS), and transforms longer than 32
    items of product tiles serve, are no launch."""
    rows = shapes([(1024, 1024, 0, 32), (1023, 1023, 0, 32), (1100, 1100, 0, 16), (2047, 2047, 0, 16), (1100, 64, 1, 16)])
    assert list(rows[:, 8]) == [0, 0, 0, 0, 0]
