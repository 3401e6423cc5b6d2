"""The one-launch coarse solve's own source on the CPU (tests/emulated), its
wavefronts in chosen orders: lowest first, highest first, one workgroup or one
wavefront of each only when nothing else can go on, random.  No order may change a
bit of the solution, which must leave the residual that the solve stops at: 1e-14
of the right-hand side by its recurrence, which differs from the true one by the
roundings of some twenty products of 49 terms (1e-13 in all)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_02708_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which(CLANG) or os.uname().machine != "x86_64":
        pytest.skip("needs ROCm's clang++ on x86-64")
    d = tmp_path_factory.mktemp("solve")
    src = open(os.path.join(CSRC, "coarse_solve.hip")).read()
    # gfx950 instructions in inline asm: waits, which the emulation does not need
    (d / "kernel.inc").write_text(re.sub(r"asm volatile\([^;]*;", "", src))
    exe = str(d / "solve")
    emulated = os.path.join(ROOT, "tests", "emulated")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-w", f'-DKERNEL="{d}/kernel.inc"', "-I", emulated,
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe, os.path.join(emulated, "solve.cpp")],
                   check=True)
    return exe


def _solves(exe, *args):
    """{solve: [(order, converged, lost, iterations, residual, hash)]}"""
    r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    got = {}
    for line in r.stdout.splitlines():
        order, solve, conv, lost, iters, res, h = line.split()
        got.setdefault(int(solve), []).append((order, int(conv), int(lost), int(iters), float(res), h))
    return got


def _same_in_every_order(got):
    assert sorted(got) == [0, 1, 2]          # extrapolated guess, the last solution as guess, given right-hand side
    for runs in got.values():
        for order, conv, lost, iters, res, h in runs:
            assert conv == 1 and lost == 0 and iters < 40 and res <= 1e-13, (order, conv, lost, iters, res)
            assert h == runs[0][-1], order


# one workgroup: part of a tile, a whole one
@pytest.mark.parametrize("M", [8, 16])
def test_wavefronts_of_a_workgroup(program, M):
    _same_in_every_order(_solves(program, M, 6))


# several: a last tile one node wide, nine tiles
@pytest.mark.parametrize("M", [17, 35])
def test_workgroups(program, M):
    _same_in_every_order(_solves(program, M, 6))
