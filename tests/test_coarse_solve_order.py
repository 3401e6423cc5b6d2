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
    """{solve: [(order, converged, lost, iterations, residual, hash, reported residual)]}"""
    r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    got = {}
    for line in r.stdout.splitlines():
        order, solve, conv, lost, iters, res, h, told = line.split()
        got.setdefault(int(solve), []).append((order, int(conv), int(lost), int(iters), float(res), h, float(told)))
    return got


def _check(got, lost):
    assert sorted(got) == [0, 1, 2]          # extrapolated guess, the last solution as guess, given right-hand side
    history, want = {}, {}                   # a solve's bits depend on how it and those before it ended
    for solve in (0, 1, 2):
        for order, conv, gone, iters, res, h, _ in got[solve]:
            assert conv == 1 and gone in lost and iters < 40 and res <= 1e-13, (order, conv, gone, iters, res)
            history[order] = history.get(order, ()) + (gone,)
            assert h == want.setdefault(history[order], h), order


# one workgroup: part of a tile, a whole one
@pytest.mark.parametrize("M", [8, 16])
def test_wavefronts_of_a_workgroup(program, M):
    _check(_solves(program, M, 6, 1 << 22), lost=(0,))


# several: a last tile one node wide, nine tiles
@pytest.mark.parametrize("M", [17, 35])
def test_workgroups(program, M):
    _check(_solves(program, M, 6, 1 << 22), lost=(0,))


# A wait that gives up at once, after a few polls (some launches are given up in
# their first phases, some not) or in the last phases: every workgroup ends the
# same way, and a launch that is given up is solved by one workgroup.
@pytest.mark.parametrize("M,polls,lost", [(17, 0, (1,)), (35, 0, (1,)), (17, 1, (1,)), (17, 3, (0, 1)), (17, 5, (0, 1)),
                                          (17, 8, (0, 1)), (16, 0, (0,))])
def test_given_up(program, M, polls, lost):
    _check(_solves(program, M, 20, polls), lost)


def test_first_iterate_that_meets_the_tolerance(program):
    """On a matrix far from symmetric the residual rises now and then.  An iterate
    that meets the tolerance by less than a factor of two may be improved by one
    iteration more, and is the result if that makes it worse or runs out."""
    run = lambda k, tol: _solves(program, 8, 0, 1 << 22, k, repr(tol), 0.8)[2][0]  # noqa: E731
    res = [run(k, 0.0)[6] for k in range(16)]
    rises = [k for k in range(1, 15) if res[k + 1] > 1.3 * res[k] and min(res[:k]) > 1.3 * res[k]]
    assert rises
    for k in rises:
        tol = 1.2 * res[k]
        for most in (k, k + 1, 200):
            _, conv, _, iters, _, _, told = run(most, tol)
            assert (conv, iters, told) == (1, k, res[k]), (k, most)
    # the next iterate is better: it is the result, whatever follows
    falls = [k for k in range(1, 15) if res[k + 1] < 0.9 * res[k] and min(res[:k]) > 1.3 * res[k]]
    for k in falls:
        assert run(200, 1.2 * res[k])[1:4] == (1, 0, k + 1)
        assert run(k, 1.2 * res[k])[1:4] == (1, 0, k)
