"""The host side of a sweep, compiled for the CPU with stand-ins for the kernels
(helpers/sweep_launches.cpp): every replica gets the half-sweeps of a sweep in order
and once, with the sweep's counter, and the end of the sweep reads the energies where
the last pass left them, whatever the route, the batches or the halves."""

import itertools
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm/include"
F32, F16, BF16, QANGLE = range(4)

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(ROCM), reason="needs g++ and HIP's headers")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launches") / "sweep_launches")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                           os.path.join(HERE, "helpers", "sweep_launches.cpp"), "-o", exe])

    def run(cases):
        """cases: (storage, n_hb, n_or, variant, batch, overlap, [(L, samples, copies, rungs, field), ...])"""
        lines = [" ".join(map(str, (*c[:6], 2, len(c[6]), *itertools.chain(*c[6])))) for c in cases]
        out = subprocess.run([exe], input="\n".join(lines) + "\n", text=True, capture_output=True, check=True)
        got = out.stdout.splitlines()
        assert len(got) == len(lines)
        return [(c, g) for c, g in zip(cases, got) if g != "ok"]
    return run


MIXES = [(1, 0), (1, 1), (1, 2), (1, 3), (1, 4), (2, 4), (0, 2)]


@pytest.mark.parametrize("storage", [F32, F16, BF16, QANGLE])
def test_one_size(check, storage):
    """Replica counts on both sides of the lines that the routes draw, whole, in batches
    with and without a remainder, and as halves of an even and an odd number of samples."""
    cases = []
    for L, reps in ((8, (3, 700)), (22, (5, 300)), (24, (2, 60, 130, 519, 1100)), (28, (60, 130, 520)),
                    (30, (60, 130, 300)), (32, (8, 70, 130, 519, 1030, 1600)), (36, (8, 100, 300)), (40, (60, 300)),
                    (48, (60, 300)), (62, (40, 260)), (64, (10, 100, 260)), (128, (1, 3))):
        for n, field, (n_hb, n_or), variant in itertools.product(reps, (0, 1), MIXES, (0, 3, 4, 5)):
            for batch in (-1, 0, 7, 50, 64):
                if 0 < batch < n and n // batch < 40:
                    cases.append((storage, n_hb, n_or, variant, batch, 0, [(L, 1, 1, n, field)] if n <= 256 else
                                  [(L, n, 1, 1, field)]))
                elif batch <= 0:
                    cases.append((storage, n_hb, n_or, variant, batch, 0, [(L, n, 1, 1, field)]))
            for samples in (2, 3):
                if 1 <= n // samples <= 256:
                    cases.append((storage, n_hb, n_or, variant, -1, 1, [(L, samples, 1, n // samples, field)]))
    assert len(cases) > 5000
    assert check(cases) == []


def test_several_sizes(check):
    """Sizes of several routes in one handle: two pairs at a time, one, single passes,
    gather passes and spins in LDS."""
    cases = []
    for storage, (n_hb, n_or), variant in itertools.product((F32, BF16, QANGLE), MIXES, (0, 1, 2, 3, 4, 5)):
        for batch, overlap in ((-1, 0), (0, 0), (20, 0), (64, 0), (-1, 1)):
            for sizes in ([(12, 3), (16, 3), (24, 40), (32, 70), (48, 9)], [(24, 3), (32, 300), (40, 50), (64, 20)],
                          [(30, 60), (32, 60), (36, 60)], [(8, 3), (18, 9), (30, 100)], [(24, 70), (28, 75), (32, 280)]):
                cases.append((storage, n_hb, n_or, variant, batch, overlap, [(L, 2, 1, n // 2 + 1, 0) for L, n in sizes]))
    assert check(cases) == []


def test_halves_in_effect(check):
    """Sizes with the spins in LDS beside sizes of the marches still sweep as two halves;
    halves of one and of two samples."""
    cases = []
    for storage, (n_hb, n_or), variant in itertools.product((F32, F16, QANGLE), MIXES, (0, 2, 3, 4, 5)):
        for sizes in ([(12, 2, 3), (16, 3, 3), (24, 2, 40), (48, 3, 9)], [(8, 2, 1), (32, 5, 100)], [(36, 2, 3)],
                      [(16, 2, 2), (20, 3, 30), (128, 2, 1)]):
            cases.append((storage, n_hb, n_or, variant, -1, 2, [(L, D, 1, T, 0) for L, D, T in sizes]))
    assert check(cases) == []


@pytest.mark.parametrize("storage", [F32, F16, QANGLE])
def test_sign_bits(check, storage):
    """Couplings of one sign bit draw the walk's lines elsewhere: replica counts on both
    sides of them, whole, in batches and as halves."""
    cases = []
    for L, n, field, (n_hb, n_or), batch in itertools.product(
            (36, 40, 48, 52, 56, 64), (190, 200, 224, 256, 260, 350, 352, 384, 400, 512, 640), (2, 3), MIXES, (-1, 64, 200)):
        if batch < n:
            cases.append((storage, n_hb, n_or, 0, batch, 0, [(L, n, 1, 1, field)]))
        if batch < 0:
            cases.append((storage, n_hb, n_or, 0, -1, 1, [(L, 4, 1, n // 4, field)]))
    assert check(cases) == []
