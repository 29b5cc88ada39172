"""K4's per-entry arithmetic in the two forms of the kernels: the table's own
slice count (plain, complex and fused), and the batch's four slices for every
N, also where the table has fewer (CPU only; the library's header built for the
host, against the oracle's integers).  The values next to +-P/2 are the ones
whose quotient estimate can be off by one."""
import os
import random
import shutil
import struct
import subprocess
import tempfile
from fractions import Fraction

import pytest

from oracle import constants, fp, ozaki2 as ref
from test_k4_host import HIPCC, ROOT, _exponents, _values


@pytest.fixture(scope="module")
def driver():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tempfile.mkdtemp()
    exe = os.path.join(d, "k4_slices_host_driver")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17",
                           "-ffp-contract=off", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2606_29129_amd", "csrc"),
                           os.path.join(ROOT, "tests", "k4_slices_host_driver.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    yield exe
    shutil.rmtree(d, ignore_errors=True)


@pytest.mark.parametrize("N", range(2, 21))
def test_own_and_four_slices_for_every_table(driver, N):
    p, P, _, _ = constants.step1(N)
    rng = random.Random(2000 + N)
    near = [s * (P // 2 - d) for d in (1, 2, 3, P >> 60, P >> 52, P >> 48, P >> 40, P >> 30)
            for s in (1, -1) if 0 < d < P // 4]
    near += [s * (P // 2 - rng.randrange(1, max(2, P >> 48))) for _ in range(40) for s in (1, -1)]
    cases = [(v, E) for v in _values(rng, P, 60) + near for E in _exponents(rng, v)]
    text = "".join(f"{N} {E} " + " ".join(str(ref.residue(v, pt)) for pt in p) + "\n"
                   for v, E in cases)
    out = subprocess.run([driver], input=text, capture_output=True, text=True, check=True).stdout
    got = [int(x, 16) for x in out.split()]
    want = []
    for v, E in cases:
        one = struct.unpack("<Q", struct.pack("<d", fp.round_dyadic(v, -E, fp.BINARY64)))
        one += struct.unpack("<I", struct.pack("<f", fp.round_dyadic(v, -E, fp.BINARY32)))
        want += one + one
    assert len(got) == len(want)
    bad = [(cases[i // 4], i % 4, hex(g), hex(w))
           for i, (g, w) in enumerate(zip(got, want)) if g != w]
    assert not bad, (len(bad), bad[:4])


def test_fast_bound_is_just_below_half_of_P(driver):
    """The fast test accepts |C''| up to P/2 (1 - 2^-30): safely below P/2,
    and above what the scaling can leave (its binary32 constants stay about
    2^-21 below P/2, relatively), so that small k does not miss it."""
    out = subprocess.run([driver, "bounds"], capture_output=True, text=True, check=True).stdout
    got = [Fraction(float.fromhex(x.split()[0])) for x in out.splitlines()]
    assert len(got) == 19
    for N, b in zip(range(2, 21), got):
        P = constants.step1(N)[1]
        assert Fraction(P, 2) * (1 - Fraction(1, 2 ** 29)) < b
        assert b < Fraction(P, 2) * (1 - Fraction(1, 2 ** 31))


def test_fused_kernel_has_the_tables_slices(driver):
    """The fused kernel's compile-time slice count is the table's, on which
    its two-slice test rests."""
    out = subprocess.run([driver, "slices"], capture_output=True, text=True, check=True).stdout
    for N, line in zip(range(2, 21), out.splitlines()):
        _, table, fused = line.split()
        assert int(table) == -(-constants.step1(N)[1].bit_length() // 39)
        assert int(fused) == (int(table) if N <= 16 else 0)
