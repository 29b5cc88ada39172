"""The kernel that scales and converts whole vectors (norms, exponents and
residues in one) at the edges of its tiles: vectors per block and per wave,
blocks of k, the chunks of the norm, and both sides of the longest k it takes;
stage by stage and in C against the oracle, bit for bit."""
import numpy as np
import pytest

from oracle import ozaki2 as ref
from paper_2606_29129_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _bits_equal, _gpu_dgemm, _gpu_sgemm, _gpu_stages  # noqa: E402

SHAPES = [(1, 9, 1), (8, 65, 63), (9, 7, 64), (17, 64, 127), (63, 33, 128), (65, 8, 129),
          (130, 3, 255), (7, 129, 257), (16, 5, 1023), (5, 17, 1025), (3, 2, 4095), (2, 9, 4096),
          (9, 3, 4097)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_stages_and_result(m, n, k, mode):
    N = 8 + (m + n + k) % 13
    A, B = inputs.problem(m, n, k, 1.0, seed=m + k)
    r = ref.gemm(A, B, N, mode)
    g = _gpu_stages(A, B, N, mode, N - 1)
    assert _bits_equal(g["SA"], np.array(r["SA"])) and _bits_equal(g["SB"], np.array(r["SB"]))
    assert list(g["eA"]) == r["e_rows"] and list(g["eB"]) == r["e_cols"]
    for t in range(N):
        assert np.array_equal(g["RA"][t], r["RA"][t]), f"RA plane {t}"
        assert np.array_equal(g["RB"][t], r["RB"][t].T), f"RB plane {t}"
    assert _bits_equal(_gpu_dgemm(A, B, N, mode, lda=m + 3, ldb=k + 5, ldc=m + 1), r["C"])


@pytest.mark.parametrize("m,n,k", [(1, 33, 60), (17, 64, 64), (33, 15, 130), (65, 7, 1100)])
def test_binary32_operands(m, n, k):
    A, B = (x.astype(np.float32) for x in inputs.problem(m, n, k, 0.5, seed=k))
    want = ref.sgemm(A, B, 7)
    assert np.array_equal(_gpu_sgemm(A, B, 7).view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m,n,k,single", [
    (1, 5, 1, False), (5, 33, 31, False), (33, 4, 32, True), (3, 65, 127, True),
    (65, 31, 128, False), (9, 7, 129, True), (4, 3, 1025, False), (2, 3, 4096, False),
    (3, 2, 4097, True)])
def test_complex_operands(m, n, k, single, mode):
    """Complex operands through the same kernel: blocks of 128 entries, norms
    over 2k components, three components' planes."""
    from oracle import complex as zref
    from test_gpu_complex import _gpu, _same
    N = 6 if single else 9 + (m + k) % 12
    A, B = inputs.complex_problem(m, n, k, 1.0, seed=m + k)
    if single:
        A, B = A.astype(np.complex64), B.astype(np.complex64)
    want = (zref.cgemm if single else zref.zgemm)(A, B, N, mode)
    assert _same(_gpu(A, B, N, mode, lda=m + 2, ldb=k + 1, ldc=m + 3, single=single), want)
