"""Which narrow products the fused kernel takes (by the filled part of its
rounds and by k), seen from what a call leaves untouched of its workspace,
and its results at long k in both orientations."""
import numpy as np
import pytest

from oracle import ozaki2 as ref
from paper_2606_29129_amd import inputs
from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _bits_equal, _forced_unfused, _gpu_dgemm, _gpu_sgemm  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("across", [False, True])
@pytest.mark.parametrize("long,k,dtype,fused", [
    (8192, 4096, "float64", True), (8192, 1024, "float64", False),
    (8192, 3072, "float32", False), (8192, 6144, "float32", True),
    (10240, 1536, "float64", True), (12287, 256, "float64", False),
    (12288, 256, "float64", True), (16384, 64, "float64", True),
    (18432, 512, "float64", False), (18432, 2048, "float64", True),
    (20480, 1024, "float64", True), (24576, 64, "float64", True),
    (9216, 64, "float64", True), (9215, 64, "float64", False), (18432, 1024, "float64", True),
    (18432, 2048, "float32", True), (8192, 4096, "float32", True),
    (7168, 4096, "float64", True), (7100, 16384, "float64", False)])
def test_route(long, k, dtype, fused, across):
    """The separate kernels fill the residue planes of both operands; the
    fused one writes nothing in the upper half of their workspace."""
    narrow, N = 40, 8
    m, n = (narrow, long) if across else (long, narrow)
    T = getattr(torch, dtype)
    A = torch.randn(k, m, dtype=T, device=DEV)
    B = torch.randn(n, k, dtype=T, device=DEV)
    C = torch.empty(n, m, dtype=T, device=DEV)
    need = oz.ozaki2_workspace_size(m, n, k, N)
    ws = torch.full((need + 256,), 0xA5, dtype=torch.uint8, device=DEV)
    at = (ws.data_ptr() + 255) // 256 * 256 - ws.data_ptr()
    oz.ozaki2_set_stream(torch.cuda.current_stream())
    assert oz.ozaki2_set_workspace(ws.data_ptr() + at, need) == 0
    try:
        gemm = oz.ozaki2_dgemm if dtype == "float64" else oz.ozaki2_sgemm
        assert gemm(m, n, k, A, m, B, k, C, m, N) == 0
        torch.cuda.synchronize()
    finally:
        oz.release_workspaces()
    untouched = bool((ws[at + need // 2:] == 0xA5).all())
    assert untouched == fused


@pytest.mark.parametrize("across", [False, True])
@pytest.mark.parametrize("long,narrow,k,N,mode,phi", [
    (8200, 64, 4097, 14, 0, 4.0), (8192, 33, 4100, 16, 1, 1.0), (12290, 5, 8191, 9, 3, 0.5),
    (12288, 64, 3001, 15, 0, 1.0), (16384, 3, 2113, 2, 0, 2.0)])
def test_long_k_equals_separate_kernels_and_oracle(long, narrow, k, N, mode, phi, across):
    m, n = (narrow, long) if across else (long, narrow)
    rng = np.random.default_rng(long + k)
    A, B = (((rng.random(s) - 0.5) * np.exp(phi * rng.standard_normal(s)))
            for s in ((m, k), (k, n)))
    C = _gpu_dgemm(A, B, N, mode)
    assert _bits_equal(C, _forced_unfused(A, B, N, mode))
    which = (ref.REVISED, ref.ORIGINAL, None, ref.EXACT)[mode]
    pick, few = [0, long - 1], slice(0, 4)
    if across:
        assert _bits_equal(C[few][:, pick], ref.gemm(A[few], B[:, pick], N, which)["C"])
    else:
        assert _bits_equal(C[pick][:, few], ref.gemm(A[pick], B[:, few], N, which)["C"])


def _small_workspace(A, B, N, mode, single=False):
    """C of a narrow B with a workspace of which the separate kernels' layout
    is more than the call gets: the fused kernel at any number of rows."""
    m, k = A.shape
    n = B.shape[1]
    Kp, Np = (k + 127) // 128 * 128, 64
    # the planes of B, and per vector exponents, norms and their chunk sums
    room = N * Np * Kp + 64 * (m + 64 + n) * (k // 64 + 8) + (64 << 10)
    T = torch.float32 if single else torch.float64
    Ad, Bd = (torch.from_numpy(np.ascontiguousarray(X.T)).to(DEV) for X in (A, B))
    C = torch.empty((n, m), dtype=T, device=DEV)
    ws = torch.full((room + 256,), 0x5A, dtype=torch.uint8, device=DEV)
    at = (ws.data_ptr() + 255) // 256 * 256
    oz.ozaki2_set_stream(torch.cuda.current_stream())
    gemm = oz.ozaki2_sgemm if single else oz.ozaki2_dgemm
    used = None
    try:
        # the least power-of-two share of it that the call accepts
        for share in (64, 32, 16, 8, 4, 2, 1):
            assert oz.ozaki2_set_workspace(at, room // share // 256 * 256) == 0
            rc = gemm(m, n, k, Ad, m, Bd, k, C, m, N, mode)
            torch.cuda.synchronize()
            if rc == 0:
                used = room // share
                break
            assert rc == 2
    finally:
        oz.release_workspaces()
    assert used is not None and used < oz.ozaki2_workspace_size(m, n, k, N, mode)
    return C.cpu().numpy().T.copy()


@pytest.mark.parametrize("m,n,k,N,mode,phi", [
    (300, 64, 500, 14, 0, 1.0), (1000, 17, 4097, 14, 0, 0.5), (65, 1, 33, 2, 0, 2.0),
    (129, 63, 129, 16, 1, 1.0), (200, 40, 300, 9, 3, 4.0), (16, 64, 64, 12, 0, 1.0),
    (1, 5, 7, 5, 0, 1.0), (90, 64, 700, 15, 0, 1.0)])
def test_few_rows_through_a_small_workspace(m, n, k, N, mode, phi):
    A, B = inputs.problem(m, n, k, phi, seed=m + 3 * n + k)
    if m > 60 and n > 16:
        A[7, 3], A[9, 5], B[11, 4] = np.nan, -np.inf, np.inf
        A[20] = 1e200 * np.sign(A[20])
    C = _small_workspace(A, B, N, mode)
    assert _bits_equal(C, _forced_unfused(A, B, N, mode))
    which = (ref.REVISED, ref.ORIGINAL, None, ref.EXACT)[mode]
    rows = [i for i in range(m) if m <= 60 or n <= 16 or i not in (7, 9, 20)]
    cols = [j for j in range(n) if m <= 60 or n <= 16 or j != 4]
    assert _bits_equal(C[np.ix_(rows, cols)], ref.gemm(A[rows], B[:, cols], N, which)["C"])


def test_binary32_few_rows_through_a_small_workspace():
    A, B = (x.astype(np.float32) for x in inputs.problem(150, 48, 260, 1.0, seed=72))
    C = _small_workspace(A, B, 7, 0, single=True)
    assert np.array_equal(C.view(np.uint32), ref.sgemm(A, B, 7).view(np.uint32))
    assert np.array_equal(C.view(np.uint32), _gpu_sgemm(A, B, 7).view(np.uint32))
