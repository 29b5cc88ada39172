"""Which products scale and convert whole vectors in one kernel and which in
the separate ones, seen from whether the chunk sums of the norms are written
to the workspace; and the one kernel's stages on vectors of up to 4096
entries, where it still takes them."""
import numpy as np
import pytest

from oracle import complex as zref
from oracle import ozaki2 as ref
from paper_2606_29129_amd import inputs
from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _bits_equal, _gpu_dgemm, _gpu_stages  # noqa: E402

DEV = "cuda:0"
GEMM = {"float64": oz.ozaki2_dgemm, "float32": oz.ozaki2_sgemm, "complex128": oz.ozaki2_zgemm,
        "complex64": oz.ozaki2_cgemm}


@pytest.mark.parametrize("m,n,k,dtype,N,one", [
    (128, 128, 4096, "float64", 14, False), (128, 128, 2816, "float64", 14, True),
    (760, 16, 4096, "float64", 14, True), (740, 16, 2817, "float64", 9, False),
    (64, 4096, 4096, "float64", 14, False), (4096, 64, 4096, "float64", 14, False),
    (64, 4096, 3000, "float64", 14, True), (300, 4096, 4096, "float64", 14, True),
    (64, 11000, 4096, "float64", 18, True), (2000, 1000, 4096, "float64", 14, True),
    (128, 128, 4096, "float32", 7, False), (128, 128, 2304, "float32", 7, True),
    (1024, 64, 3071, "float32", 7, True), (1024, 64, 3072, "float32", 7, False),
    (2048, 64, 4096, "float32", 7, True), (64, 3072, 4096, "complex128", 14, False),
    (3072, 64, 4096, "complex128", 14, True), (128, 128, 4096, "complex64", 7, True),
    (200, 4000, 4096, "complex64", 7, False)])
def test_route(m, n, k, dtype, N, one):
    T, cplx = getattr(torch, dtype), dtype.startswith("complex")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(m + n + k)
    A = torch.randn(k, m, dtype=T, device=DEV, generator=gen)
    B = torch.randn(n, k, dtype=T, device=DEV, generator=gen)
    C = torch.empty(n, m, dtype=T, device=DEV)
    size = oz.ozaki2_zgemm_workspace_size if cplx else oz.ozaki2_workspace_size
    need = size(m, n, k, N, 0)
    ws = torch.full((need + 256,), 0xA5, dtype=torch.uint8, device=DEV)
    at = (ws.data_ptr() + 255) // 256 * 256 - ws.data_ptr()
    oz.ozaki2_set_stream(torch.cuda.current_stream())
    assert oz.ozaki2_set_workspace(ws.data_ptr() + at, need) == 0
    try:
        assert GEMM[dtype](m, n, k, A, m, B, k, C, m, N) == 0
        torch.cuda.synchronize()
    finally:
        oz.release_workspaces()
    # behind status, exponents and norms: the chunk sums of all vectors
    start = 256 + 4 * (m + n + 512) + 8 * (m + n) + 2048
    sums = 8 * ((2 * k if cplx else k) // 64) * (m + n)
    untouched = bool((ws[at + start:at + start + sums // 2] == 0xA5).all())
    assert untouched == one
    # the same entries by the oracle, from their rows and columns alone
    rows, cols = [0, m - 1], [0, n // 2, n - 1]
    a, b = A.T[rows].cpu().numpy(), B.T[:, cols].cpu().numpy()
    want = {"float64": ref.dgemm, "float32": ref.sgemm, "complex128": zref.zgemm,
            "complex64": zref.cgemm}[dtype](a, b, N)
    got = C.T[rows][:, cols].cpu().numpy()
    assert np.ascontiguousarray(got).tobytes() == np.ascontiguousarray(want).tobytes()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m,n,k,N", [(1030, 5, 4096, 14), (1025, 9, 4095, 9), (3, 1040, 3001, 17),
                                     (7, 1100, 4096, 12), (1025, 2, 2897, 20)])
def test_stages_of_long_vectors(m, n, k, N, mode):
    A, B = inputs.problem(m, n, k, 1.0, seed=m + k)
    rows, cols = sorted({0, m // 2, m - 1}), sorted({0, n // 2, n - 1})
    r = ref.gemm(A[rows], B[:, cols], N, mode)
    g = _gpu_stages(A, B, N, mode, N - 1)
    assert _bits_equal(g["SA"][rows], np.array(r["SA"]))
    assert _bits_equal(g["SB"][cols], np.array(r["SB"]))
    assert list(g["eA"][rows]) == r["e_rows"] and list(g["eB"][cols]) == r["e_cols"]
    for t in range(N):
        assert np.array_equal(g["RA"][t][rows], r["RA"][t]), f"RA plane {t}"
        assert np.array_equal(g["RB"][t][cols], r["RB"][t].T), f"RB plane {t}"
    C = _gpu_dgemm(A, B, N, mode, lda=m + 3, ldb=k + 5, ldc=m + 1)
    assert _bits_equal(C[np.ix_(rows, cols)], r["C"])
