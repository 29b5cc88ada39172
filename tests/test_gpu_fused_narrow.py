"""The fused kernel of narrow products in both orientations (rows of A or
columns of B as the long operand): at the least number of long vectors that
takes it and one fewer, ragged ends, every kind of moduli count (one limb up
to 13, two above, odd and even), against the separate kernels on every entry
and against the oracle on the first and last vectors."""
import numpy as np
import pytest

from oracle import ozaki2 as ref
from paper_2606_29129_amd import inputs
from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _bits_equal, _forced_unfused, _gpu_dgemm, _gpu_sgemm  # noqa: E402

LONG = 192 * 64


@pytest.mark.parametrize("across", [False, True])
@pytest.mark.parametrize("long,narrow,k,N,mode", [
    (LONG, 64, 64, 14, 0), (LONG + 1, 1, 63, 2, 0), (LONG + 63, 33, 65, 13, 1),
    (LONG - 1, 64, 40, 16, 0), (LONG + 130, 63, 200, 15, 3), (LONG + 5, 17, 129, 16, 1),
    (LONG, 5, 1, 7, 0), (LONG + 64, 32, 191, 12, 0)])
def test_equals_separate_kernels_and_oracle(long, narrow, k, N, mode, across):
    m, n = (narrow, long) if across else (long, narrow)
    A, B = inputs.problem(m, n, k, 1.0, seed=long + k)
    C = _gpu_dgemm(A, B, N, mode, lda=m + 1, ldb=k + 3, ldc=m + 2)
    assert _bits_equal(C, _forced_unfused(A, B, N, mode))
    which = (ref.REVISED, ref.ORIGINAL, None, ref.EXACT)[mode]
    pick = [0, 1, long - 1]
    if across:
        assert _bits_equal(C[:, pick], ref.gemm(A, B[:, pick], N, which)["C"])
    else:
        assert _bits_equal(C[pick], ref.gemm(A[pick], B, N, which)["C"])


@pytest.mark.parametrize("across", [False, True])
def test_flagged_vectors(across):
    m, n = (64, LONG) if across else (LONG, 64)
    A, B = inputs.problem(m, n, 100, 1.0, seed=5)
    A[3, 5], A[9, 7], A[9, 8], B[11, 4] = -np.inf, np.inf, np.nan, np.inf
    A[20] = 1e200 * np.sign(A[20])
    for N in (12, 14):
        C = _gpu_dgemm(A, B, N)
        assert np.isnan(C[[3, 9, 20]]).all() and np.isnan(C[:, 4]).all()
        assert _bits_equal(C, _forced_unfused(A, B, N))


@pytest.mark.parametrize("across", [False, True])
def test_binary32(across):
    m, n = (40, LONG + 3) if across else (LONG + 3, 40)
    A, B = (x.astype(np.float32) for x in inputs.problem(m, n, 150, 0.5, seed=6))
    C = _gpu_sgemm(A, B, 7)
    assert oz.ozaki2_set_tile(3) == 0
    try:
        want = _gpu_sgemm(A, B, 7)
    finally:
        oz.ozaki2_set_tile(0)
    assert np.array_equal(C.view(np.uint32), want.view(np.uint32))


def test_small_workspace_still_takes_a_narrow_b():
    """A workspace that holds only the fused kernel's regions (no residue
    planes of A) is enough for n <= 64 at any m, and the result is the same."""
    A, B = inputs.problem(900, 20, 500, 1.0, seed=8)
    want = _gpu_dgemm(A, B, 14)
    Ad, Bd = (torch.from_numpy(x.T.copy()).to("cuda:0") for x in (A, B))
    C = torch.empty((20, 900), dtype=torch.float64, device="cuda:0")
    ws = torch.empty(2 << 20, dtype=torch.uint8, device="cuda:0")
    at = (ws.data_ptr() + 255) // 256 * 256
    assert oz.ozaki2_workspace_size(900, 20, 500, 14) > (2 << 20)
    assert oz.ozaki2_set_workspace(at, (2 << 20) - 256) == 0
    try:
        assert oz.ozaki2_dgemm(900, 20, 500, Ad, 900, Bd, 500, C, 900, 14) == 0
        torch.cuda.synchronize()
    finally:
        oz.release_workspaces()
    assert _bits_equal(C.cpu().numpy().T, want)
