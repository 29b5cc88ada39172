"""The non-finite status of the fast modes with k <= 4096, where the CRT
kernel sets it: reported for a flagged row or column wherever it lies, for
outputs of one block and of many, and not at the cost of the call."""
import numpy as np
import pytest

from paper_2606_29129_amd import inputs
from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
GEMM = {"float64": oz.dgemm, "float32": oz.sgemm, "complex128": oz.zgemm, "complex64": oz.cgemm}


@pytest.mark.parametrize("dtype", list(GEMM))
@pytest.mark.parametrize("m,n", [(1, 1), (33, 70), (1500, 1501)])
def test_any_flagged_row_or_column_is_reported(m, n, dtype):
    k, cplx = 40, dtype.startswith("complex")
    A, B = (inputs.complex_problem if cplx else inputs.problem)(m, n, k, 0.5, seed=m + n)
    A, B = (torch.from_numpy(x.astype(dtype)).to(DEV) for x in (A, B))
    oz.ozaki2_get_device_status()                       # clear
    clean = GEMM[dtype](A, B, N=8)
    assert oz.ozaki2_get_device_status() == 0
    for row, col in {(0, None), (m - 1, None), (m // 2, None), (None, 0), (None, n - 1),
                     (None, n // 2)}:
        A1, B1 = A.clone(), B.clone()
        if row is not None:
            A1[row, k - 1] = float("nan")
        else:
            B1[3, col] = float("inf")
        C = GEMM[dtype](A1, B1, N=8)
        assert oz.ozaki2_get_device_status() == 1, (row, col)
        assert oz.ozaki2_get_device_status() == 0
        want = clean.clone()
        if row is not None:
            want[row] = complex(np.nan, np.nan) if cplx else np.nan
        else:
            want[:, col] = complex(np.nan, np.nan) if cplx else np.nan
        got, want = (torch.view_as_real(x) if cplx else x for x in (C, want))
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        assert torch.equal(torch.nan_to_num(got), torch.nan_to_num(want))


@pytest.mark.parametrize("dtype", ["float64", "complex128"])
def test_flagged_products_cost_no_more(dtype):
    """A product of NaNs runs the same kernels over the same bytes as a finite
    one: within twice its time (it took 13 and 4 times with one status update
    per output)."""
    A = torch.randn(4096, 256, dtype=torch.float64, device=DEV).to(getattr(torch, dtype))
    B = torch.randn(256, 4096, dtype=torch.float64, device=DEV).to(getattr(torch, dtype))

    def time(A, B):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = float("inf")
        for _ in range(5):
            ev[0].record()
            GEMM[dtype](A, B, N=14)
            ev[1].record()
            torch.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]))
        return best

    finite = time(A, B)
    assert time(torch.full_like(A, float("nan")), B) < 2 * finite
    oz.ozaki2_get_device_status()                       # clear
