"""The library's own workspace (the opt-in policy) and narrow products: a
narrow B takes what the fused kernel needs, not the residue planes of A, and
gives the same bits once a larger workspace is there."""
import pytest

from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("mode", [0, 3])
def test_narrow_b_does_not_grow_the_workspace_to_the_planes_of_a(mode):
    m, n, k, N = 4096, 64, 16384, 14
    full = oz.ozaki2_workspace_size(m, n, k, N, mode)
    assert full > 800 << 20
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    A = torch.randn(k, m, dtype=torch.float64, device=DEV, generator=gen)     # column-major m x k
    B = torch.randn(n, k, dtype=torch.float64, device=DEV, generator=gen)
    C = [torch.empty(n, m, dtype=torch.float64, device=DEV) for _ in range(2)]

    def run(out):
        oz.ozaki2_set_stream(torch.cuda.current_stream())
        assert oz.ozaki2_dgemm(m, n, k, A, m, B, k, out, m, N, mode) == 0
        torch.cuda.synchronize()

    oz.release_workspaces()
    oz.ozaki2_finalize()                    # frees what earlier calls had grown
    assert oz.ozaki2_set_workspace_policy(oz.WORKSPACE_LIBRARY) == 0
    try:
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        run(C[0])
        # the planes of B (14.7 MB) and some vectors, not those of A (940 MB)
        assert free - torch.cuda.mem_get_info()[0] < 100 << 20
        oz.ensure_workspace(full)
        run(C[1])
    finally:
        oz.ozaki2_set_workspace_policy(oz.WORKSPACE_CALLER)
        oz.release_workspaces()
        oz.ozaki2_finalize()
    assert torch.equal(C[0], C[1])
