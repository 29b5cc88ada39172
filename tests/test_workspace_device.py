"""ensure_workspace takes CUDA devices only (CPU only: refused before anything
touches a GPU)."""
import pytest

from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("device", ["cpu", torch.device("cpu"), "meta"])
def test_other_devices_are_refused(device):
    before = dict(oz._workspaces)
    with pytest.raises(ValueError):
        oz.ensure_workspace(1024, device)
    assert oz._workspaces == before
