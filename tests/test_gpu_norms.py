"""The rounded-up squared norms of K1 against the oracle's exact rationals,
where directed rounding matters most: squares below the subnormals, subnormal
squares, sums next to a power of two, the largest finite squares and sums that
round up to infinity."""
import numpy as np
import pytest

from oracle import scaling

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _gpu_stages  # noqa: E402

KINDS = ("ordinary", "tiny", "subnormal", "boundary", "huge", "overflow")


def _vectors(kind, count, k, rng):
    x = rng.standard_normal((count, k))
    if kind == "tiny":            # squares from 2^-1200 to 2^-900
        x *= 2.0 ** rng.integers(-600, -450, (count, k))
    elif kind == "subnormal":     # entries themselves subnormal, or zero
        x = rng.integers(0, 5, (count, k)) * 2.0 ** -1074
    elif kind == "boundary":      # 2^52 + tiny squares: every addition is raised by one ulp
        x = np.full((count, k), 2.0 ** -40)
        x[:, 0] = 2.0 ** 26
    elif kind == "huge":          # squares up to 2^1020
        x = np.clip(x, -1, 1) * 2.0 ** 509
    elif kind == "overflow":      # the sum passes the largest finite number
        x = np.full((count, k), 2.0 ** 511)
        x[:, -1] = 2.0 ** 400
    return x


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("k", [1, 63, 64, 65, 200])
def test_squared_norms_round_up(kind, k):
    rng = np.random.default_rng(KINDS.index(kind) * 1000 + k)
    A = _vectors(kind, 5, k, rng)
    B = _vectors(kind, 3, k, rng).T.copy()
    got = _gpu_stages(A, B, 14, 0, 0)
    want_a = np.array([scaling.norm_sq_ru(r) for r in A], dtype=np.float64)
    want_b = np.array([scaling.norm_sq_ru(c) for c in B.T], dtype=np.float64)
    assert np.array_equal(got["SA"].view(np.uint64), want_a.view(np.uint64))
    assert np.array_equal(got["SB"].view(np.uint64), want_b.view(np.uint64))
