"""Batches whose problems lie on both sides of the longest k that scales and
converts whole vectors in one kernel (4096): the stages of the longer ones --
norms, folds, conversion -- in both fast modes, alone, mixed with shorter
ones, and replayed with other data; against single calls and the oracle."""
import numpy as np
import pytest

from oracle import ozaki2 as ref
from paper_2606_29129_amd import inputs
from paper_2606_29129_amd import ozaki2 as oz

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHORT = [(33, 70, 4096, 14), (130, 5, 64, 6), (1, 1, 4095, 20), (64, 129, 1000, 9)]
LONG = [(9, 65, 4097, 17), (70, 33, 6001, 14), (1, 3, 8192, 5), (129, 2, 4160, 20),
        (17, 64, 20011, 11)]


def _bits(x):
    return np.ascontiguousarray(x, dtype=np.float64).view(np.uint64)


@pytest.mark.parametrize("mode", ["revised", "original"])
@pytest.mark.parametrize("which", ["long", "short", "mixed"])
def test_long_and_short_problems(which, mode):
    shapes = {"long": LONG, "short": SHORT,
              "mixed": [s for pair in zip(LONG, SHORT) for s in pair] + LONG[4:]}[which]
    host = [inputs.problem(m, n, k, 0.5 + 0.4 * i, seed=70 + i)
            for i, (m, n, k, _) in enumerate(shapes)]
    Ns = [N for _, _, _, N in shapes]
    pairs = [tuple(torch.from_numpy(x).to(DEV) for x in p) for p in host]
    other = [(a * 0.75, b * -2.5) for a, b in pairs]
    for batch in (pairs, other, pairs):        # the later ones replay the graph
        outs = oz.dgemm_batched(batch, Ns, mode=mode)
        torch.cuda.synchronize()
        for (a, b), N, C in zip(batch, Ns, outs):
            single = oz.dgemm(a, b, N=N, mode=mode)
            assert np.array_equal(_bits(C.cpu().numpy()), _bits(single.cpu().numpy()))
    for (A, B), N, C in zip(host, Ns, outs):
        r, c = sorted({0, A.shape[0] - 1}), sorted({0, B.shape[1] - 1})
        # the conveniences' row-major product is the transposed one
        want = ref.gemm(np.ascontiguousarray(B[:, c].T), np.ascontiguousarray(A[r].T), N,
                        ref.REVISED if mode == "revised" else ref.ORIGINAL)["C"].T
        assert np.array_equal(_bits(C.cpu().numpy()[np.ix_(r, c)]), _bits(want))


def test_flagged_vectors_of_a_long_problem():
    A, B = inputs.problem(20, 30, 5000, 1.0, seed=81)
    C, D = inputs.problem(20, 30, 300, 1.0, seed=82)
    A[3, 4999], B[0, 7] = np.nan, np.inf
    pairs = [tuple(torch.from_numpy(x).to(DEV) for x in p) for p in ((A, B), (C, D))]
    oz.ozaki2_get_device_status()                       # clear
    X, Y = (x.cpu().numpy() for x in oz.dgemm_batched(pairs, [14, 14]))
    assert oz.ozaki2_get_device_status() == 1
    assert np.isnan(X[3]).all() and np.isnan(X[:, 7]).all() and np.isfinite(Y).all()
    rows, cols = [i for i in range(20) if i != 3], [j for j in range(30) if j != 7]
    assert np.isfinite(X[np.ix_(rows, cols)]).all()
    assert np.array_equal(_bits(X[rows]), _bits(oz.dgemm(*pairs[0], N=14).cpu().numpy()[rows]))
