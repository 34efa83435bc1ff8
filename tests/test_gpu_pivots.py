"""Sub-panels of the dense factorization with and without replaced pivots:
one dense front whose rows at chosen positions are stored but zero, so that
the pivot there is exactly zero and the static-pivot rule replaces it, in
fronts of every path (one wave, LDS with one and two rows per lane, panels
with full and ragged last panels).  Reference: numpy's dense solve of the
remaining rows."""
import numpy as np
import pytest

from paper_2510_05885_amd import ncl_kkt as nk
from paper_2510_05885_amd import synth

from gpu_util import colmajor, dev

pytestmark = pytest.mark.gpu


def _dense_input(n, zeros, seed=3):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((n, n))
    A = A + A.T + 4.0 * n * np.eye(n)       # diagonally dominant: condition number below 10
    A[zeros, :] = 0.0
    A[:, zeros] = 0.0
    colptr = np.concatenate([[0], np.cumsum(np.arange(n, 0, -1))]).astype(np.int32)
    rowidx = np.concatenate([np.arange(j, n) for j in range(n)]).astype(np.int32)
    vals = np.concatenate([A[j:, j] for j in range(n)])
    inp = synth.KKTInput(n, 0, colptr, rowidx, vals, np.zeros(n), np.zeros(1, np.int32), np.zeros(0, np.int32),
                         np.zeros(0), 1.0)
    return inp, A


# orders at the edges of the paths: one wave (<= 32), one row per lane (<= 64),
# two (<= 128), then panels of 64: a lone one of each 16-column remainder, ragged last ones
SIZES = [1, 16, 17, 32, 33, 64, 65, 80, 81, 97, 128, 129, 145, 160, 176, 192, 193, 209, 320, 335]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("with_zeros", [False, True])
def test_dense_front_subpanels(n, precision, with_zeros):
    zeros = sorted({k for k in (0, 15, 16, 63, 64, 100, 127, 128, 200, n - 1) if k < n and n > 1}) if with_zeros else []
    inp, A = _dense_input(n, zeros)
    kkt = nk.KKT.from_input(inp, precision=precision, ordering="natural")
    rc = kkt.factor(dev(inp.W_val), dev(inp.Sigma), None, 1.0)
    keep = np.setdiff1d(np.arange(n), zeros)
    B = synth.rhs(n, 2, seed=n)
    B[zeros] = 0.0
    X, info = kkt.solve(colmajor(B))
    X = X.cpu().numpy()
    assert rc == 0 and kkt.inertia() == (n, 0, 0, len(zeros))
    ref = np.zeros_like(B)
    ref[keep] = np.linalg.solve(A[np.ix_(keep, keep)], B[keep])
    # refined to a normwise backward error of 1e-12 at a condition number below 10
    assert np.abs(X - ref).max() <= 1e-11 * np.abs(ref).max()
    assert not X[zeros].any()
    kkt.close()
