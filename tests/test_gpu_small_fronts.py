"""Sweeps of the small fronts as a batch of dense systems, one front each: few of
them (a workgroup a front in the backward sweep) and more than 512 (a wave each),
one right-hand side and the sixteen that make the sub-panels' inverses, in either
order on one factor.  Reference: numpy's dense solve."""
import numpy as np
import pytest

from paper_2510_05885_amd import ncl_kkt as nk
from paper_2510_05885_amd import synth

from gpu_util import colmajor, dev

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 79, 80, 81, 96, 97, 112, 113, 127, 128]


def _system(n, rng):
    A = rng.standard_normal((n, n))
    A = A + A.T + 4.0 * n * np.eye(n)       # diagonally dominant: condition number below 10
    colptr = np.concatenate([[0], np.cumsum(np.arange(n, 0, -1))]).astype(np.int32)
    rowidx = np.concatenate([np.arange(j, n) for j in range(n)]).astype(np.int32)
    vals = np.concatenate([A[j:, j] for j in range(n)])
    inp = synth.KKTInput(n, 0, colptr, rowidx, vals, np.zeros(n), np.zeros(1, np.int32), np.zeros(0, np.int32),
                         np.zeros(0), 1.0)
    return inp, A


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("sizes", [EDGES, [3 + k % 30 for k in range(520)]], ids=["few", "many"])
@pytest.mark.parametrize("columns", [(1, 16), (16, 1), (3,)], ids=["1-16", "16-1", "3"])
def test_batch_of_dense_fronts(sizes, columns, precision):
    rng = np.random.default_rng(11)
    systems = [_system(n, rng) for n in sizes]
    inps = [i for i, _ in systems]
    kkt = nk.KKT.analyze_batched(inps, precision=precision, ordering="natural")
    kkt.factor(dev(np.concatenate([i.W_val for i in inps])), dev(np.concatenate([i.Sigma for i in inps])), None,
               np.ones(len(inps)))
    off = np.concatenate([[0], np.cumsum(sizes)])
    for nrhs in columns:
        B = synth.rhs(int(off[-1]), nrhs, seed=nrhs).reshape(int(off[-1]), nrhs)
        X, _ = kkt.solve(colmajor(B))
        X = X.cpu().numpy().reshape(B.shape)
        for k, (_, A) in enumerate(systems):
            ref = np.linalg.solve(A, B[off[k]:off[k + 1]])
            # refined to a normwise backward error of 1e-12 at a condition number below 10
            assert np.abs(X[off[k]:off[k + 1]] - ref).max() <= 1e-10 * np.abs(ref).max()
    kkt.close()
