"""Static pivots of the dual block inside fronts of every size, and the block rule's own thresholds.  A row of J
whose stored values are zero keeps its pivot at -1/rho whatever was eliminated before it, in the middle of a front
with children, if the variables come first: every other dual pivot is then -1/rho minus a square.  Reference: numpy's
dense solve of the remaining rows."""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2510_05885_amd import ncl_kkt as nk
from paper_2510_05885_amd import synth

from gpu_util import colmajor, dev

pytestmark = pytest.mark.gpu


# last fronts of 43 rows (one wave), 80 to 95 (four waves), 411 and 992 (panels)
@pytest.mark.parametrize("n,m", [(40, 12), (80, 30), (100, 30), (300, 120), (700, 300)])
@pytest.mark.parametrize("scale", ["global", "block", "absolute"])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_zero_rows_of_j(n, m, scale, nrhs):
    inp = synth.random_system(n, m, seed=3, rho=1e14)
    zero = np.arange(0, m, 3)
    for r in zero:
        inp.J_val[inp.J_rowptr[r]:inp.J_rowptr[r + 1]] = 0.0
    kkt = nk.KKT.from_input(inp, form="stabilized", ordering="natural", pivot_scale=scale)
    rc = kkt.factor(dev(inp.W_val), dev(inp.Sigma), dev(inp.J_val), inp.rho)
    # 1/rho = 1e-14 is below eps ||K||_max and eps = 1e-10, above eps / rho
    assert rc == 0 and kkt.inertia() == (n, m, 0, 0 if scale == "block" else len(zero))
    keep = np.setdiff1d(np.arange(n + m), n + zero)
    B = synth.rhs(n + m, nrhs, seed=n).reshape(n + m, nrhs)
    B[n + zero] = 0.0
    X, _ = kkt.solve(colmajor(B))
    X = X.cpu().numpy().reshape(B.shape)
    K = O.assemble(inp, O.STABILIZED).dense()[np.ix_(keep, keep)]
    ref = np.linalg.solve(K, B[keep])
    kappa = np.abs(K).sum(1).max() * np.abs(np.linalg.inv(K)).sum(1).max()
    # refined to a normwise backward error of 1e-12
    assert np.abs(X[keep] - ref).max() <= 4e-12 * kappa * np.abs(ref).max()
    assert not X[n + zero].any()
    kkt.close()


def test_block_rule_costs_what_the_absolute_rule_costs():
    """With Sigma up to 1e8 the primal threshold of the block rule is above the dual pivots of -1/rho, which are
    tested against the dual one: such a factorization once took 1.75 times as long as with the absolute rule."""
    inp = synth.opf_network(N=1000, seed=2)
    inp.Sigma[:] = 10.0 ** np.random.default_rng(1).uniform(-8.0, 8.0, inp.n)
    args = [dev(inp.W_val), dev(inp.Sigma), dev(inp.J_val)]
    best = {}
    handles = {s: nk.KKT.from_input(inp, form="stabilized", pivot_scale=s, pivot_eps=1e-10)
               for s in ("absolute", "block")}
    for _ in range(6):
        for s, kkt in handles.items():
            kkt.factor(*args, 1e4)
            t = time.perf_counter()
            for _ in range(10):
                kkt.factor(*args, 1e4)   # waits for the GPU
            best[s] = min(best.get(s, 1e9), time.perf_counter() - t)
    for kkt in handles.values():
        kkt.close()
    assert best["block"] <= 1.35 * best["absolute"]
