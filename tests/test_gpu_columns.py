"""Unrefined solves of several columns against the same columns one at a time: the forward and backward errors of
the two paths are the same, up to the spread of their rounding.  Both substitute within the small fronts; with the
triangles' explicit inverses the several-column sweeps' residuals were 1.22 to 1.59 times as large."""
import numpy as np
import pytest

from paper_2510_05885_amd import ncl_kkt as nk
from paper_2510_05885_amd import synth

from gpu_util import colmajor, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes,rho", [(125, 1e2), (125, 1e6), (400, 1e4), (400, 1e6), (1500, 1e4)])
def test_several_columns_are_as_accurate_as_one(nodes, rho):
    inp = synth.opf_network(N=nodes, seed=2)
    kkt = nk.KKT.from_input(inp, pivot_scale="absolute", pivot_eps=1e-12, ir_max_steps=0)
    rng = np.random.default_rng(nodes)
    logs = []
    for k in range(12):
        sigma = 10.0 ** rng.uniform(-8.0, 8.0, inp.n)
        kkt.factor(dev(inp.W_val), dev(sigma), dev(rng.standard_normal(len(inp.J_val))), rho)
        B = rng.standard_normal((inp.n, 16))
        for q in range(16):
            # the column alone, and with zero columns beside it: the residual of the call is its own
            one, many = colmajor(B[:, q]), np.zeros((inp.n, 3))
            many[:, 1] = B[:, q]
            _, a = kkt.solve(one)
            _, b = kkt.solve(colmajor(many))
            logs.append((np.log(b.resid_rel2 / a.resid_rel2), np.log(b.backward_error / a.backward_error)))
    kkt.close()
    ratio = np.exp(np.mean(logs, 0))
    print("several columns / one: 2-norm residual, normwise backward error", ratio)
    assert (ratio <= 1.15).all()
