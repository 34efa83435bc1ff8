"""Fronts with children at the edges of the small-front kernels: chosen elimination trees, unrefined
solutions against the matrix itself, equal bits over passes.

Tolerance: an LDL^T solve of order n has a row-wise backward error of 3 n u |L||D||L^T|, and |L||D||L^T| stays
within a small multiple of |A| for a diagonally dominant A: 10 n u."""
import numpy as np
import pytest

from paper_2510_05885_amd import ncl_kkt as nk
from paper_2510_05885_amd import synth

from front_trees import OPTIONS, Tree, plan_orders, row_error
from gpu_util import colmajor, dev

pytestmark = pytest.mark.gpu

UNIT = {"fp64": 2.0 ** -53, "fp32_ir": 2.0 ** -24}


def _check(tree, precision, columns=(1,), passes=3, seed=5, **opts):
    A, pat = tree.matrix(seed)
    inp = tree.input(A, pat)
    # ir_tol: any useful factor meets it without refinement
    kkt = nk.KKT.from_input(inp, precision=precision, ir_tol=1e-2, **OPTIONS, **opts)
    assert plan_orders(kkt) == tree.orders()
    first = {}
    for _ in range(passes):
        assert kkt.factor(dev(inp.W_val), dev(inp.Sigma), None, 1.0) == 0
        assert kkt.inertia() == (tree.n, 0, 0, 0)
        for q in columns:
            B = synth.rhs(tree.n, q, seed=q).reshape(tree.n, q)
            X, info = kkt.solve(colmajor(B))
            X = X.cpu().numpy().reshape(B.shape)
            assert info.ir_steps == 0 and row_error(A, X, B) <= 10 * tree.n * UNIT[precision]
            assert np.array_equal(first.setdefault(q, X), X)
    kkt.close()


def _below(rng, top, k):
    """k rows of a front of `top` pivots, its first among them (where the child hangs)."""
    return np.concatenate([[0], np.sort(1 + rng.choice(top - 1, k - 1, replace=False))])


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("children", [0, 1, 4])
@pytest.mark.parametrize("order", [97, 113, 128])
def test_dense_first_subpanel(order, children, precision):
    """More than 512 entries of K in the first 16 columns of a front of four waves with at most four
    children, whose leaves share a launch with another such front and so are factored by four waves too."""
    rng = np.random.default_rng(order + children)
    root = 200
    mid = np.concatenate([np.arange(16), 16 + _below(rng, root, order - 16)])
    tree = Tree(16 + root)
    for k in range(children):
        tree.add(17 + k, mid[_below(rng, order, 24)])
    tree.add(16, 16 + _below(rng, root, order - 16))   # a leaf of the same shape
    tree.add(16, mid[16:])
    tree.add(root)
    _check(tree, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("children", [0, 1, 4, 5])
@pytest.mark.parametrize("order", [65, 80, 81, 96])
def test_dense_first_subpanel_of_21_tiles(order, children, precision):
    """The same in launches whose largest front has 65 to 96 rows: 21 tiles in the 24 slots of four waves."""
    rng = np.random.default_rng(order + children)
    root = 200
    mid = np.concatenate([np.arange(16), 16 + _below(rng, root, order - 16)])
    tree = Tree(16 + root)
    for k in range(children):
        tree.add(17 + k, mid[_below(rng, order, 24)])
    tree.add(16, 16 + _below(rng, root, order - 16))
    tree.add(16, mid[16:])
    tree.add(root)
    _check(tree, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("children", [0, 1, 4, 5, 9])
@pytest.mark.parametrize("root", [33, 64, 65, 80, 96, 97, 128, 193])
def test_star(root, children, precision):
    """A root of every class (one wave, four waves, panels) under leaves whose pivots and rows are no multiples
    of 16, with 1, 3 and 16 right-hand sides: more children than maps in LDS at a time, several entries a row in
    the sweeps' gather tables, contribution blocks and rows of ancestors at every offset."""
    rng = np.random.default_rng(root + children)
    tree = Tree(root)
    for k in range(children):
        # (with enough pivots not to be merged into the root)
        tree.add([15, 16, 17, 31, 33, 47, 48, 49, 65][k], _below(rng, root, [14, 13, 15, 17, 30, 16, 9, 25, 21][k]))
    tree.add(root)
    _check(tree, precision, columns=(1, 3, 16), passes=2)


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("root", [30, 64, 128, 193])
def test_many_children_on_one_row(root, precision):
    """60 leaves with the root's first row in common: that row's update entries go beyond the sweeps' gather table
    into its list, with 1, 3 and 16 right-hand sides."""
    rng = np.random.default_rng(root)
    tree = Tree(root)
    for _ in range(60):
        tree.add(25, _below(rng, root, 3))
    tree.add(root)
    _check(tree, precision, columns=(1, 3, 16), passes=2)
