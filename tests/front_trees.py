"""Systems whose elimination trees have prescribed fronts, for the kernels that
factor and sweep them."""
import numpy as np

from paper_2510_05885_amd import synth

# natural ordering, and fronts of more than 128 rows merged only where that adds
# next to no zeros, so that the fronts stay as they are given
OPTIONS = dict(ordering="natural", relax_big_zeros=0.0)


class Tree:
    """Fronts in elimination order.  add(p, below) appends a front of p pivots
    whose other rows `below` are pivots of later fronts, counted from the end:
    row r is the r-th of the last `top` pivots, which the last calls must add."""

    def __init__(self, top):
        self.top, self.fronts, self.n = top, [], 0

    def add(self, p, below=()):
        self.fronts.append((self.n, p, np.asarray(below, dtype=np.int64)))
        self.n += p
        return self

    def orders(self):
        """(pivots, order) of every front, sorted."""
        return sorted((p, p + len(b)) for _, p, b in self.fronts)

    def matrix(self, seed, negative=()):
        """Symmetric matrix with a dense clique a front, diagonally dominant by a factor of 1.5, the
        diagonal of the rows in `negative` negative."""
        rng = np.random.default_rng(seed)
        A = np.zeros((self.n, self.n))
        pat = np.zeros((self.n, self.n), dtype=bool)
        for first, p, below in self.fronts:
            rows = np.concatenate([np.arange(first, first + p), self.n - self.top + below])
            pat[np.ix_(rows, rows)] = True
            R = rng.uniform(0.5, 1.5, (len(rows), len(rows))) * rng.choice([-1.0, 1.0], (len(rows), len(rows)))
            A[np.ix_(rows, rows)] += R + R.T
        np.fill_diagonal(A, 0.0)
        d = 1.5 * np.abs(A).sum(1) + 1.0
        d[list(negative)] *= -1.0
        np.fill_diagonal(A, d)
        return A, pat

    def input(self, A, pat):
        """The system as W of a condensed KKT system without constraints."""
        n = self.n
        col = [np.nonzero(pat[j:, j])[0] + j for j in range(n)]
        colptr = np.concatenate([[0], np.cumsum([len(c) for c in col])]).astype(np.int32)
        rowidx = np.concatenate(col).astype(np.int32)
        vals = np.concatenate([A[c, j] for j, c in enumerate(col)])
        return synth.KKTInput(n, 0, colptr, rowidx, vals, np.zeros(n), np.zeros(1, np.int32), np.zeros(0, np.int32),
                              np.zeros(0), 1.0)


def plan_orders(kkt):
    """(pivots, order) of every front of an analysed handle, sorted."""
    first, _, rowptr, _ = kkt.supernodes()
    return sorted(zip(np.diff(first).tolist(), np.diff(rowptr).tolist()))


def row_error(A, X, B):
    """max_i |b - A x|_i / (|A| |x|)_i over the columns."""
    return float((np.abs(B - A @ X) / (np.abs(A) @ np.abs(X))).max())
