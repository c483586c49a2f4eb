"""What a state is built with at the edges of its kernels, against the oracle.

* log S^n_t by the likelihood of one word that occurs n times in one topic with
  t tables, with n and t on both sides of a band of Stirling rows (64) and of a
  block's columns (192).  A row adds at most 8 rounding errors (log, exp,
  log1p, three sums) to a value of at most M = max |log S|, on either side, and
  the likelihood adds a few terms of the size of n log n, so the difference is
  at most 32 n eps (M + n log n + 10).
* The row index over more than one range of the state route (2^21 row positions
  each), with most rows of a wavefront empty and rows that reach across a range's
  end: the counts after a sweep are the oracle's rebuild of its states.
"""
import numpy as np
import pytest

import synth
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 192, 193, 257, 449])
@pytest.mark.parametrize("a", [0.0, 0.7])
def test_stirling_rows_at_band_edges(n, a):
    print(f"stirling n={n} a={a}", flush=True)
    cp = synth.Corpus(np.zeros(n, np.int32), np.array([0, n]), np.zeros(1, np.int32),
                      np.zeros(n, np.int32), np.ones(n, np.uint8), 1, 2)
    wl = synth.workload(0)
    wl = type(wl)(**{**wl.__dict__, "K": 1, "a": a})
    s, m = parity.make_pair(cp, wl)
    z = np.zeros(n, np.int32)
    for t in sorted({x for x in (1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 384,
                                 385, n - 1, n) if 1 <= x <= n}):
        r = np.zeros(n, np.uint8)
        r[:t] = 1
        s.set_assignments(z, r)
        want = m.loglik(z, r, m.rebuild(z, r))
        M = np.abs(m.logS[np.isfinite(m.logS)]).max()
        bound = 32 * n * np.finfo(float).eps * (M + n * np.log(n + 1) + 10)
        assert abs(s.loglik() - want) <= bound, (t, s.loglik(), want)
    s.close()


def test_row_index_across_route_ranges():
    rng = np.random.default_rng(3)
    D, L, V = 44000, 100, 3000
    law = np.zeros(V)
    law[rng.choice(V, 300, replace=False)] = rng.dirichlet(np.full(300, 0.5))
    w = rng.choice(V, size=D * L, p=law).astype(np.int32)
    zero = np.zeros(D * L, np.int32)
    cp = synth.Corpus(w, np.arange(D + 1) * L, np.sort(rng.integers(0, 3, D)).astype(np.int32),
                      zero, zero.astype(np.uint8), 3, V)
    s, m = parity.make_pair(cp, synth.workload(0), K=4)
    for sw in range(2):
        s.sweep(sw, 5)
        z, r = s.assignments()
        parity.assert_counts_equal(s, m.rebuild(z, r))
        print(f"route: sweep {sw}", flush=True)
    assert s.check() == 0
    s.close()
