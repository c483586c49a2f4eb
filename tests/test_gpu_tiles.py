"""Edges of the launch shapes of the Hellinger and estimate kernels.

* Distances with topic counts and outcome counts that leave ragged 128-wide
  tiles and a ragged last slice, against the oracle (|H^2 difference| <= 1e-12:
  fp64 sums over at most 1e5 outcomes).
* Estimates at topic counts on both sides of a block's topic range (512) and of
  a wavefront, over a vocabulary that is no multiple of the words a thread
  takes, with rows of both widths, and a document count that is no multiple of
  the documents a wave takes (relative 1e-13 / 1e-12, as for the other
  estimate tests: each value is one fp64 expression).
"""
import numpy as np
import pytest

import oracle
import synth
from paper_1510_06549_amd import spdp as sp
from tests import parity
from tests.test_gpu_rows import _corpus

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kp,kq,V", [(130, 255, 33007), (128, 128, 70001), (257, 129, 20016)])
def test_hellinger_in_large_tiles(kp, kq, V):
    print(f"hellinger kp={kp} kq={kq} V={V}", flush=True)
    rng = np.random.default_rng(V)
    P = np.ascontiguousarray(rng.dirichlet(np.full(V, 0.05), size=kp).T)
    Q = np.ascontiguousarray(rng.dirichlet(np.full(V, 0.05), size=kq).T)
    Q[:, kq - 1] = P[:, kp - 1]
    s = sp.Sampler(np.arange(8), np.array([0, 8]), np.array([0]), 1, 8, 2, 0.1, 0.5, 10.0, 0.01)
    H = s.hellinger(Q, P)
    rows = np.unique(np.concatenate([[0, 15, 16, 63, 64, 127, kp - 1], rng.choice(kp, 5)]))
    Ho = oracle.hellinger(P[:, rows].T, Q.T)
    assert np.all(np.abs(H[rows] ** 2 - Ho ** 2) <= 1e-12)
    s.close()


@pytest.mark.parametrize("K,S", [(1, 0), (65, 0), (512, 0), (513, 0), (1024, 0), (70, 3)])
def test_estimates_at_range_edges(K, S):
    print(f"estimates K={K} sources={S}", flush=True)
    cp = _corpus(1001, K, 5 * K)
    wl = synth.workload(0)
    assoc = synth.associations(3, cp.vocab, S, 0.3, 5) if S else None
    s, m = parity.make_pair(cp, wl, K=K, assoc=assoc)
    s.sweep(0, 3)
    st = parity.state_of(s, m)
    th_o, p0_o, pg_o = m.estimates(st[0], m.rebuild(*st))
    th, p0, pg = s.estimates()
    np.testing.assert_allclose(th, th_o, rtol=1e-13)
    np.testing.assert_allclose(p0, p0_o.T, rtol=1e-13)
    np.testing.assert_allclose(pg, pg_o.transpose(0, 2, 1), rtol=1e-12)
    s.close()
