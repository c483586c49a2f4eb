"""Edges of the launch shapes of the Hellinger and estimate kernels.

* Distances with topic counts and outcome counts that leave ragged 128-wide
  tiles and a ragged last slice, against the oracle (|H^2 difference| <= 1e-12:
  fp64 sums over at most 1e5 outcomes).
* Estimates at topic counts on both sides of a block's topic range (512) and of
  a wavefront, over a vocabulary that is no multiple of the words a thread
  takes, with rows of both widths, and a document count that is no multiple of
  the documents a wave takes (relative 1e-13 / 1e-12, as for the other
  estimate tests: each value is one fp64 expression).
* Estimates whose divisors b + N and V gamma + B_k have no reciprocal in fp64
  (subnormal or infinite, for topics and groups without customers) or lie at
  the ends of the range where one is used; the same tolerances, and a few
  subnormal units (8 x 5e-324) where the values themselves are subnormal.
* A fold-in of more test documents than 256-thread blocks fit one launch (2^24),
  nearly all of them empty, against the fold-in of the others alone: a token's
  draws depend on its index, which is the same in both, and an empty document
  adds 0, so topics and sums are equal.
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


@pytest.mark.parametrize("b,gamma", [(1e-310, 0.01), (20.0, 1e-320), (5e-324, 5e-324),
                                     (1e-280, 1e-290), (1e308, 0.01), (20.0, 1e308),
                                     (1e270, 1e265), (1e275, 1e-275)])
@pytest.mark.parametrize("S", [0, 2])
def test_estimates_with_extreme_divisors(b, gamma, S):
    print(f"estimates b={b} gamma={gamma} sources={S}", flush=True)
    V, K = 13, 70  # fewer tokens than topics, so most topics have no customer
    rng = np.random.default_rng(4)
    cp = synth.Corpus(rng.integers(0, V, 20).astype(np.int32), np.array([0, 9, 20]),
                      np.array([0, 1], np.int32), np.zeros(20, np.int32), np.zeros(20, np.uint8),
                      2, V)
    wl = synth.workload(0)
    wl = type(wl)(**{**wl.__dict__, "b": b, "gamma": gamma})
    assoc = synth.associations(2, V, S, 0.3, 5) if S else None
    s, m = parity.make_pair(cp, wl, K=K, assoc=assoc)
    st = parity.state_of(s, m)
    _, p0_o, pg_o = m.estimates(st[0], m.rebuild(*st))
    _, p0, pg = s.estimates()
    assert np.array_equal(np.isnan(p0), np.isnan(p0_o.T))
    np.testing.assert_allclose(p0, p0_o.T, rtol=1e-13, atol=4e-323)
    np.testing.assert_allclose(pg, pg_o.transpose(0, 2, 1), rtol=1e-12, atol=4e-323)
    s.close()


def test_foldin_of_more_documents_than_blocks_of_a_launch():
    D = (1 << 24) + 77
    print(f"fold-in of {D} documents", flush=True)
    cp = _corpus(1001, 5, 9)
    s, _ = parity.make_pair(cp, synth.workload(0), K=5)
    rng = np.random.default_rng(1)
    # the first and the last document, those on both sides of 2^20 and 2^24, and some others
    at = np.unique(np.concatenate([[0, (1 << 20) - 1, 1 << 20, (1 << 24) - 1, 1 << 24, D - 1],
                                   rng.integers(0, D, 60)]))
    lens = rng.integers(1, 80, at.size)
    words = rng.integers(0, cp.vocab, lens.sum()).astype(np.int32)
    group = rng.integers(0, 3, at.size).astype(np.int32)
    small = s.heldout(words, np.concatenate([[0], np.cumsum(lens)]), group, 3, 7)
    full = np.zeros(D, np.int64)
    full[at] = lens
    group_of = np.zeros(D, np.int32)
    group_of[at] = group
    got = s.heldout(words, np.concatenate([[0], np.cumsum(full)]), group_of, 3, 7)
    assert got[:2] == small[:2]
    assert np.array_equal(got[2], small[2])
    s.close()
