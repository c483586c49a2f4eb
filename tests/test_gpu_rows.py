"""The sampler over weight rows at the edges of its shapes, against the oracle.

The lanes per document follow the number of documents (16 above 32 768, 32 or
64 below), the topics per lane the topic count; chunks hold 16 tokens.  The
small-corpus tests elsewhere reach the 32- and 64-lane instances at every
topic count; these corpora have enough documents for the 16-lane ones, with
lengths around whole chunks, empty documents, and (K = 520) a lane layout with
a remainder at 64 lanes.  The bounds are the parity protocol's.

Hyperparameters whose fp32 weights overflow or are no numbers, or are small but
still normal: a draw that fp32 cannot decide is decided in fp64, so the states
(and sources) are the oracle's.
"""
import numpy as np
import pytest

import synth
from paper_1510_06549_amd import spdp as sp
from tests import parity

pytestmark = pytest.mark.gpu


def _corpus(docs, K, seed):
    """`docs` documents in 3 groups: lengths mostly 0 to 3, some around the
    chunk edges; 150 words with a Zipf law each group permutes."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 4, docs)
    edge = rng.choice(docs, 400, replace=False)
    lens[edge] = rng.choice([15, 16, 17, 31, 32, 33, 48, 70], 400)
    off = np.zeros(docs + 1, dtype=np.int64)
    np.cumsum(lens, out=off[1:])
    group = np.sort(rng.integers(0, 3, docs)).astype(np.int32)
    V = 150
    law = 1.0 / np.arange(1, V + 1)
    w = rng.choice(V, size=int(off[-1]), p=law / law.sum())
    w = (w + 41 * np.repeat(group, lens)) % V
    z = np.zeros(int(off[-1]), dtype=np.int32)
    return synth.Corpus(w.astype(np.int32), off, group, z, z.astype(np.uint8), 3, V)


@pytest.mark.parametrize("docs,K", [(33000, 1), (33000, 16), (33000, 17), (33000, 60),
                                    (33000, 112), (33000, 144), (33000, 208), (33000, 256),
                                    (3000, 130), (3000, 520)])
def test_sweeps_match_oracle_at_every_lane_layout(docs, K):
    print(f"weight rows: docs={docs} K={K}", flush=True)
    cp = _corpus(docs, K, 100 * K + docs % 97)
    wl = synth.workload(0)
    s, m = parity.make_pair(cp, wl, K=K)
    for sweep in range(2):
        rep, _, _ = parity.one_step(s, m, sweep, 77)
        assert rep.mismatches == 0
    s.check()
    s.close()


@pytest.mark.parametrize("docs,K,S", [(33000, 40, 3), (33000, 200, 8), (3000, 70, 1)])
def test_sweeps_with_associations_match_oracle(docs, K, S):
    print(f"weight rows: docs={docs} K={K} sources={S}", flush=True)
    cp = _corpus(docs, K, 7 * K + S)
    wl = synth.workload(0)
    assoc = synth.associations(3, cp.vocab, S, 0.3 if S > 1 else 0.0, 5)
    s, m = parity.make_pair(cp, wl, K=K, assoc=assoc)
    for sweep in range(2):
        rep, _, _ = parity.one_step(s, m, sweep, 78)
        assert rep.mismatches == 0
    s.check()
    s.close()


@pytest.mark.parametrize("sparse", [False, True])
def test_captured_sweeps(sparse):
    """Replays of two captured sweeps, with the calls that read the counts between
    them and eager sweeps between two, leave what eager sweeps leave."""
    import torch

    print(f"captured sweeps, {'count' if sparse else 'weight'} rows", flush=True)
    cp = _corpus(450, 60, 60)
    if sparse:
        cp = _sparse(cp, 6000, 3)
    args = (cp.words, cp.doc_off, cp.doc_group, cp.n_groups, cp.vocab, 60, 0.1, 0.5, 20.0, 0.01)
    stream = torch.cuda.Stream()
    s, e = sp.Sampler(*args, hip_stream=stream.cuda_stream), sp.Sampler(*args)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        s.sweep(0, 7)
        s.sweep(1, 7)
    for rep in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        e.sweep(0, 7)
        e.sweep(1, 7)
        for got, want in zip(parity.state_of(s, None), parity.state_of(e, None)):
            assert np.array_equal(got, want), rep
        for got, want in zip(s.counts() + s.totals(), e.counts() + e.totals()):
            assert np.array_equal(got, want), rep
        for got, want in zip(s.conditionals(9, 7, 0, 99), e.conditionals(9, 7, 0, 99)):
            assert np.array_equal(got, want), rep
        assert s.check() == 0
        for x in (s, e) if rep == 1 else ():
            x.sweep(2, 7)
            x.sweep(3, 7)
    s.close()
    e.close()


EXTREMES = [(0.1, 20.0, 0.01), (1e38, 20.0, 0.01), (1e300, 20.0, 0.01), (1e-310, 20.0, 0.01),
            (0.1, 1e-40, 0.01), (0.1, 1e300, 0.01), (0.1, 20.0, 1e-25), (0.1, 20.0, 1e300)]


def _extreme(alpha, b, gamma):
    wl = synth.workload(0)
    return type(wl)(**{**wl.__dict__, "alpha": alpha, "b": b, "gamma": gamma})


def _sweeps_equal_oracle(s, m, sweeps):
    for sweep in range(sweeps):
        st = [x.copy() for x in parity.state_of(s, m)]
        c = m.rebuild(*st)
        m.sample_docs(c, *st, sweep, 7)
        m.repair(*st, m.rebuild(*st))
        s.sweep(sweep, 7)
        for got, want in zip(parity.state_of(s, m), st):
            assert np.array_equal(got, want), sweep
    assert s.check() == 0


@pytest.mark.parametrize("S", [0, 3])
@pytest.mark.parametrize("alpha,b,gamma", EXTREMES)
def test_sweeps_where_single_precision_does_not_reach(alpha, b, gamma, S):
    print(f"weight rows: alpha={alpha} b={b} gamma={gamma} sources={S}", flush=True)
    wl = _extreme(alpha, b, gamma)
    for K in (10, 20, 140):  # 16, 32 and 64 lanes
        cp = _corpus(450, K, K)
        assoc = synth.associations(3, cp.vocab, S, 0.3, 5) if S else None
        s, m = parity.make_pair(cp, wl, K=K, assoc=assoc)
        _sweeps_equal_oracle(s, m, 3)
        s.close()


def _sparse(cp, words, seed):
    """cp with every other token one of `words` more words, equally likely."""
    rng = np.random.default_rng(seed)
    w = np.where(np.arange(cp.words.size) % 2, cp.words,
                 cp.vocab + rng.integers(0, words, cp.words.size)).astype(np.int32)
    z = np.zeros_like(w)
    return synth.Corpus(w, cp.doc_off, cp.doc_group, z, z.astype(np.uint8), 3, cp.vocab + words)


@pytest.mark.parametrize("S", [0, 3])
@pytest.mark.parametrize("alpha,b,gamma", EXTREMES)
def test_sparse_sweeps_where_single_precision_does_not_reach(alpha, b, gamma, S):
    """The same over count rows: too few tokens per row for weight rows."""
    print(f"count rows: alpha={alpha} b={b} gamma={gamma} sources={S}", flush=True)
    wl = _extreme(alpha, b, gamma)
    for K in (60, 140):  # padding topics in a lane's slice, and lanes of them only
        cp = _sparse(_corpus(450, K, K), 6000, 3)
        assoc = synth.associations(3, cp.vocab, S, 0.3, 5) if S else None
        s, m = parity.make_pair(cp, wl, K=K, assoc=assoc)
        sp.spdp_kernel_timing(s.h, True)
        _sweeps_equal_oracle(s, m, 3)
        assert sp.spdp_kernel_times(s.h)["base"][1] == 3  # a 16-bit base each: over count rows
        s.close()


@pytest.mark.parametrize("alpha,b,gamma", EXTREMES)
def test_asynchronous_sweeps_where_single_precision_does_not_reach(alpha, b, gamma):
    print(f"asynchronous sweep: alpha={alpha} b={b} gamma={gamma}", flush=True)
    cp = _corpus(450, 60, 60)
    s, m = parity.make_pair(cp, _extreme(alpha, b, gamma), K=60)
    z, r = s.assignments()
    c = m.rebuild(z, r)
    for sweep in range(2):
        s.sweep_async(sweep, 7, waves=1, live_totals=True)
        m.sweep(c, z, r, sweep, 7, mode="ordered", order=m.interleaved_order())
        zg, rg = s.assignments()
        assert np.array_equal(zg, z) and np.array_equal(rg, r), sweep
    s.close()
