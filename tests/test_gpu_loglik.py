"""The log-likelihood at the edges of its parts, against the oracle.

Topic counts on both sides of the row widths (a thread takes four cells and a
block as many rows as fit it), narrow and wide rows, an empty document, and
documents, shadow-base and cell counts on both sides of the 1 024 entries of the
log-gamma tables.  Every sum is of fp64 terms: at most 1e4 of them in a chain,
so 1e-12 of their magnitudes' sum, which is below 100 times the result's, and a
log Stirling entry of n <= 3 000 carries at most 16 n eps = 1.1e-11 of its size:
a bound of 1.2e-10 relative.
"""
import numpy as np
import pytest

import synth
from paper_1510_06549_amd import spdp as sp
from tests import parity
from tests.test_gpu_rows import _corpus

pytestmark = pytest.mark.gpu


def _with_long_documents(cp):
    """cp and documents of one word with 1 023, 1 024, 1 025 and 0 tokens."""
    lens = np.array([1023, 1024, 1025, 0])
    off = np.concatenate([cp.doc_off, cp.doc_off[-1] + np.cumsum(lens)])
    words = np.concatenate([cp.words, np.full(lens.sum(), 7, np.int32)])
    group = np.concatenate([cp.doc_group, np.array([0, 1, 1, 2], np.int32)])
    z = np.zeros(words.size, np.int32)
    return synth.Corpus(words, off, group, z, z.astype(np.uint8), 3, cp.vocab)


@pytest.mark.parametrize("K,S", [(1, 0), (32, 0), (33, 0), (100, 0), (257, 0), (1024, 0), (40, 3)])
def test_loglik_at_part_edges(K, S):
    print(f"loglik K={K} sources={S}", flush=True)
    cp = _with_long_documents(_corpus(1001, K, 7 * K))
    assoc = synth.associations(3, cp.vocab, S, 0.3, 5) if S else None
    s, m = parity.make_pair(cp, synth.workload(0), K=K, assoc=assoc)
    # one topic for the long documents: histogram entries past the table
    z, r = s.assignments()
    z[cp.doc_off[-5]:] = 0
    r[cp.doc_off[-5]:] = 1
    s.set_assignments(z, r, *([np.zeros_like(r)] if S else []))
    for sweep in range(2):
        st = parity.state_of(s, m)
        want, got = m.loglik(*st, m.rebuild(*st)), s.loglik()
        assert abs(got - want) <= 1.2e-10 * abs(want), (sweep, got, want)
        assert s.loglik() == got
        s.sweep(sweep, 3)
    s.close()


@pytest.mark.parametrize("word", [7, 149])  # a wide row, a narrow one
@pytest.mark.parametrize("dt", [1, -1])
def test_loglik_refuses_a_cell_without_probability(word, dt):
    cp = _with_long_documents(_corpus(1001, 3, 11))
    s, m = parity.make_pair(cp, synth.workload(0), K=33)
    n, t = s.counts()
    ll = s.loglik()
    g = int(np.argmax(n[:, :, word].sum(1)))
    k = int(np.argmax(n[g, :, word]))
    d = int(n[g, k, word] - t[g, k, word]) + 1 if dt > 0 else -int(t[g, k, word])
    s.poke(g, word, k, 0, d)
    with pytest.raises(sp.SpdpError) as e:
        s.loglik()
    assert e.value.code == sp.SPDP_E_STATE
    s.poke(g, word, k, 0, -d)
    assert s.loglik() == ll
    s.close()
