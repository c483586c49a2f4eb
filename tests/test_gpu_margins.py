"""The fp32 sampling path against the rounding bound that its fp64 re-decision
margin rests on, through the C ABI.

The samplers take a draw again in fp64 when the target lies within
(4 KPL + 32) 2^-24 of the total from a CDF boundary (plain model) or
(4 KPL + SP + 32) 2^-24 (word associations).  The bound behind those margins
counts at most 9 roundings in a plain fp32 weight (alpha, gamma, the per-topic
constant and the ratio pair rounded once each from fp64, two sums with counts,
three products); a traced association weight, formed as hq (p bv), carries at
most 11.  Checked here, over several sweeps of three corpora, each plain and
with word associations:
  (a) every traced fp32 weight is within that many roundings of the oracle's
      fp64 weight (relative);
  (b) no token's sample differs from the oracle's: a margin below the sampler's
      real error would let some decision near a boundary come out differently.
The traced weights are those of the samplers over count rows.  The sampler over
weight rows takes a draw again within (2 KPL + SP + 40) 2^-24 of the total from a
topic's boundary, which counts at most 7 roundings in a row's weight before the
document's factor (the per-topic constant, gamma, the ratio pair and the sum with
B rounded once each, two products, the sum of both outcomes), and within
(2 KPL + 3 SP + 64) 2^-24 from one inside the topic, where the share of r = 1
carries 11 (the first term's six, the second's three, their sum, the division);
with word associations SP + 3 more each (p and its product, the sum over SP
sources).  Checked here too:
  (c) every weight and share of the rows that have tokens is within that many
      roundings of the oracle's fp64 value.
Each test prints the case it runs before touching the GPU.
"""
import numpy as np
import pytest

import synth
from tests import parity

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
PLAIN_WEIGHT_ROUNDINGS = 9
ASSOC_WEIGHT_ROUNDINGS = 11


def say(*a):
    print(*a, flush=True)


def _run(idx, sweeps, roundings, assoc_sources=0):
    wl = synth.workload(idx)
    cp = synth.generate(wl, 0)
    assoc = (synth.associations(cp.n_groups, cp.vocab, assoc_sources, 0.3, 5)
             if assoc_sources else None)
    s, m = parity.make_pair(cp, wl, init_seed=3, assoc=assoc)
    worst = 0.0
    for sw in range(sweeps):
        say(f"margins, workload {wl.name}, sources {assoc_sources}, sweep {sw}")
        rep, changed, _ = parity.one_step(s, m, sw, seed=77 + idx)
        say(f"  {rep}")
        assert rep.mismatches == 0, f"{rep.mismatches} samples differ from the oracle"
        worst = max(worst, rep.max_w_rel)
        assert changed > 0
    s.close()
    say(f"  largest relative weight error {worst:.3e} = {worst / U:.2f} u")
    # first order in u; the second-order term is below 1e-6 of the bound
    assert worst <= roundings * U * (1.0 + 1e-6)


@pytest.mark.parametrize("idx,sweeps", [(0, 6), (1, 3), (2, 1)])
def test_plain_weights_within_bound_and_draws_exact(idx, sweeps):
    _run(idx, sweeps, PLAIN_WEIGHT_ROUNDINGS)


@pytest.mark.parametrize("idx,sweeps,sources", [(0, 6, 2), (1, 3, 4), (2, 1, 4)])
def test_assoc_weights_within_bound_and_draws_exact(idx, sweeps, sources):
    _run(idx, sweeps, ASSOC_WEIGHT_ROUNDINGS, sources)


# (500 documents of 20 tokens: 16, 32 and 64 lanes a document, whole 16-byte chunks
# of topics per lane and remainders)
@pytest.mark.parametrize("K,S", [(10, 0), (45, 0), (128, 0), (500, 0), (10, 3), (45, 1), (140, 8)])
def test_weight_rows_within_bound(K, S):
    say(f"weight rows, K = {K}, sources {S}")
    rng = np.random.default_rng(K + S)
    G, V, D, L = 2, 30, 500, 20
    law = 1.0 / np.arange(1, V - 1)  # (the last two words do not occur)
    words = rng.choice(V - 2, size=D * L, p=law / law.sum()).astype(np.int32)
    zero = np.zeros(D * L, np.int32)
    cp = synth.Corpus(words, np.arange(D + 1) * L, np.arange(D, dtype=np.int32) * G // D, zero,
                      zero.astype(np.uint8), G, V)
    assoc = synth.associations(G, V, S, 0.3, 5) if S else None
    s, m = parity.make_pair(cp, synth.workload(0), K=K, assoc=assoc)
    for sw in range(3):
        s.sweep(sw, 9)
    st = parity.state_of(s, m)
    c = m.rebuild(*st)
    pw, rho = s.weight_rows()
    used = np.zeros(G * V, bool)
    used[np.repeat(cp.doc_group, L) * V + words] = True
    assert not pw[~used].any() and used.any() and not used.all()
    Sp = next(x for x in (0, 1, 2, 4, 8) if x >= S)
    extra = Sp + 3 if S else 0
    checked, worst = 0, [0.0, 0.0]
    for q in np.flatnonzero(used):
        g, w = divmod(int(q), V)
        # the oracle's weights of a token of topic k0 hold for every other topic
        for k0 in np.flatnonzero(c.n[g, :, w])[:2]:
            crow = np.zeros(K, np.int32)
            crow[k0] = 1
            args = (c, crow, g, w, k0, 0) + ((0,) if S else ())
            o = m.token_weights(*args).reshape(K, -1) / m.alpha
            other = np.arange(K) != k0
            total, head = o.sum(axis=1)[other], o[:, :max(S, 1)].sum(axis=1)[other]
            worst[0] = max(worst[0], np.abs(pw[q, other] / total - 1.0).max())
            worst[1] = max(worst[1], np.abs(rho[q, other] / (head / total) - 1.0).max())
            checked += int(other.sum())
    say(f"  {checked} weights, largest errors {worst[0] / U:.2f} u, share {worst[1] / U:.2f} u")
    assert checked >= K * used.sum() / 2
    assert worst[0] <= (7 + extra) * U * (1.0 + 1e-6)
    assert worst[1] <= (11 + extra) * U * (1.0 + 1e-6)
    s.close()
