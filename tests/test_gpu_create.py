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
* A state whose weight rows find no room, or are given back to a call that needs
  their memory, sweeps as one that has them.
"""
import numpy as np
import pytest

import synth
from paper_1510_06549_amd import spdp as sp
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


@pytest.fixture
def return_memory():
    """What torch holds goes back to the device, also after a failure."""
    import gc

    import torch

    yield
    gc.collect()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("S", [0, 2])
def test_states_without_room_for_weight_rows(S, return_memory):
    import torch

    print(f"weight rows without room, sources={S}", flush=True)
    rng = np.random.default_rng(8)
    G, V, K, N = 8, 1 << 15, 1024, 20000  # 2^18 rows: 1.6 GB of counts, 2.1 GB of weight rows
    w = rng.integers(0, 25, N).astype(np.int32)
    args = (w, np.arange(0, N + 1, 100), np.arange(200, dtype=np.int32) % G, G, V, K, 0.1, 0.5,
            20.0, 0.01)
    assoc = synth.associations(G, V, S, 0.3, 5) if S else None
    weights = 2 * 4 * G * V * K

    def base_launches(s):
        """16-bit copies of the shadow base that a sweep made: none over weight rows."""
        sp.spdp_kernel_timing(s.h, True)
        s.sweep(0, 3)
        n = sp.spdp_kernel_times(s.h)["base"][1]
        sp.spdp_kernel_timing(s.h, False)
        return n

    full = sp.Sampler(*args, assoc=assoc)
    held = full.info["device_bytes"]
    assert base_launches(full) == 0
    want = parity.state_of(full, None) + ((full.slots(),) if S else ())

    def leave(room):
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        return torch.empty(free - room, dtype=torch.uint8, device="cuda")

    def check(s):
        got = parity.state_of(s, None) + ((s.slots(),) if S else ())
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
        assert s.check() == 0

    # no room for them
    ballast = [leave(held - weights // 2)]
    s = sp.Sampler(*args, assoc=assoc)
    assert s.info["device_bytes"] <= held - weights
    assert base_launches(s) == 1
    del ballast
    check(s)
    s.close()

    # room for them, until the staging buffer of an estimate (256 MiB) needs it: what is left
    # goes in pieces of 64 MiB, a few more than the free memory counts
    ballast = [leave(held + (1 << 30))]
    s = sp.Sampler(*args, assoc=assoc)
    assert s.info["device_bytes"] > held - weights // 2
    for _ in range(64):
        try:
            ballast.append(torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            break
    sp.spdp_estimates(s.h, 0, 0, None, np.empty((V, K)), None)
    assert sp.spdp_info(s.h)["device_bytes"] <= held - weights
    assert base_launches(s) == 1
    del ballast
    check(s)
    s.close()
    full.close()
