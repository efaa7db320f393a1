"""The select of the top-k path's launches where one workgroup does a row's (few candidates) and where several do, each with the
slots of small and of large k, at sizes on both sides of the rules: messages and state against the oracle, the row's guess in
use at the end; ties by the hundred, which leave the candidates for the exact way."""
import numpy as np
import pytest

import oracle
from paper_1907_07346_amd import binding as b
from paper_1907_07346_amd import workloads as wl
from test_gpu_parity import assert_close, oracle_state, say, small, upload

pytestmark = pytest.mark.gpu

LAUNCHES = {"variant": 2}


def run(w, gradients, steps, candidates, plan=LAUNCHES):
    ds = b.DeepSqueeze.from_workload(w, plan)
    st = oracle_state(w)
    for t in range(steps):
        g = gradients(t)
        ds.ds_step(upload(g))
        _, msg = oracle.step(st, g, want_cv=False)
        assert np.array_equal(ds.ds_read_messages(), msg), (w.name, t)
        if t % 3 == 2:
            x, d = ds.ds_read_state()
            assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0
    if candidates:
        assert ds.ds_topk_candidate_rows() == w.n, ds.ds_topk_candidate_rows()
    x, d = ds.ds_read_state()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0
    ds.ds_destroy()


@pytest.mark.parametrize("n,N,k", [(5, 4096 * 3 + 1, 123), (5, 4096 * 3 + 1, 1300), (3, 4096 * 128, 5000), (3, 4096 * 128 + 1, 5000), (3, 200_000, 16_384),
                                   (3, 200_000, 16_385), (3, 65_000, 2031), (3, 65_000, 2032), (3, 30_000, 15_000), (3, 9_000, 9_000)])
def test_select_at_the_edges_of_its_rules(n, N, k):
    w = small(wl.KIND_TOPK, n, N, k=k)
    say("case", w.name)
    run(w, lambda t: wl.gradient(w, t), 10, candidates=k < N // 3)


@pytest.mark.parametrize("k", [700, 4000])
def test_ties_by_the_thousand(k):
    """Three magnitudes only: the threshold's bin holds more keys than are listed."""
    w = small(wl.KIND_TOPK, 3, 20_011, k=k)
    rng = np.random.default_rng(3)
    gs = [rng.choice(np.array([0.5, -0.5, 1.0, -2.0], np.float32), (w.n, w.N)) for _ in range(4)]
    run(w, lambda t: gs[t], 4, candidates=False)


def test_large_k_in_small_slots():
    """What a state whose larger slots could not be allocated does: 1.3 k candidates aimed at, 512 places for 640 of them, rows that go the
    exact way.  (300 x 8 chunks are too many for one launch.)"""
    w = small(wl.KIND_TOPK, 300, 4096 * 7 + 5, k=3_584)
    run(w, lambda t: wl.gradient(w, t), 4, candidates=False, plan={"variant": 3})
