"""Tiles whose rows are split over a team of workgroups (csrc/dsq_team_impl.h): every shape at sizes with ragged tiles and uneven
parts, the path of a workgroup that finds the other parts of its tile unclaimed, the row-streaming plan's steps in one launch,
a captured step whose graph is replaced by one with more to fetch, and graphs with more to fetch than a workgroup's LDS holds.  State and messages bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1907_07346_amd import binding as b
from paper_1907_07346_amd import workloads as wl
from test_gpu_parity import assert_close, lock_step, oracle_state, say, small, upload

pytestmark = pytest.mark.gpu

CASES = [small(wl.KIND_QUANT_MAXABS, 65, 512 * 3 + 77, bits=4, block=512),
         small(wl.KIND_QUANT_MAXABS, 20, 2048 * 2 + 9, bits=2, block=2048),
         small(wl.KIND_SIGN_MEANABS, 100, 64 * 9 + 33, block=64),
         small(wl.KIND_QUANT_MAXABS, 130, 1024 * 2 + 1001, bits=8, block=1024, topo=wl.TOPO_TORUS2D, torus=(10, 13)),
         small(wl.KIND_QUANT_MAXABS, 33, 128 * 9 + 3, bits=2, block=128),
         small(wl.KIND_SIGN_MEANABS, 66, 256 * 5, block=256),
         small(wl.KIND_SIGN_MEANABS, 48, 512 * 4 + 1, block=512)]


@pytest.mark.parametrize("variant", [0, 3])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_team_shapes(w, variant):
    """variant 3: one workgroup of each tile works and claims all parts, one after the other."""
    seen = []
    for i in range(12):
        plan = {"tile_plan": i, "variant": variant}
        ds = b.DeepSqueeze.from_workload(w, plan)
        name = ds.ds_plan_name()
        ds.ds_destroy()
        if name in seen:
            break
        seen.append(name)
        if "/team/" in name:
            say("case", w.name, "plan", name)
            lock_step(w, steps=2, plan=plan)
    assert sum("/team/" in s for s in seen) >= 2, seen


@pytest.mark.parametrize("shape", [0, 1, 2, 3])
def test_streamed_and_whole_steps_in_turn(shape):
    """A handle of the row-streaming plan: x read after every step, after several, and after every step again; shape 0 never takes a
    step whole."""
    w = CASES[0]
    ds = b.DeepSqueeze.from_workload(w, {"variant": 1, "tile_plan": shape})
    st = oracle_state(w)
    for t in range(14):
        g = wl.gradient(w, t)
        ds.ds_step(upload(g))
        _, msg = oracle.step(st, g, want_cv=False)
        assert np.array_equal(ds.ds_read_messages(), msg), t
        if t in (0, 1, 4, 7, 8, 9, 12, 13):
            x, d = ds.ds_read_state()
            assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0
    ds.ds_destroy()


def _ring_of_every(n, stride):
    W = np.zeros((n, n))
    for i in range(n):
        for d in (-1, 0, 1):
            W[i * stride % n, (i + d) * stride % n] = 1 / 3
    rp = np.concatenate([[0], np.cumsum((W != 0).sum(1))]).astype(np.int32)
    return W, (rp, np.nonzero(W)[1].astype(np.int32), W[W != 0].astype(np.float32))


@pytest.mark.parametrize("plan", [{"tile_plan": 3}, {"variant": 1, "tile_plan": 3}, {"variant": 1, "tile_plan": 0}],
                         ids=["team", "stream, whole steps", "stream"])
def test_captured_step_outlives_its_graph(plan):
    """A step captured with a ring of adjacent workers, replayed with a ring of as many entries whose neighbours are all in other parts
    (more rows to fetch than the captured launch has LDS for), eager steps in between."""
    w = CASES[0]
    (W0, csr0), (W1, csr1) = _ring_of_every(w.n, 1), _ring_of_every(w.n, 22)
    cfg, keep = b.make_config(w.n, w.N, wl.TOPO_CSR, w.kind, w.gamma, w.eta, bits=w.bits, block=w.block, seed=w.seed, W_csr=csr0)
    ds = b.DeepSqueeze(cfg, keep, plan)
    st = oracle_state(w, W0)
    g = wl.gradient(w, 0)
    gd = upload(g)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ds.ds_step(gd)
        oracle.step(st, g, want_cv=False, want_msg=False)
        ds.ds_read_state()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            ds.ds_step(gd)
        for W, csr in ((W0, csr0), (W1, csr1)):
            ds.ds_set_mixing(csr)
            now = oracle_state(w, W)
            now.x, now.delta, now.t = st.x, st.delta, st.t
            st = now
            for r in range(4):
                graph.replay()
                oracle.step(st, g, want_cv=False, want_msg=False)
                if r == 1:
                    ds.ds_step(gd)
                    oracle.step(st, g, want_cv=False, want_msg=False)
                if r != 2:
                    x, d = ds.ds_read_state()
                    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0, (W is W1, r)
    side.synchronize()
    del graph
    ds.ds_destroy()


def _circulant(n, offsets):
    W = np.zeros((n, n))
    for i in range(n):
        for d in offsets:
            W[i, (i + d) % n] = 1 / len(offsets)
    rp = np.concatenate([[0], np.cumsum((W != 0).sum(1))]).astype(np.int32)
    return W, (rp, np.nonzero(W)[1].astype(np.int32), W[W != 0].astype(np.float32))


@pytest.mark.parametrize("capture", [False, True])
@pytest.mark.parametrize("wide", [[0, *range(5, 53, 6), *range(-47, 0, 6)], list(range(100))], ids=["as many entries", "dense"])
def test_a_graph_too_wide_for_the_team(wide, capture):
    """100 workers, blocks of 2048, 8 bits: a part's 15 rows and the 16 they fetch take 64 KB; with the wide graphs they fetch all others,
    205 KB, which no workgroup has.  Steps go on after such a W, one by one and in runs, and after the way back."""
    w = small(wl.KIND_QUANT_MAXABS, 100, 2048 * 2 + 9, bits=8, block=2048)
    near = _circulant(w.n, range(-8, 9))
    cfg, keep = b.make_config(w.n, w.N, wl.TOPO_CSR, w.kind, w.gamma, w.eta, bits=w.bits, block=w.block, seed=w.seed, W_csr=near[1])
    ds = b.DeepSqueeze(cfg, keep, {"variant": 1, "tile_plan": 1})
    st = oracle_state(w, near[0])
    g = wl.gradient(w, 0)
    gd = upload(g)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def compare(what):
        x, d = ds.ds_read_state()
        assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0, what

    with torch.cuda.stream(side):
        ds.ds_step(gd)
        oracle.step(st, g, want_cv=False, want_msg=False)
        compare("first")
        graph = None
        if capture:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                ds.ds_state_ptrs()
                ds.ds_step(gd)
        for W, csr in (near, _circulant(w.n, wide), near):
            ds.ds_set_mixing(csr)
            now = oracle_state(w, W)
            now.x, now.delta, now.t = st.x, st.delta, st.t
            st = now
            if len(wide) == 100 and W is not near[0]:
                graph = None                                 # another number of entries: graphs are gone
            for turn, steps in enumerate((1, 1, 3, 1)):
                say("entries", len(csr[1]), "capture", capture, "turn", turn)
                for s in range(steps):
                    if graph is not None and turn == 1:
                        graph.replay()
                    else:
                        ds.ds_step(gd)
                    oracle.step(st, g, want_cv=False, want_msg=False)
                compare((len(csr[1]), turn))
    side.synchronize()
    del graph
    ds.ds_destroy()
