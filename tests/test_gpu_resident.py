"""The kernels that take a whole step of a small problem in one launch (csrc/dsq_resident.h), against the CPU oracle.

Three ways through every case (ds_plan_request.variant): 0, the resident kernel; 3, the same kernel calling its first
meeting off at once, so that the workgroup that leaves last does the whole step alone; 2, the launches that large
problems use.  Messages byte for byte, state bit for bit, with and without the state being read between steps.
"""
import numpy as np
import pytest

import oracle
from paper_1907_07346_amd import binding as b
from paper_1907_07346_amd import workloads as wl
from test_gpu_parity import assert_close, lock_step, oracle_state, say, small, upload

pytestmark = pytest.mark.gpu

# one parameter, one ragged chunk, whole chunks, ragged ones, over 256 chunks in a row (several tree leaves per thread),
# and graphs whose rows have more than four neighbours
CASES = [
    small(wl.KIND_QUANT_L2NORM, 3, 1, bits=4),
    small(wl.KIND_QUANT_L2NORM, 5, 4095, bits=2),
    small(wl.KIND_QUANT_L2NORM, 4, 4096 * 2, bits=8),
    small(wl.KIND_QUANT_L2NORM, 9, 4096 * 3 + 17, bits=4, topo=wl.TOPO_TORUS2D, torus=(3, 3)),
    small(wl.KIND_QUANT_L2NORM, 3, 4096 * 180 + 1, bits=2),
    small(wl.KIND_QUANT_L2NORM, 35, 4096 * 2 + 2, bits=8),
]
# top-k: the same sizes; everything sent; k whose keys are gathered and k that takes the radix select; chunks that send nothing, a
# few pairs, one per thread and more
TOPK = [
    small(wl.KIND_TOPK, 3, 1, k=1),
    small(wl.KIND_TOPK, 5, 4095, k=41),
    small(wl.KIND_TOPK, 4, 4096 * 2, k=4096 * 2),
    small(wl.KIND_TOPK, 9, 4096 * 3 + 17, k=150, topo=wl.TOPO_TORUS2D, torus=(3, 3)),
    small(wl.KIND_TOPK, 3, 4096 * 180 + 1, k=2500),
    small(wl.KIND_TOPK, 3, 4096 * 90 + 1, k=30_000, grad="student_t3"),
    small(wl.KIND_TOPK, 35, 4096 * 2 + 2, k=900),
]
# GSpar: the same sizes; few and many kept per chunk
GSPAR = [
    small(wl.KIND_GSPAR, 3, 1, k=1),
    small(wl.KIND_GSPAR, 5, 4095, k=41),
    small(wl.KIND_GSPAR, 4, 4096 * 2, k=4096 * 2),
    small(wl.KIND_GSPAR, 9, 4096 * 3 + 17, k=150, topo=wl.TOPO_TORUS2D, torus=(3, 3), grad="student_t3"),
    small(wl.KIND_GSPAR, 3, 4096 * 180 + 1, k=2500),
    small(wl.KIND_GSPAR, 3, 4096 * 90 + 1, k=36_000),
    small(wl.KIND_GSPAR, 35, 4096 * 2 + 2, k=900),
]
CASES += TOPK + GSPAR


def _plan(variant):
    return {"variant": variant}


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
@pytest.mark.parametrize("variant", [0, 3, 2])
def test_resident_lock_step(w, variant):
    say("case", w.name, "variant", variant)
    ds = b.DeepSqueeze.from_workload(w, _plan(variant))
    assert ("resident" in ds.ds_plan_name()) == (variant != 2), ds.ds_plan_name()
    for t in range(2):                                         # which way the step went: variant 3 must have been done by one workgroup
        ds.ds_step(upload(wl.gradient(w, t)))
        if variant == 3:
            assert ds.ds_topk_candidate_rows() == 0
        elif variant == 0 and w.kind != wl.KIND_TOPK:
            assert ds.ds_topk_candidate_rows() == w.n
    ds.ds_destroy()
    lock_step(w, steps=2, plan=_plan(variant))


@pytest.mark.parametrize("w", [CASES[3], CASES[4]] + TOPK + GSPAR, ids=lambda w: w.name)
@pytest.mark.parametrize("variant", [0, 3, 2])
def test_resident_free_run(w, variant):
    """Nothing read or written between the steps but the messages (the guesses of one step serve the next)."""
    ds = b.DeepSqueeze.from_workload(w, _plan(variant))
    st = oracle_state(w)
    for t in range(6):
        g = wl.gradient(w, t)
        ds.ds_step(upload(g))
        _, msg = oracle.step(st, g, want_cv=False)
        assert np.array_equal(ds.ds_read_messages(), msg), f"step {t}: messages differ"
    x, d = ds.ds_read_state()
    assert ds.ds_step_count() == 6
    ds.ds_destroy()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0


@pytest.mark.parametrize("w", [small(wl.KIND_QUANT_L2NORM, 40, 300, bits=4), small(wl.KIND_TOPK, 40, 300, k=60), small(wl.KIND_GSPAR, 40, 300, k=60)], ids=lambda w: w.name)
def test_resident_dense_graph(w):
    """Every worker averages with all 40: more neighbours than are put together at once."""
    n = w.n
    W = np.full((n, n), 1.0 / n, np.float32)
    csr = (np.arange(n + 1, dtype=np.int32) * n, np.tile(np.arange(n, dtype=np.int32), n), W.reshape(-1))
    lock_step(w, steps=2, W=W, csr=csr)


@pytest.mark.parametrize("k", [1, 700, 2600, 9000])
@pytest.mark.parametrize("variant", [0, 3, 2])
def test_resident_topk_many_equal_magnitudes(k, variant):
    """Values of seven levels, most of them zero and half of the columns without a gradient: hundreds of equal magnitudes at
    the threshold, which stays where it is for some steps and moves by a level, or to zero, in others."""
    w = small(wl.KIND_TOPK, 5, 4096 * 2 + 1001, k=k, gamma=1.0)
    rng = np.random.default_rng(k)
    level = lambda p: rng.choice(np.arange(-3, 4).astype(np.float32), size=(w.n, w.N), p=p)
    ds = b.DeepSqueeze.from_workload(w, _plan(variant))
    st = oracle_state(w)
    st.delta = level([0.05, 0.05, 0.1, 0.6, 0.1, 0.05, 0.05])
    ds.ds_write_state(st.x, st.delta, st.t)
    for t in range(8):
        g = level([0.01, 0.01, 0.08, 0.8, 0.08, 0.01, 0.01]) if t in (2, 5) else np.zeros((w.n, w.N), np.float32)
        ds.ds_step(upload(g))
        _, msg = oracle.step(st, g, want_cv=False)
        assert np.array_equal(ds.ds_read_messages(), msg), f"step {t}: messages differ"
    x, d = ds.ds_read_state()
    ds.ds_destroy()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0


@pytest.mark.parametrize("other", [small(wl.KIND_QUANT_L2NORM, 8, 4096 * 40 + 1001, bits=4, seed=9), TOPK[4], GSPAR[4]], ids=lambda w: w.name)
def test_two_resident_handles_on_two_streams(other):
    """Two handles step side by side on streams of their own; the second takes one launch or the chain, as there is room."""
    import torch
    ws = [CASES[4], other]
    dss = [b.DeepSqueeze.from_workload(w) for w in ws]
    sts = [oracle_state(w) for w in ws]
    streams = [torch.cuda.Stream() for _ in ws]
    gs = [[wl.gradient(w, t) for t in range(8)] for w in ws]
    ups = [[upload(g) for g in one] for one in gs]
    torch.cuda.synchronize()
    for t in range(8):
        for ds, up, s in zip(dss, ups, streams):
            ds.ds_step(up[t], s)
    for w, ds, st, one in zip(ws, dss, sts, gs):
        for g in one:
            oracle.step(st, g, want_cv=False, want_msg=False)
        x, d = ds.ds_read_state()
        ds.ds_destroy()
        assert assert_close(f"{w.name} x", x, st.x) + assert_close(f"{w.name} delta", d, st.delta) == 0


def _crowd(kind, variants, **kw):
    """Handles of 536 workgroups each, a stream for each."""
    import torch
    ws = [small(kind, 8, 272_474, seed=5 + q, **kw) for q in range(len(variants))]
    return ws, [b.DeepSqueeze.from_workload(w, _plan(v)) for w, v in zip(ws, variants)], [torch.cuda.Stream() for _ in ws]


KINDS = [(wl.KIND_QUANT_L2NORM, {"bits": 4}), (wl.KIND_TOPK, {"k": 2724}), (wl.KIND_GSPAR, {"k": 27_247})]


@pytest.mark.parametrize("kind,kw", KINDS)
@pytest.mark.parametrize("variants", [(0, 0, 0), (0, 0, 2), (0, 0, 0, 0)], ids=str)
def test_steps_that_start_together_on_several_streams(kind, kw, variants):
    """Three or four steps that the GPU has not got the room (or, next to another kernel's registers, not in the right pieces) to
    run in one launch each, set off together.  None may wait for its meeting in vain: that takes 10 ms, and a step of all of them
    some 0.1 ms."""
    import time

    import torch
    ws, dss, streams = _crowd(kind, variants, **kw)
    gs = [torch.randn((w.n, (w.N + 3) // 4 * 4), device="cuda") * 0.5 for w in ws]
    a = torch.randn((4096, 4096), device="cuda")
    out = torch.empty_like(a)
    torch.cuda.synchronize()
    took = []
    for _ in range(25):
        torch.mm(a, a, out=out)                                # the steps are enqueued while this keeps the GPU busy
        torch.mm(a, a, out=out)
        go = torch.cuda.Event()
        go.record()
        for ds, g, s in zip(dss, gs, streams):
            s.wait_event(go)
            ds.ds_step(g, s)
        go.synchronize()
        began = time.perf_counter()
        torch.cuda.synchronize()
        took.append(time.perf_counter() - began)
    for ds in dss:
        assert ds.ds_step_count() == 25
        ds.ds_destroy()
    took = sorted(took[3:])
    say("ms:", [round(1e3 * t, 3) for t in took])
    assert took[-3] < 5e-3, took                               # two of 22 may have been held up by something else


def test_steps_on_the_per_thread_default_streams():
    """hipStreamPerThread names another stream in every thread: four threads step a handle each, all at once."""
    import threading
    import time

    import torch
    ws, dss, _ = _crowd(wl.KIND_QUANT_L2NORM, (0, 0, 0, 0), bits=4)
    ups = [[upload(wl.gradient(w, t)) for t in range(2)] for w in ws]
    torch.cuda.synchronize()
    steps, meet, took, failed = 20, threading.Barrier(len(ws)), [], []

    def work(ds, gs, first):
        torch.cuda.set_device(0)
        for t in range(steps):
            meet.wait(30)
            began = time.perf_counter()
            if ds.ds_step_raw(gs[t % 2].data_ptr(), gs[t % 2].stride(0), 2) != b.DS_OK:
                failed.append(t)
            meet.wait(30)
            if first:
                torch.cuda.synchronize()
                took.append(time.perf_counter() - began)

    threads = [threading.Thread(target=work, args=(ds, gs, q == 0)) for q, (ds, gs) in enumerate(zip(dss, ups))]
    for th in threads:
        th.start()
    for th in threads:
        th.join(60)
    assert not failed and not any(th.is_alive() for th in threads)
    say("ms:", [round(1e3 * t, 2) for t in took])
    assert sorted(took[2:])[-3] < 5e-3, took
    st = oracle_state(ws[3])
    for t in range(steps):
        oracle.step(st, wl.gradient(ws[3], t % 2), want_cv=False, want_msg=False)
    x, d = dss[3].ds_read_state()
    for ds in dss:
        assert ds.ds_step_count() == steps
        ds.ds_destroy()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0


@pytest.mark.parametrize("kind,kw", KINDS)
def test_one_launch_and_chain_take_turns(kind, kw):
    """A handle whose stream finds no room next to two others takes the launches of large problems, and one launch again on a stream
    that has room: both work on the same state.  Messages after every step, x and delta after every other one."""
    import torch
    _, others, streams = _crowd(kind, (0, 0), **kw)
    w = small(kind, 8, 272_474, seed=3, **kw)
    st = oracle_state(w)
    ds = b.DeepSqueeze.from_workload(w)
    third = torch.cuda.Stream()
    g0 = upload(wl.gradient(w, 0))
    for ds_, s in zip(others, streams):
        ds_.ds_step(g0, s)                                   # takes its seat
    for t, s in enumerate([third, streams[0], streams[0], third, third, streams[1], third, streams[0]]):
        g = wl.gradient(w, t)
        gd = upload(g)
        torch.cuda.synchronize()
        ds.ds_step(gd, s)
        _, msg = oracle.step(st, g, want_cv=False)
        torch.cuda.synchronize()
        assert np.array_equal(ds.ds_read_messages(), msg), f"step {t}: messages differ"
        if t % 2:
            x, d = ds.ds_read_state()
            assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0, f"step {t}"
    for ds_ in others:
        ds_.ds_destroy()
    g = wl.gradient(w, 8)
    ds.ds_step(upload(g), third)                             # there is room now
    _, msg = oracle.step(st, g, want_cv=False)
    assert np.array_equal(ds.ds_read_messages(), msg)
    x, d = ds.ds_read_state()
    assert ds.ds_step_count() == 9
    ds.ds_destroy()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0


@pytest.mark.parametrize("k", [1, 64, 65, 128, 129, 300])
@pytest.mark.parametrize("n,torus", [(5, None), (9, (3, 3)), (8, "dense")])
def test_sparse_tail_by_fullness_of_a_chunk(k, n, torus):
    """Everything that is sent lies in one chunk of four, in some of the same columns for all workers: the tail on its own with
    one pair per lane, two, and more than a wave takes at once; with 3, 5 and 8 neighbours."""
    w = small(wl.KIND_TOPK, n, 4096 * 3 + 1001, k=k, **({"topo": wl.TOPO_TORUS2D, "torus": torus} if isinstance(torus, tuple) else {}))
    W = np.full((n, n), 1.0 / n, np.float32) if torus == "dense" else None
    if W is not None:
        cfg, keep = b.make_config(n, w.N, wl.TOPO_CSR, w.kind, w.gamma, w.eta, k=k, seed=w.seed,
                                  W_csr=(np.arange(n + 1, dtype=np.int32) * n, np.tile(np.arange(n, dtype=np.int32), n), W.reshape(-1)))
        ds = b.DeepSqueeze(cfg, keep, _plan(2))
    else:
        ds = b.DeepSqueeze.from_workload(w, _plan(2))
    st = oracle_state(w, W)
    rng = np.random.default_rng(k)
    st.delta = rng.normal(size=(n, w.N)).astype(np.float32)
    st.delta[:, 4096 + 7:4096 + 7 + 2 * k:2] *= 1000.0
    ds.ds_write_state(st.x, st.delta, st.t)
    for t in range(3):
        g = wl.gradient(w, t)
        ds.ds_step(upload(g))
        _, msg = oracle.step(st, g, want_cv=False)
        assert np.array_equal(ds.ds_read_messages(), msg), f"step {t}: messages differ"
        x, d = ds.ds_read_state()
        assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0, f"step {t}"
    ds.ds_destroy()
