"""A training loop captured into a graph whole: x borrowed (which completes the last step), read, then the step.  The borrowing has
to be in the graph whatever was pending when it was captured, and to do the right thing in every replay."""
import pytest
import torch

import oracle
from paper_1907_07346_amd import binding as b
from paper_1907_07346_amd import workloads as wl
from test_gpu_parity import _device_view, assert_close, oracle_state, say, small, upload

pytestmark = pytest.mark.gpu

CASES = [(small(wl.KIND_TOPK, 8, 4096 * 3 + 1001, k=130), {"variant": 2}), (small(wl.KIND_TOPK, 8, 30_011, k=300), {}),
         (small(wl.KIND_GSPAR, 8, 4096 * 3 + 1001, k=900), {"variant": 2}),
         (small(wl.KIND_QUANT_L2NORM, 8, 4096 * 3 + 1001, bits=4), {"variant": 2}),
         (small(wl.KIND_QUANT_MAXABS, 33, 512 * 3 + 77, bits=4, block=512), {"variant": 1, "tile_plan": 0}),
         (small(wl.KIND_QUANT_MAXABS, 33, 512 * 3 + 77, bits=4, block=512), {"variant": 1, "tile_plan": 1}),
         (small(wl.KIND_SIGN_MEANABS, 40, 256 * 9 + 37, block=256), {})]


@pytest.mark.parametrize("warm", ["s", "sr", "ssr", "ss", "srsr"])
@pytest.mark.parametrize("w,plan", CASES, ids=lambda v: v.name if hasattr(v, "name") else "-".join(map(str, v.values())) or "auto")
def test_borrow_and_step_in_a_graph(w, plan, warm):
    """warm: eager steps (s) and borrowings (r) before the capture; between the replays eager steps, reads and neither."""
    say("case", w.name, plan, warm)
    ds = b.DeepSqueeze.from_workload(w, plan)
    st = oracle_state(w)
    side = torch.cuda.Stream()
    gd = upload(wl.gradient(w, 0))
    torch.cuda.synchronize()
    t = 0

    def feed():
        nonlocal t
        g = wl.gradient(w, t)
        gd[:, :w.N].copy_(torch.from_numpy(g).cuda())
        torch.cuda.synchronize()
        t += 1
        return g

    with torch.cuda.stream(side):
        for what in warm:
            if what == "s":
                g = feed()
                ds.ds_step(gd, side)
                oracle.step(st, g, want_cv=False, want_msg=False)
            else:
                ds.ds_state_ptrs()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        xp, _, ld = ds.ds_state_ptrs()
        seen = _device_view(xp, (w.n, ld))[:, :w.N].clone()
        ds.ds_step(gd, side)
    for after in ["", "", "r", "", "sr", "", "s", "", ""]:
        before = st.x.copy()
        g = feed()
        graph.replay()
        torch.cuda.synchronize()
        assert assert_close(f"{warm} {t} borrowed x", seen.cpu().numpy(), before) == 0
        oracle.step(st, g, want_cv=False, want_msg=False)
        for what in after:
            if what == "s":
                g = feed()
                ds.ds_step(gd, side)
                oracle.step(st, g, want_cv=False, want_msg=False)
                torch.cuda.synchronize()
            else:
                ds.ds_state_ptrs()
        torch.cuda.synchronize()
    x, d = ds.ds_read_state()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0
    assert ds.ds_step_count() == t
    ds.ds_destroy()


@pytest.mark.parametrize("warm", ["", "s", "sr", "ss"])
@pytest.mark.parametrize("w,plan", CASES, ids=lambda v: v.name if hasattr(v, "name") else "-".join(map(str, v.values())) or "auto")
def test_borrow_and_step_in_a_graph_of_another_stream(w, plan, warm):
    """The same graph where the steps before it, if there are any, ran on another stream than the one that is captured: borrowing x enqueues
    nothing into it, so that its step has to leave x complete, and so do the eager steps between the replays."""
    say("case", w.name, plan, warm)
    ds = b.DeepSqueeze.from_workload(w, plan)
    st = oracle_state(w)
    first, side = torch.cuda.Stream(), torch.cuda.Stream()
    gd = upload(wl.gradient(w, 0))
    torch.cuda.synchronize()
    t = 0

    def feed():
        nonlocal t
        g = wl.gradient(w, t)
        gd[:, :w.N].copy_(torch.from_numpy(g).cuda())
        torch.cuda.synchronize()
        t += 1
        return g

    def eager(what, stream):
        if what == "r":
            ds.ds_state_ptrs()
        else:
            g = feed()
            ds.ds_step(gd, stream)
            oracle.step(st, g, want_cv=False, want_msg=False)
        torch.cuda.synchronize()

    for what in warm:
        eager(what, first)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        xp, _, ld = ds.ds_state_ptrs()
        seen = _device_view(xp, (w.n, ld))[:, :w.N].clone()
        ds.ds_step(gd, side)
    for after in ["", "", "r", "", "sr", "", "s", "", "ss", "", ""]:
        before = st.x.copy()
        g = feed()
        graph.replay()
        torch.cuda.synchronize()
        assert assert_close(f"{warm} {t} borrowed x", seen.cpu().numpy(), before) == 0
        oracle.step(st, g, want_cv=False, want_msg=False)
        for what in after:
            eager(what, first)
    x, d = ds.ds_read_state()
    assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0
    assert ds.ds_step_count() == t
    ds.ds_destroy()
