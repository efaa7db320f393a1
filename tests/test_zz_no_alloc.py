"""ds_step_static (one step on caller-owned arrays, nothing allocated, nothing in device memory beside them) against
ds_step on a handle: bit for bit, on calls in a row, later ones with a smaller input, and on two streams at once."""
import numpy as np
import pytest
import torch

from paper_1907_07346_amd import binding as b
from paper_1907_07346_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _case(n, N, topo, torus, kind, bits, block, seed, t):
    w = wl.Config(f"static_n{n}_N{N}_k{kind}", n=n, N=N, topo=topo, torus=torus, kind=kind, gamma=0.1, eta=0.4, steps=1,
                  grad="normal", grad_scale=0.5, bits=bits, block=block, seed=seed)
    x0, d0 = wl.random_state(w, seed=seed + 100)
    g = wl.gradient(w, t)
    return w, x0, d0, g, t


def _by_handle(w, x0, d0, g, t):
    ds = b.DeepSqueeze.from_workload(w)
    ds.ds_write_state(x0, d0, t)
    pitch = (w.N + 3) // 4 * 4
    gd = torch.zeros((w.n, pitch), dtype=torch.float32, device="cuda")
    gd[:, :w.N] = torch.from_numpy(g).cuda()
    ds.ds_step(gd)
    x, d = ds.ds_read_state()
    m = ds.ds_read_messages()
    ds.ds_destroy()
    return x, d, m


def _static(w, x0, d0, g, t):
    cfg, _ = b.config_from_workload(w)
    ld = (w.N + 4095) // 4096 * 4096 + 2560
    x = torch.zeros((w.n, ld), dtype=torch.float32, device="cuda")
    d = torch.zeros((w.n, ld), dtype=torch.float32, device="cuda")
    gd = torch.zeros((w.n, ld), dtype=torch.float32, device="cuda")
    x[:, :w.N] = torch.from_numpy(x0).cuda()
    d[:, :w.N] = torch.from_numpy(d0).cuda()
    gd[:, :w.N] = torch.from_numpy(g).cuda()
    msg = torch.full((b.ds_message_bytes(cfg),), 0xAB, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    b.ds_step_static(cfg, x, d, gd, msg, t)
    torch.cuda.synchronize()
    assert float(x[:, w.N:].abs().max()) == 0.0 and float(d[:, w.N:].abs().max()) == 0.0, "padding columns touched"
    return x[:, :w.N].cpu().numpy(), d[:, :w.N].cpu().numpy(), msg.cpu().numpy()


def test_static_step_equals_handle_step_twice_second_smaller():
    cases = [
        _case(64, 512 * 37 + 100, wl.TOPO_TORUS2D, (8, 8), wl.KIND_QUANT_MAXABS, 4, 512, seed=3, t=7),    # the larger input first
        _case(5, 1024 * 3 + 74, wl.TOPO_RING, (0, 0), wl.KIND_QUANT_MAXABS, 2, 1024, seed=4, t=2),        # then a smaller one
        _case(8, 256 * 11 + 40, wl.TOPO_RING, (0, 0), wl.KIND_SIGN_MEANABS, 0, 256, seed=5, t=0),
        _case(3, 700, wl.TOPO_RING, (0, 0), wl.KIND_IDENTITY, 0, 0, seed=6, t=1),
    ]
    for w, x0, d0, g, t in cases:
        print("case", w.name, flush=True)
        want = _by_handle(w, x0, d0, g, t)
        got = _static(w, x0, d0, g, t)
        assert np.array_equal(got[2], want[2]), f"{w.name}: messages differ"
        assert np.array_equal(got[0].view(np.uint32), want[0].view(np.uint32)), f"{w.name}: x differs"
        assert np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32)), f"{w.name}: delta differs"


Q4 = (wl.KIND_QUANT_MAXABS, 4, 512)


@pytest.mark.parametrize("n,torus,comp,N", [
    (9, (3, 3), Q4, 700), (15, (3, 5), Q4, 512 * 3 + 1), (15, (5, 3), Q4, 512 * 3 + 1), (24, (4, 6), (wl.KIND_SIGN_MEANABS, 0, 64), 901),
    (3, None, Q4, 1), (16, None, Q4, 512 * 2), (33, None, (wl.KIND_QUANT_MAXABS, 2, 1024), 1500), (65, None, Q4, 1100),
    (17, None, (wl.KIND_QUANT_MAXABS, 8, 2048), 2049), (300, None, Q4, 600), (300, (15, 20), Q4, 600), (500, None, (wl.KIND_SIGN_MEANABS, 0, 256), 513),
    (1024, None, (wl.KIND_SIGN_MEANABS, 0, 64), 300), (40, (5, 8), (wl.KIND_IDENTITY, 0, 0), 777)])
def test_static_step_by_graph_and_launch_shape(n, torus, comp, N):
    """The graph that the kernel works out for itself: sides of three (where the wrap-around changes the neighbours' order),
    rows and columns that differ, more entries than threads, the largest number of workers; and every rows-per-wave shape."""
    w, x0, d0, g, t = _case(n, N, wl.TOPO_TORUS2D if torus else wl.TOPO_RING, torus or (0, 0), *comp, seed=n, t=5)
    print("case", w.name, flush=True)
    want, got = _by_handle(w, x0, d0, g, t), _static(w, x0, d0, g, t)
    assert np.array_equal(got[2], want[2]), "messages differ"
    assert np.array_equal(got[0].view(np.uint32), want[0].view(np.uint32)) and np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32))


def test_static_steps_on_two_streams_share_nothing():
    """Two problems of different graphs, sizes and step numbers, a stream each, ten steps of both under way together."""
    steps = 10
    cases = [_case(15, 512 * 40 + 3, wl.TOPO_TORUS2D, (3, 5), *Q4, seed=11, t=0), _case(8, 256 * 90 + 1, wl.TOPO_RING, (0, 0), wl.KIND_QUANT_MAXABS, 2, 256, seed=12, t=100)]
    sides = []
    for w, x0, d0, g, t in cases:
        cfg, _ = b.config_from_workload(w)
        ld = (w.N + 4095) // 4096 * 4096
        rows = [torch.zeros((w.n, ld), device="cuda") for _ in range(3)]
        for a, v in zip(rows, (x0, d0, g)):
            a[:, :w.N] = torch.from_numpy(v).cuda()
        sides.append((cfg, rows, torch.zeros(b.ds_message_bytes(cfg), dtype=torch.uint8, device="cuda"), t, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for q in range(steps):
        for cfg, (x, d, g), msg, t, stream in sides:
            b.ds_step_static(cfg, x, d, g, msg, t + q, stream)
    torch.cuda.synchronize()
    for (w, x0, d0, _, t), (_, (x, d, g), msg, _, _) in zip(cases, sides):
        ds = b.DeepSqueeze.from_workload(w)
        ds.ds_write_state(x0, d0, t)
        for _ in range(steps):
            ds.ds_step(g)
        xw, dw = ds.ds_read_state()
        assert np.array_equal(msg.cpu().numpy(), ds.ds_read_messages()), f"{w.name}: messages differ"
        assert np.array_equal(x[:, :w.N].cpu().numpy().view(np.uint32), xw.view(np.uint32)), f"{w.name}: x differs"
        assert np.array_equal(d[:, :w.N].cpu().numpy().view(np.uint32), dw.view(np.uint32)), f"{w.name}: delta differs"
        ds.ds_destroy()


def test_static_step_refuses_what_it_does_not_serve():
    x = torch.zeros((4, 4096 + 2560), dtype=torch.float32, device="cuda")
    msg = torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")

    def attempt(**kw):
        args = dict(n=4, N=4000, topo=wl.TOPO_RING, kind=wl.KIND_QUANT_MAXABS, gamma=0.1, eta=0.4, bits=4, block=512)
        args.update(kw)
        cfg, keep = b.make_config(args.pop("n"), args.pop("N"), args.pop("topo"), args.pop("kind"), args.pop("gamma"),
                                  args.pop("eta"), **args)
        with pytest.raises(b.DsqError) as e:
            b.ds_step_static(cfg, x, x, x, msg, 0)
        assert e.value.status == b.DS_EINVAL
        return str(e.value)

    assert "1024" in attempt(n=1025, N=16)
    assert "serves" in attempt(kind=wl.KIND_TOPK, k=40)
    assert "serves" in attempt(kind=wl.KIND_RAND_SPARSE, k=40)
    rp, co, va = np.array([0, 1, 2, 3, 4], np.int32), np.arange(4, dtype=np.int32), np.ones(4, np.float32)
    assert "RING" in attempt(topo=wl.TOPO_CSR, W_csr=(rp, co, va))
    assert "ld" in attempt(N=7000)                                     # the arrays' pitch is too small for N
