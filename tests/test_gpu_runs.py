"""Steps that follow one another with x asked for only at the end: where the state is large enough (or small enough to stay in the L2s;
of any size where messages are whole values) the fused kernel has a form of its own that reads a part of the state with plain loads.
Sizes on both sides of the lines, ragged rows, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1907_07346_amd import binding as b
from paper_1907_07346_amd import workloads as wl
from test_gpu_parity import assert_close, oracle_state, say, small, upload

pytestmark = pytest.mark.gpu

MIB = 2**20 // 8                                             # elements whose x and delta take 1 MiB
CASES = [small(wl.KIND_QUANT_MAXABS, 9, 72 * MIB // 9 + 35, bits=4, block=512), small(wl.KIND_QUANT_MAXABS, 3, 72 * MIB // 3 - 1, bits=2, block=1024),
         small(wl.KIND_QUANT_MAXABS, 20, 72 * MIB // 20 + 1, bits=8, block=64), small(wl.KIND_SIGN_MEANABS, 5, 72 * MIB // 5 + 1, block=256),
         small(wl.KIND_SIGN_MEANABS, 5, 20 * MIB // 5 + 3, block=256), small(wl.KIND_RAND_SPARSE, 5, 128 * MIB // 5 + 1, k=33_000),
         small(wl.KIND_IDENTITY, 5, 100_003), small(wl.KIND_IDENTITY, 3, 700)]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_runs_of_steps(w):
    say("case", w.name, w.n * w.N / MIB, "MiB")
    ds = b.DeepSqueeze.from_workload(w)
    st = oracle_state(w)
    gs = [wl.gradient(w, t) for t in range(2)]
    gd = [upload(g) for g in gs]
    t = 0
    for run in (3, 1, 2):
        for _ in range(run):
            ds.ds_step(gd[t % 2])
            _, msg = oracle.step(st, gs[t % 2], want_cv=False)
            t += 1
        x, d = ds.ds_read_state()
        assert assert_close("x", x, st.x) + assert_close("delta", d, st.delta) == 0, (run, t)
        assert np.array_equal(ds.ds_read_messages(), msg), (run, t)
    ds.ds_destroy()
