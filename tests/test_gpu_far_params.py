"""Spans of far sums follow the parameters in force: a handle whose parameters
were set after its start steps bit for bit as one that was made with them."""
import math

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Solver():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_06123_amd import Solver as S
    return S


# spans of 32 steps <-> none, <-> 128 (a channel without thinning), and the
# same values again
@pytest.mark.parametrize("first,then", [(0.1, 1e-3), (1e-3, 0.1), (0.1, math.inf),
                                        (math.inf, 0.02), (0.1, 0.1)])
@pytest.mark.parametrize("kind", ["uni", "2d", "finger", "two"])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_spans_follow_set_params(Solver, precision, kind, first, then):
    base = workloads.plain_f64().channels[0].replace(
        lx=1 if kind in ("uni", "two") else 3, ly=24, n_hist=600, tau_m=60.0, gx=2e-5,
        finger=kind == "finger")
    chans = [base] + ([base.replace(ly=40, n_hist=900)] if kind == "two" else [])
    print(f"case set_params {kind} {precision} {first} -> {then}", flush=True)
    out = []
    start = None
    for gamma_c in (then, first):
        with Solver([c.replace(gamma_c=gamma_c) for c in chans], precision=precision) as s:
            s.set_block(16 if kind == "finger" else 32)
            s.set_graph(64)
            if start is None:
                start = s.save_state()
            else:
                s.step(64)  # spans of the first parameters, their graph
                for i, c in enumerate(chans):
                    assert s.lib.lb_set_params(s.h, i, c.g_inf, c.tau_m, then) == 0
            s.load_state(start)
            for n in (200, 90, 64, 1):
                s.step(n)
            out.append([v for i in range(len(chans)) for v in s.fields(i) + s.stress(i)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
