"""Spans of far sums and the calls that a run is cut into: where a span begins
follows from the steps done, so the cuts change nothing, and a saved state
goes on inside its span."""
import struct

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


JET = np.zeros((2, 60, 8))
JET[0, 20:24] = 0.08


def channels(kind):
    base = workloads.plain_f64().channels[0].replace(lx=3, ly=60, n_hist=600, tau_m=60.0, gx=2e-5)
    uni = base.replace(lx=1)
    return {"2d": [base], "uni": [uni], "finger": [base.replace(finger=True)],
            "strain": [base.replace(law="strain_damping")],
            # tiles that fall back beside ones that hold
            "jet": [base.replace(lx=8, gx=0.0, u0=JET)], "jet finger": [
                base.replace(lx=8, gx=0.0, u0=JET, finger=True)],
            "coupling": [base.replace(paper_coupling=True)],
            # spans of 128, 32 and no steps side by side, and a strain window
            "mixed": [base, uni.replace(ly=20, n_hist=300), uni.replace(n_hist=90),
                      base.replace(law="strain_damping", n_hist=200)],
            # spans only where the block is the grid's
            "grid": [base, base.replace(hist_blocks=4, hist_block_len=40)]}[kind]


def outputs(s):
    return [v for i in range(len(s.channels)) for v in s.fields(i) + s.stress(i)]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def close(a, b):
    """FP64 rounding apart: 1e-12 of the largest density, speed and stress."""
    for i in range(0, len(b), 5):
        for group in ((0,), (1, 2), (3, 4)):
            scale = max(np.abs(b[i + k]).max() for k in group)
            if any(np.abs(a[i + k] - b[i + k]).max() >= 1e-12 * scale for k in group):
                return False
    return True


def split(s, kind):
    """Windows split into many short chunks: one wavefront per far tile."""
    if kind.startswith("jet"):
        s.set_tiling(0, s.max_chunks(0), 1)


def run(Solver, kind, precision, block, calls, graph=0, **kw):
    with Solver(channels(kind), precision=precision) as s:
        split(s, kind)
        s.set_block(block)
        s.set_graph(graph)
        s.set_fused(kw.get("fused", 1))
        for n in calls:
            s.step(n)
        return outputs(s)


CUTS = [(100, 233), (1,) * 40 + (293,), (7, 64, 128, 134), (32, 32, 64, 1, 204), (332, 1)]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["2d", "uni", "finger", "strain", "coupling", "mixed", "grid",
                                  "jet", "jet finger"])
def test_cuts_change_nothing(Solver, kind, precision):
    print(f"case cuts {kind} {precision}", flush=True)
    top = 16 if kind.endswith("finger") else 32
    for block in (1, 8, top):
        whole = run(Solver, kind, precision, block, (333,))
        for calls in CUTS:
            assert same(run(Solver, kind, precision, block, calls), whole), (block, calls)
        for graph in (top, 64, 160, 256):
            for calls in ((333,), CUTS[2]):
                assert same(run(Solver, kind, precision, block, calls, graph=graph), whole), \
                    (block, graph, calls)
    assert same(run(Solver, kind, precision, top, CUTS[2], fused=0), whole)


@pytest.mark.parametrize("kind", ["2d", "uni", "finger", "strain", "mixed", "grid", "jet",
                                  "jet finger"])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_a_saved_state_goes_on_inside_its_span(Solver, kind, precision):
    print(f"case resume {kind} {precision}", flush=True)
    top = 16 if kind.endswith("finger") else 32
    for block in (1, 8, top):
        for at in (1, 5, 48, 64, 128, 129, 200):
            with Solver(channels(kind), precision=precision) as s:
                split(s, kind)
                s.set_block(block)
                s.step(at)
                buf = s.save_state()
                s.step(150)
                want = outputs(s)
                s.step(33)
                s.load_state(buf)
                s.step(90)
                s.step(60)
                assert same(outputs(s), want), (block, at, "same handle")
            for graph, n in ((2 * top, 150), (block, 10)):
                with Solver(channels(kind), precision=precision) as s:
                    split(s, kind)
                    s.set_block(block)
                    s.set_graph(graph)
                    s.load_state(buf)
                    for _ in range(150 // n):
                        s.step(n)
                    assert same(outputs(s), want), (block, at, "new handle", graph)


def test_states_of_other_settings(Solver):
    """A state loads where it did: at a block's end into any block length,
    inside one into the same; one without a span position (a handle that takes
    none, and earlier files) finishes its block and starts a span."""
    print("case states of other settings", flush=True)
    ch = channels("2d")
    with Solver(ch, precision="f64") as s:
        s.set_block(8)
        s.step(205)
        inside = s.save_state()
        s.step(3)
        ended = s.save_state()
        s.step(100)
        want = outputs(s)
    from paper_1504_06123_amd import LBError
    for block in (1, 4, 8, 32):
        with Solver(ch, precision="f64") as s:
            s.set_block(block)
            if block == 8:
                s.load_state(inside)
                s.step(103)
                assert same(outputs(s), want)
            else:
                with pytest.raises(LBError):
                    s.load_state(inside)
            s.load_state(ended)
            s.step(100)
            assert close(outputs(s), want), block
    # a general 32-step block left after 20 steps: the span position taken out
    # of a state whose span has just begun leaves that
    with Solver(ch, precision="f64") as s:
        s.set_block(32)
        s.step(128 + 20)
        old = s.save_state()
        s.step(100)
        want = outputs(s)
        head = old[:256].cpu().numpy()
        assert struct.unpack_from("<i", head, 28)[0] == (128 << 16) + 20
        old[28:32] = 0
        s.load_state(old)
        s.step(100)
        assert close(outputs(s), want)


def test_tiling_set_inside_a_span(Solver):
    """Another chunk split takes effect at the next block; rounding only."""
    print("case tiling inside a span", flush=True)
    for kind in ("2d", "finger", "uni", "strain"):
        out = []
        for chunks in (1, 3):
            with Solver(channels(kind), precision="f64") as s:
                s.set_block(16 if kind == "finger" else 32)
                s.step(170)
                s.set_tiling(0, min(chunks, s.max_chunks(0)), 1)
                s.step(100)
                out.append(outputs(s))
        assert close(*out), kind


def test_a_gradient_does_not_depend_on_the_sampling(Solver):
    """The forward run is cut at the samples, its replay at the segments."""
    import torch
    from paper_1504_06123_amd import adjoint
    print("case gradient and sampling", flush=True)
    ch = workloads.plain_f64().channels[0].replace(lx=1, ly=60, n_hist=600, tau_m=60.0, gx=2e-5)
    got = []
    for block in (8, 32):
        for every in (600, 150, 100):
            with Solver([ch], precision="f32") as s:
                s.set_block(block)
                s.set_graph(64)
                theta = torch.tensor([[ch.g_inf, ch.tau_m, ch.gamma_c, ch.gx]],
                                     dtype=torch.float64, requires_grad=True)
                u = adjoint.LBFunction.apply(theta, s, s.save_state(), 600, every, 250)
                (u[-1] ** 2).sum().backward()
                got.append((u[-1].detach().numpy(), theta.grad.numpy()))
    for u, g in got[1:]:
        assert np.array_equal(u, got[0][0]) and np.array_equal(g, got[0][1])


@pytest.mark.parametrize("kind,block,graph,calls,launches", [
    ("2d", 32, 64, (64,) * 6, 6),          # a graph at each of a span's halves
    ("2d", 32, 96, (96,) * 8, 8),          # four places, one after the other
    ("2d", 32, 64, (64, 340), 4),          # to a span's end, two whole spans, 20 by themselves
    ("2d", 32, 256, (300, 300), 2),        # whole spans: 256 of 300, then from 384 on
    ("uni", 8, 8, (8,) * 40, 40),          # shorter than a span's block
    ("uni", 1, 64, (130, 64), 3),          # no spans
    ("2d", 1, 5, (1,) + (5,) * 30, 30),    # any place
    ("finger", 16, 48, (48,) * 9, 9),
])
def test_graphs_of_the_length_set(Solver, kind, block, graph, calls, launches):
    """A call of as many steps as the graph is long replays one, wherever in a
    span it starts, and the results are the plain launches'."""
    print(f"case graph length {kind} {block} {graph}", flush=True)
    with Solver(channels(kind), precision="f32") as s:
        s.set_block(block)
        s.set_graph(graph)
        for n in calls:
            s.step(n)
        assert s.run_info()["graph_launches"] == launches
        got = outputs(s)
    assert same(got, run(Solver, kind, "f32", block, calls))
