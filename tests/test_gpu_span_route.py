"""Which of the passes over the history a run takes, and the general pass in
its launch shapes where spans of far sums would otherwise take its place (a
fresh block for every step, or a grid channel in the handle)."""
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


def outputs(s, ci=0):
    _, ux, uy = s.fields(ci)
    return (ux, uy) + s.stress(ci)


def error(a, b):
    """Largest error of the velocity and of the stress, each over its scale."""
    out = 0.0
    for group in ((0, 1), (2, 3)):
        scale = max(np.abs(b[k]).max() for k in group)
        out = max([out] + [np.abs(a[k] - b[k]).max() / scale for k in group])
    return float(out)


def base(**kw):
    return workloads.plain_f64().channels[0].replace(
        **{**dict(lx=4, ly=64, n_hist=600, tau_m=60.0, gx=2e-5), **kw})


def jet(**kw):
    u0 = np.zeros((2, 64, 8))
    u0[0, 20:24] = 0.08
    return base(lx=8, u0=u0, gx=0.0, gamma_c=0.1, **kw)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["2d", "uni", "finger"])
def test_smooth_flows_mark_no_tile_and_a_jet_marks_some(Solver, precision, kind):
    print(f"case routes {kind} {precision}", flush=True)
    kw = dict(uni=dict(lx=1), finger=dict(finger=True)).get(kind, {})
    with Solver([base(**kw)], precision=precision) as s:
        s.set_block(16 if kind == "finger" else 32)
        assert s.run_info() == dict(span=128, span_pos=0, graph_launches=0,
                                    far_tiles=1 if kind == "uni" else 4, marked_tiles=0)
        for n in (100, 300, 500):
            s.step(n)
            assert s.run_info()["marked_tiles"] == 0
        assert s.run_info()["span_pos"] == 900 % 128
    if kind == "uni":
        return
    with Solver([jet(**kw)], precision=precision) as s:
        s.set_block(16 if kind == "finger" else 32)
        marks = []
        for n in (150,) * 4:
            s.step(n)
            marks.append(s.run_info()["marked_tiles"])
        assert s.run_info()["far_tiles"] == 8
        assert any(0 < m < 8 for m in marks), marks


def test_settings_that_take_no_spans(Solver):
    print("case settings without spans", flush=True)
    grid = base(hist_blocks=4, hist_block_len=40)
    for chans, block, span in (([base(n_hist=127)], 32, 0), ([base(n_hist=128)], 32, 32),
                               ([base(lx=1)], 1, 0), ([base(lx=1)], 8, 128), ([base()], 1, 128),
                               ([base(), grid], 8, 0), ([base(), grid], 32, 128),
                               ([base(finger=True), base()], 16, 0),
                               ([base(gamma_c=1e-3)], 32, 0),
                               ([base(ly=32)], 32, 32), ([base(ly=36)], 32, 64),
                               # spans of 32 steps: not beyond 65536 nodes
                               ([base(lx=2048, ly=32, gamma_c=0.05)], 32, 32),
                               ([base(lx=2049, ly=32, gamma_c=0.05)], 32, 0),
                               ([base(lx=2049, ly=32)], 32, 64),
                               ([base(law="strain_damping", gamma_c=1e-3)], 32, 128)):
        with Solver(chans, precision="f32") as s:
            s.set_block(block)
            assert s.run_info()["span"] == span, (chans, block)


def test_general_pass_lane_widths(Solver):
    """Widths 1 and 2 group the same rows per partial sum: bit for bit; 4 to
    rounding (FP32: the bounds of the lane-width test of short runs)."""
    ch = base(lx=40, ly=30, n_hist=700)
    print("case general pass, lane widths", flush=True)
    for precision, tol in (("f32", 1e-6), ("f64", 1e-13)):
        got = []
        for vec in (1, 2, 4):
            with Solver([ch], precision=precision) as s:
                for _ in range(300):
                    s.set_tiling(0, 3, vec)
                    s.set_block(1)
                    assert s.tiling(0) == (3, vec)
                    s.step(1)
                assert s.run_info()["marked_tiles"] == 0
                got.append(outputs(s))
        assert all(np.array_equal(a, b) for a, b in zip(got[0], got[1])), precision
        assert error(got[2], got[0]) < tol, precision


@pytest.mark.parametrize("kind", ["2d", "uni", "strain", "finger"])
def test_general_pass_block_lengths(Solver, kind):
    """Blocks of 2 to 16 steps of the general pass, lane widths where it has
    them, and spans, against a fresh pass per step in FP64."""
    kw = dict(uni=dict(lx=1), strain=dict(law="strain_damping"), finger=dict(finger=True))
    ch = base(**kw.get(kind, {}))
    grid = base(lx=1, ly=16, hist_blocks=4, hist_block_len=40)
    # beside the tensor, another window channel keeps the handle off the spans
    beside = base(ly=8, n_hist=40) if kind == "finger" else grid
    print(f"case general pass, block lengths {kind}", flush=True)
    with Solver([ch], precision="f64") as s:
        for _ in range(760):
            s.set_block(1)
            s.step(1)
        want = outputs(s)
    for block, vec in ((2, 1), (2, 2), (4, 1), (4, 2), (8, 1), (16, 1)):
        with Solver([ch, beside], precision="f64") as s:
            s.set_block(block)
            s.set_tiling(0, min(2, s.max_chunks(0)), vec)
            s.step(760)
            assert s.run_info()["span"] == 0
            assert error(outputs(s), want) < 1e-12, (block, vec)
    with Solver([ch], precision="f64") as s:
        s.set_block(16 if kind == "finger" else 32)
        s.step(760)
        assert s.run_info()["span_pos"] == 760 % 128
        assert error(outputs(s), want) < 1e-12


# old entries far slower than the newest: the oldest far one, one row before it,
# the older half, one column of nodes alone, and none
@pytest.mark.parametrize("rows", ["last", "one", "half", "column", "none"])
@pytest.mark.parametrize("kind,chunks", [("2d", 1), ("2d", 9), ("uni", 1), ("uni", 9),
                                         ("finger", 1)])
def test_old_rates_beyond_the_expansion(Solver, kind, chunks, rows):
    from test_gpu_far_rates import channel, history, run_general, written_state
    ch = channel(kind, 288, 900, tau_m=1000.0, gamma_c=0.02)
    print(f"case old rates beyond the expansion {kind} {chunks} {rows}", flush=True)
    s = history(ch, 0.002)
    slow = s[0] * np.float32(0.2)
    if rows in ("last", "one"):
        s[900 - 128 - 2 - (0 if rows == "last" else 11)] = slow
    elif rows == "half":
        s[450:] = slow
    elif rows == "column":
        s[450:, 70] = slow[70]
    want = run_general(Solver, ch, "f64", s, 40)
    for precision, tol in (("f64", 1e-12), ("f32p64", 1e-5)):
        with Solver([ch], precision=precision) as sol:
            sol.set_block(16 if kind == "finger" else 32)
            sol.set_tiling(0, min(chunks, sol.max_chunks(0)), 1)
            sol.load_state(written_state(ch, precision, s))
            sol.step(40)
            info = sol.run_info()
            got = outputs(sol)
        tiles = -(-ch.nodes // 64)
        assert info["far_tiles"] == tiles
        assert info["marked_tiles"] == {"none": 0, "column": 1}.get(rows, tiles)
        assert error(got, tuple(want[k] for k in ("ux", "uy", "sxy", "n1"))) < tol
