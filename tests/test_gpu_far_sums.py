"""Spans of far sums (one window pass for up to 128 steps of an lb_step call).

A call of n steps against n calls of one step: single steps of a 2D or
window-blocked handle never take far sums, so they are the general path.
FP64: the sums differ by rounding and by the expansion's truncation (1e-16
of each term), so 1e-12 of the field's scale, the bound of the other
launch-shape comparisons; FP32: the FP32 tolerances against the oracle.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Solver():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_06123_amd import Solver as S
    return S


def nerr(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


def twod(lx, ly, n_hist, **kw):
    return workloads.large_2d(lx=lx, ly=ly, n_hist=n_hist).channels[0].replace(
        **{"tau_m": 60.0, **kw})


def uni(ly, n_hist, **kw):
    return workloads.plain_f64().channels[0].replace(lx=1, ly=ly, n_hist=n_hist, gx=2e-5,
                                                     **{"tau_m": 60.0, **kw})


def advance(Solver, chans, precision, calls, block=1, chunks=None, persistent=False, graph=0,
            fused=1):
    out = []
    with Solver(chans, precision=precision) as s:
        for ci, nc in enumerate(chunks or []):
            s.set_tiling(ci, nc, 1)
        s.set_block(block)
        s.set_persistent(persistent)
        s.set_graph(graph)
        s.set_fused(fused)
        for n in calls:
            s.step(n)
        for ci in range(len(chans)):
            _, ux, _ = s.fields(ci)
            out.append((ux,) + s.stress(ci))
    return out


# windows at and around four spans of 32, 64 and 128 steps; node counts around
# one and four wavefronts and one node tile; window ends inside and outside
# the far ages; chunks whose far part is empty
@pytest.mark.parametrize("lx,ly,n_hist,chunks", [
    (3, 21, 127, None), (2, 32, 128, None), (5, 13, 129, None), (8, 32, 255, [1]),
    (3, 43, 256, [2]), (16, 16, 300, [2]), (9, 57, 511, [3]), (7, 37, 512, [4]),
    (65, 16, 640, [5]), (4, 32, 700, [1]),
])
def test_calls_of_many_steps_equal_single_steps_f64(Solver, lx, ly, n_hist, chunks):
    ch = twod(lx, ly, n_hist)
    print(f"case far sums {lx}x{ly}, window {n_hist}, chunks {chunks}", flush=True)
    calls = [200, 150, 8, 7, 31, 32, 33, 64, 100, 129]  # past the window's first fill
    one = advance(Solver, [ch], "f64", [1] * sum(calls), chunks=chunks)[0]
    for block, fused in ((1, 1), (8, 1), (32, 0)):
        got = advance(Solver, [ch], "f64", calls, block=block, chunks=chunks, fused=fused)[0]
        for k, a, b in zip(("ux", "sxy", "n1"), got, one):
            assert nerr(a, b) < 1e-12, (block, k, nerr(a, b))


@pytest.mark.parametrize("precision", ["f32", "f32p64"])
@pytest.mark.parametrize("case", ["2d", "uni", "uneven"])
def test_far_sums_f32_match_the_oracle(Solver, precision, case):
    chans = {"2d": [twod(24, 40, 600)], "uni": [uni(96, 2000, tau_m=200.0)],
             # windows too short for far sums beside ones that take them
             "uneven": [uni(16, 520), uni(130, 40), uni(70, 900), uni(257, 1500)]}[case]
    print(f"case far sums {case} {precision}", flush=True)
    got = advance(Solver, chans, precision, [300, 77, 400], block=32)
    for ch, g in zip(chans, got):
        oc = oracle.OracleChannel(ch)
        oc.step(777)
        _, ux, _ = oc.fields()
        for k, tol, a, b in zip(("ux", "sxy", "n1"), (1e-5, 1e-4, 1e-4), g, (ux,) + oc.stress()):
            assert nerr(a, b) < tol, (k, nerr(a, b))


def test_launch_forms_are_bitwise_equal(Solver):
    """Graph replay, the persistent general pass and fused in-block steps
    change nothing: spans follow from the call's length alone."""
    chans = [uni(40, 900), uni(100, 600, gamma_c=0.002), uni(130, 60)]
    print("case far sums, launch forms", flush=True)
    base = advance(Solver, chans, "f32", [300, 200], block=32, fused=0)
    for kw in (dict(graph=64), dict(persistent=True), dict(fused=2), dict(fused=1, graph=32)):
        got = advance(Solver, chans, "f32", [300, 200], block=32, **{"fused": 0, **kw})
        for a, b in zip(base, got):
            for x, y in zip(a, b):
                assert np.array_equal(x, y), kw


@pytest.mark.parametrize("precision,tol", [("f64", 1e-12), ("f32", 1e-4)])
@pytest.mark.parametrize("chunks", [[1], [4]])
def test_rates_beyond_the_expansion_take_the_general_pass(Solver, precision, tol, chunks):
    """A jet whose shear rates leave the expansion in part of the channel:
    its tiles fall back, the others keep their far sums."""
    ly, lx = 64, 8
    u0 = np.zeros((2, ly, lx))
    u0[0, 20:24] = 0.08
    ch = twod(lx, ly, 600, u0=u0, gx=0.0, gamma_c=0.1)
    calls = [64, 200, 300]
    print(f"case far sums, rates beyond the expansion, {precision}, chunks {chunks}", flush=True)
    one = advance(Solver, [ch], precision, [1] * sum(calls), chunks=chunks)[0]
    got = advance(Solver, [ch], precision, calls, chunks=chunks)[0]
    for k, a, b in zip(("ux", "sxy", "n1"), got, one):
        assert nerr(a, b) < tol, (k, nerr(a, b))


def test_resume_inside_a_span_is_bitwise(Solver):
    """A state saved inside a block (the span ended with its call) resumes bit
    for bit with the same calls."""
    ch = twod(8, 40, 700)
    print("case far sums, save and load", flush=True)
    with Solver([ch], precision="f32") as s:
        s.set_block(32)
        s.step(150)
        buf = s.save_state()
        s.step(170)
        want = s.fields(0) + s.stress(0)
        s.step(40)
        s.load_state(buf)
        s.step(170)
        got = s.fields(0) + s.stress(0)
    for a, b in zip(want, got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("lx,ly,n_hist", [(1, 40, 127), (1, 64, 128), (5, 13, 300), (3, 43, 700),
                                          (65, 16, 515)])
def test_strain_damping_spans(Solver, lx, ly, n_hist):
    """Accumulated-strain damping: calls of many steps against single steps in
    FP64 (1e-12), and the FP32 forms against the FP64 run (its tolerances)."""
    ch = (twod(lx, ly, n_hist) if lx > 1 else uni(ly, n_hist)).replace(law="strain_damping")
    calls = [200, 150, 8, 7, 31, 32, 33, 64, 100, 129]
    print(f"case strain damping spans {lx}x{ly}, window {n_hist}", flush=True)
    one = advance(Solver, [ch], "f64", [1] * sum(calls))[0]
    for prec, block, fused, bound in (("f64", 1, 1, 1e-12), ("f64", 32, 0, 1e-12),
                                      ("f32", 32, 1, 1e-4), ("f32p64", 8, 0, 1e-4)):
        got = advance(Solver, [ch], prec, calls, block=block, fused=fused)[0]
        for k, a, b in zip(("ux", "sxy", "n1"), got, one):
            assert nerr(a, b) < bound, (prec, block, k, nerr(a, b))


@pytest.mark.parametrize("lx,ly,n_hist,chunks", [
    (5, 13, 127, [1]), (4, 16, 128, [1]), (1, 40, 257, [2]), (8, 32, 300, [2]), (65, 16, 530, [3]),
])
def test_full_tensor_spans(Solver, lx, ly, n_hist, chunks):
    """The full tensor: calls of many steps against single steps in FP64
    (1e-12), the FP32 forms against the FP64 run (the FP32 tolerances), and a
    jet whose rates leave the expansion."""
    ch = twod(lx, ly, n_hist, finger=True) if lx > 1 else uni(ly, n_hist, finger=True)
    calls = [150, 8, 7, 15, 16, 17, 33, 100]
    print(f"case full-tensor spans {lx}x{ly}, window {n_hist}", flush=True)
    one = advance(Solver, [ch], "f64", [1] * sum(calls), chunks=chunks)[0]
    for prec, block, fused, pers, bound in (
            ("f64", 1, 1, False, 1e-12), ("f64", 16, 0, True, 1e-12), ("f64", 4, 0, False, 1e-12),
            ("f32", 16, 1, True, 1e-4), ("f32p64", 8, 0, False, 1e-4)):
        got = advance(Solver, [ch], prec, calls, block=block, chunks=chunks, persistent=pers,
                      fused=fused)[0]
        for k, a, b in zip(("ux", "sxy", "n1"), got, one):
            assert nerr(a, b) < bound, (prec, block, k, nerr(a, b))


@pytest.mark.parametrize("chunks", [[1], [3]])
def test_full_tensor_rates_beyond_the_expansion(Solver, chunks):
    ly, lx = 64, 8
    u0 = np.zeros((2, ly, lx))
    u0[0, 20:24] = 0.08
    ch = twod(lx, ly, 600, u0=u0, gx=0.0, gamma_c=0.1, finger=True)
    calls = [64, 150, 100]
    print(f"case full tensor, rates beyond the expansion, chunks {chunks}", flush=True)
    one = advance(Solver, [ch], "f64", [1] * sum(calls), chunks=chunks)[0]
    got = advance(Solver, [ch], "f64", calls, chunks=chunks)[0]
    for k, a, b in zip(("ux", "sxy", "n1"), got, one):
        assert nerr(a, b) < 1e-12, (k, nerr(a, b))
