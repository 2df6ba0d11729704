"""Far sums where entries decay within a few steps: short relaxation times and
shear rates of the order of gamma_c and above.

A state with a written history (every entry of the window given) is advanced
in a call of many steps, whose sums come from a span's moments, and step by
step with a fresh pass each (lb_set_block starts a new block), the general
path; the run of the FP64 handle is the reference.  FP64: 1e-12, the bound of the
other launch-shape comparisons.  FP32 histories: an entry's power, its product
and its terms are each rounded to 2^-24 of the entry's term, a few of them per
sum where a few entries carry it, and its exponent k rate to k rate 2^-24, so
the error's root mean square stays below max(4, rate) x 2^-24.  Split storage
adds the rounding of its FP32 remainders: the FP32 velocity tolerance.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

HALF_ULP = 2.0 ** -24


@pytest.fixture(scope="module")
def Solver():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_06123_amd import Solver as S
    return S


def channel(kind, ly, n_hist, **kw):
    """From rest without a body force: what moves is the history's stress."""
    law = dict(finger=dict(finger=True), strain=dict(law="strain_damping")).get(kind, {})
    return workloads.plain_f64().channels[0].replace(
        lx=1 if kind == "uni" else 3, ly=ly, n_hist=n_hist, gx=0.0, **law, **kw)


def history(ch, s0, seed=3):
    """Shear rates [age - 1][node]: sign and size by node, a slow swing."""
    rng = np.random.default_rng(seed)
    s = s0 * (1.0 + 0.002 * rng.uniform(-1.0, 1.0, ch.nodes)) * rng.choice((-1.0, 1.0), ch.nodes)
    age = np.arange(1, ch.n_hist)[:, None]
    return (s * (1.0 + 0.002 * np.cos(age / 40.0))).astype(np.float32)


def written_state(ch, precision, s, t=5000):
    """State after t steps: fluid at rest, entries s[age - 1][node] of pure
    shear."""
    import torch
    from paper_1504_06123_amd.solver import pack_state_header, state_layout
    layout, total = state_layout([ch], precision)
    buf = np.zeros(total, dtype=np.uint8)
    buf[:256] = np.frombuffer(pack_state_header(t, 1, precision, total), dtype=np.uint8)
    dt = np.float64 if precision == "f64" else np.float32
    slots = (t - np.arange(1, ch.n_hist)) % ch.n_hist

    def put(name, plane, v):
        off, rows, n = layout[0][name]
        a = buf[off:off + rows * n * dt().itemsize].view(dt).reshape(-1, ch.n_hist, n)
        a[plane][slots] = v

    if ch.finger:  # kappa (xx, xy, yx, yy), then exp(kappa) - I: kappa itself
        put("ring", 1, s)
        put("ring", 5, s)
    else:
        put("ring_s", 0, s)
        if ch.lx > 1:
            put("ring_r", 0, np.abs(s))
    return torch.from_numpy(buf).cuda()


def outputs(s):
    _, ux, uy = s.fields(0)
    return dict(zip(("ux", "uy", "sxy", "n1"), (ux, uy) + s.stress(0)))


def run(Solver, ch, precision, s, calls, block):
    with Solver([ch], precision=precision) as sol:
        sol.set_block(block)
        sol.load_state(written_state(ch, precision, s))
        for n in calls:
            sol.step(n)
        return outputs(sol)


def run_general(Solver, ch, precision, s, steps):
    """A fresh one-step pass for every step."""
    with Solver([ch], precision=precision) as sol:
        sol.load_state(written_state(ch, precision, s))
        for _ in range(steps):
            sol.set_block(1)
            sol.step(1)
        return outputs(sol)


def error(got, want, key):
    """Largest error over the largest speed or stress component."""
    of = ("ux", "uy") if key in ("ux", "uy") else ("sxy", "n1")
    scale = max(np.abs(want[k]).max() for k in of if k in want)
    return float(np.abs(got[key] - want[key]).max() / scale) if scale > 0 else 0.0


def rms(a, b):
    return float(np.sqrt(np.mean((a - b) ** 2)) / np.sqrt(np.mean(b ** 2)))


# (tau, gamma_c, shear rate, width): by the relaxation time alone, and steady
# rates of 1.5 and 4 gamma_c
FAST = [(0.05, 0.1, 1e-3, 64), (0.5, 0.1, 1e-3, 64), (0.7, 0.1, 1e-3, 64), (2.0, 0.1, 1e-3, 64),
        (10.0, 0.1, 1e-3, 64), (1000.0, 0.02, 0.03, 288), (1000.0, 0.02, 0.08, 288)]


@pytest.mark.parametrize("tau,gamma_c,s0,ly", FAST)
@pytest.mark.parametrize("kind", ["2d", "uni", "finger", "strain"])
def test_fast_decays_equal_the_general_pass(Solver, kind, tau, gamma_c, s0, ly):
    ch = channel(kind, ly, 600, tau_m=tau, gamma_c=gamma_c)
    print(f"case fast decays {kind} tau {tau} rate {s0 / gamma_c:g}", flush=True)
    s = history(ch, s0)
    block = 16 if kind == "finger" else 32
    # the velocity of a call that ends inside a span of 128 steps, and the
    # stress of a span's first step (which the fluid feels a step later)
    for calls, key in (((65,), "ux"), ((1,), "sxy")):
        want = run_general(Solver, ch, "f64", s, sum(calls))
        got = run(Solver, ch, "f64", s, calls, block)
        for k in want:
            assert error(got, want, k) < 1e-12, (calls, k, error(got, want, k))
        got = run(Solver, ch, "f32p64", s, calls, block)
        bound = max(4.0, 1.0 / tau + s0 / gamma_c) * HALF_ULP
        assert rms(got[key], want[key]) < bound, (calls, rms(got[key], want[key]))
        got = run(Solver, ch, "f32", s, calls, block)
        assert rms(got[key], want[key]) < 1e-5, (calls, rms(got[key], want[key]))


@pytest.mark.parametrize("rate", [0.6, 1.42, 1.5, 4.0])
@pytest.mark.parametrize("kind", ["2d", "uni", "finger"])
def test_a_fast_young_entry_is_not_taken_as_damped(Solver, kind, rate):
    """One entry far above the others' rate, two steps old: its term is a
    good part of the sum, though it has decayed by the middle of the span."""
    ch = channel(kind, 288, 600, tau_m=1000.0, gamma_c=0.02)
    print(f"case fast young entry {kind} rate {rate}", flush=True)
    s = history(ch, 0.002)
    s[1] = np.sign(s[1]) * rate * ch.gamma_c
    want = run_general(Solver, ch, "f64", s, 65)["ux"]
    got = run(Solver, ch, "f64", s, (65,), 16 if kind == "finger" else 32)["ux"]
    assert np.abs(got - want).max() < 1e-12 * np.abs(want).max()
    got = run(Solver, ch, "f32p64", s, (65,), 16 if kind == "finger" else 32)["ux"]
    assert rms(got, want) < 4 * HALF_ULP, rms(got, want)


@pytest.mark.parametrize("tau", [0.05, 0.5, 0.7, 2.0, 10.0])
@pytest.mark.parametrize("kind", ["2d", "uni", "finger"])
def test_short_relaxation_times_match_the_oracle(Solver, kind, tau):
    """Startup runs past the window's first fill, at the tolerances of the
    other oracle comparisons."""
    ch = channel(kind, 24, 520, tau_m=tau).replace(gx=2e-5)
    print(f"case short relaxation times {kind} tau {tau}", flush=True)
    calls = [300, 130, 200, 1]
    oc = oracle.OracleChannel(ch)
    oc.step(sum(calls))
    want = dict(zip(("ux", "sxy", "n1"), (oc.fields()[1],) + oc.stress()))
    for precision, block, tol in (("f64", 1, (1e-11,) * 3), ("f64", 16, (1e-11,) * 3),
                                  ("f32", 16, (1e-5, 1e-4, 1e-4)),
                                  ("f32p64", 16, (1e-5, 1e-4, 1e-4))):
        with Solver([ch], precision=precision) as s:
            s.set_block(block if kind == "finger" or block == 1 else 32)
            for n in calls:
                s.step(n)
            got = outputs(s)
        for k, bound in zip(want, tol):
            assert error(got, want, k) < bound, (precision, block, k, error(got, want, k))
