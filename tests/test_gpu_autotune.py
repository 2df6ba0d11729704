"""What the autotuner times: launch shapes that differ, and whole spans."""
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


def channel(**kw):
    return workloads.plain_f64().channels[0].replace(
        **{**dict(lx=4, ly=64, n_hist=600, tau_m=60.0, gx=2e-5), **kw})


# (channel, blocks, those left): in spans the longest block alone, the
# unblocked steps of the adjoint's kind beside it, without spans all
@pytest.mark.parametrize("kw,blocks,left", [
    ({}, (1, 8, 16, 32), {32: {1}}), ({}, (1, 8), {8: {1}}),
    (dict(lx=1), (1, 8, 32), {1: {1, 2, 4}, 32: {1}}),
    (dict(finger=True), (1, 4, 16), {16: {1}}),
    (dict(n_hist=100), (1, 2, 8, 32), {1: {1, 2, 4}, 2: {1, 2}, 8: {1}, 32: {1}}),
])
def test_trials_differ_and_take_whole_spans(Solver, kw, blocks, left):
    from paper_1504_06123_amd import autotune
    print(f"case autotune {kw} {blocks}", flush=True)
    with Solver([channel(**kw)], precision="f32") as s:
        s.step(40)
        cands = autotune.candidates(s, blocks=blocks, chunk_lens=(300, 1 << 30), graphs=(0, 96))
        kept = autotune._distinct(s, cands)
        assert {b: {c["vec"] for c in kept if c["block"] == b}
                for b in {c["block"] for c in kept}} == left
        assert all(c in cands for c in kept)
        assert len({tuple(sorted(c.items())) for c in kept}) == len(kept)
        # every split and both graph lengths are still there
        assert {(c["chunk_len"], c["graph"], c["persistent"]) for c in kept} == \
            {(c["chunk_len"], c["graph"], c["persistent"]) for c in cands}
        for c in kept:
            assert autotune.time_config(s, c, 32) > 0
            info = s.run_info()
            if info["span"]:
                assert info["span_pos"] == info["span"], c
        best = autotune.tune(s, cands, min_steps=16)
        assert len(best["table"]) == len(kept) and s.t >= 40


def test_tuned_state_is_restored(Solver):
    import numpy as np
    from paper_1504_06123_amd import autotune
    print("case autotune restores", flush=True)
    with Solver([channel()], precision="f32") as s:
        s.set_block(32)
        s.step(75)
        before = s.fields(0) + s.stress(0)
        autotune.tune(s, autotune.candidates(s, blocks=(1, 32), chunk_lens=(1 << 30,)))
        assert s.t == 75
        assert all(np.array_equal(a, b) for a, b in zip(before, s.fields(0) + s.stress(0)))
