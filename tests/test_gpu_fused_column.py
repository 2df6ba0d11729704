"""The column form of the fused in-block steps at the edges of its workgroup
sizes (64, 256, 512, 1024 threads): bit for bit the separate launches."""
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


@pytest.mark.parametrize("precision", ["f64", "f32p64", "f32"])
@pytest.mark.parametrize("ly", [3, 63, 64, 65, 256, 257, 512, 513, 1024])
def test_column_form_equals_separate_launches(Solver, precision, ly):
    """Windows shorter than, at and beyond the block; calls that end inside a
    block, so that spans start at every kind of position."""
    base = workloads.plain_f64().channels[0].replace(lx=1, gx=2e-5, tau_m=30.0)
    chans = [base.replace(ly=ly, n_hist=400)] + [
        base.replace(ly=min(ly, 40), n_hist=h) for h in (2, 31, 32, 33)]
    from paper_1504_06123_amd import state_layout
    print(f"case column form, {ly} nodes, {precision}", flush=True)
    out = []
    for mode in (1, 0):
        with Solver(chans, precision=precision) as s:
            s.set_block(32)
            s.set_fused(mode)
            got = []
            for n in (37, 1, 30, 64, 90):
                s.step(n)
                for ci in range(len(chans)):
                    got += s.fields(ci) + s.stress(ci)
            state = s.save_state().cpu().numpy()
            for sec, ch in zip(state_layout(chans, precision)[0], chans):
                for name, (off, rows, n) in sec.items():
                    size = 4 if precision == "f32" and name == "pop" or (
                        precision != "f64" and name == "ring_s") else 8
                    got.append(state[off:off + rows * n * size])
            out.append(got)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
