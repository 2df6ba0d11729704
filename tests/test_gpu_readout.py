"""Readouts of written states: the values, the count of non-finite ones and the
Mach guard, through the pinned buffer (one part and two) and through the
workspace, against the host scans of lbmax_checks.h."""
import ctypes
import os
import re
import shutil
import subprocess
import warnings

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1504_06123_amd", "csrc")
SHIM = """
#include "lbmax_checks.h"
extern "C" long nonfinite(const double *a, size_t n) {
    return (long)lbmax::scan_values(a, n).nonfinite;
}
extern "C" int trips(const double *ux, const double *uy, size_t n) {
    return lbmax::mach_guard_trips(lbmax::max_speed(ux, uy, n)) ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1504_06123_amd as lb
    return lb


@pytest.fixture(scope="module")
def scans(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("scans")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o",
                    str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    P = ctypes.POINTER(ctypes.c_double)
    lib.nonfinite.argtypes = [P, ctypes.c_size_t]
    lib.nonfinite.restype = ctypes.c_long
    lib.trips.argtypes = [P, P, ctypes.c_size_t]
    return lib


def state(lb, ch, precision, planes):
    import torch
    layout, total = lb.state_layout([ch], precision)
    buf = np.zeros(total, dtype=np.uint8)
    buf[:256] = np.frombuffer(lb.pack_state_header(7, 1, precision, total), dtype=np.uint8)
    for name, v in planes.items():
        off, rows, n = layout[0][name]
        buf[off:off + rows * n * 8].view(np.float64).reshape(rows, n)[:len(v)] = v
    return torch.from_numpy(buf).cuda()


# nodes: a part of a workgroup, one and a bit, many, and two parts of the pinned
# buffer (8 MiB of four planes each: 254208 nodes) and a rest
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("lx,ly", [(2, 3), (1, 257), (40, 100), (513, 1000)])
def test_planted_values(lb, scans, lx, ly, precision):
    ch = workloads.plain_f64().channels[0].replace(lx=lx, ly=ly, n_hist=2, u0=None)
    n = lx * ly
    print(f"case readout {lx}x{ly} {precision}", flush=True)
    rng = np.random.default_rng(11)
    clean = {"drho": rng.uniform(-1e-3, 1e-3, (1, n)), "vel": rng.uniform(-0.05, 0.05, (2, n)),
             "sig": rng.uniform(-1e-3, 1e-3, (2, n))}
    if lx == 1:
        clean["vel"][1] = 0.0
    part = 254208 if n > 254208 else n // 2
    plants = [[], [("vel", 0, 0, 0.11)], [("vel", 0, n - 1, np.nan)],
              [("drho", 0, part, np.inf), ("vel", 0, part - 1, -np.inf), ("vel", 0, n - 1, 0.2),
               ("sig", 0, 0, np.nan), ("sig", 1, n - 1, np.inf), ("sig", 0, part, -np.inf)]]
    with lb.Solver([ch], precision=precision) as s:
        for plant in plants:
            planes = {k: v.copy() for k, v in clean.items()}
            for name, row, node, value in plant:
                planes[name][row, node] = value
            want_f = np.concatenate((1.0 + planes["drho"], planes["vel"]))
            s.load_state(state(lb, ch, precision, planes))
            for pinned in (True, False):
                s.set_pinned(pinned)
                s.set_checks(finite=False, mach=False)
                got_f = np.array(s.fields(0)).reshape(3, n)
                got_s = np.array(s.stress(0)).reshape(2, n)
                assert np.array_equal(got_f, want_f, equal_nan=True), (plant, pinned)
                assert np.array_equal(got_s, planes["sig"], equal_nan=True), (plant, pinned)
                s.set_checks()
                for read, values in ((s.fields, want_f), (s.stress, planes["sig"])):
                    values = np.ascontiguousarray(values)
                    P = ctypes.POINTER(ctypes.c_double)
                    bad = scans.nonfinite(values.ctypes.data_as(P), values.size)
                    with warnings.catch_warnings(record=True) as w:
                        warnings.simplefilter("always")
                        if bad:
                            with pytest.raises(lb.LBError) as e:
                                read(0)
                            assert int(re.search(r": (\d+) non-finite", str(e.value)).group(1)) \
                                == bad, (plant, pinned)
                        else:
                            read(0)
                    if read == s.fields:
                        ux, uy = np.ascontiguousarray(want_f[1]), np.ascontiguousarray(want_f[2])
                        trips = scans.trips(ux.ctypes.data_as(P), uy.ctypes.data_as(P), n)
                        raised = len(w) == 1 or bool(s.lib.lb_warnings(s.h))
                        assert raised == bool(trips), (plant, pinned)


def test_readouts_through_the_workspace(lb):
    """A run's readouts are the same either way, switched between reads."""
    chans = [workloads.plain_f64().channels[0].replace(lx=lx, ly=ly, n_hist=50)
             for lx, ly in ((4, 16), (1, 300), (31, 77))]
    print("case readout through the workspace", flush=True)
    with lb.Solver(chans, precision="f32") as s:
        s.step(40)
        for i in range(len(chans)):
            s.set_pinned(True)
            a = s.fields(i) + s.stress(i) + (s.grad(i),)
            s.set_pinned(False)
            b = s.fields(i) + s.stress(i) + (s.grad(i),)
            assert all(np.array_equal(x, y) for x, y in zip(a, b))
