"""A spectral bound that has no Chebyshev schedule: the call returns a status
(nothing is thrown across the ABI), and the context goes on with the next
state.  At T = 1e200 a power law's conductivity overflows, a cell without mass
has an infinite 1/rho, and a caller's frozen bound can be any number.  Steps after the state is set again: FP64 1e-12, FP32 form 1e-5 of the
oracle's fields."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2106_00282_amd import tlim, workloads as W
from paper_2106_00282_amd.tlim import StepOpts, TlimError
from _cases import make_solver, oracle_dt, rel_err, run_oracle

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32": 1e-5}


def workload(kind):
    if kind == "1d":
        wl = W.heat1d(200)
        for p in wl["phases"]:
            p["npow"] = 2.0
        return wl
    if kind == "2d":
        return W.levelset2d(64)
    wl = W.bubbles3d(24, nbubbles=3, shape=(24, 20, 12))
    wl["viscous"] = False
    return wl


def spoil(s, wl):
    T = wl["fields"]["T1"].copy()
    T.flat[np.abs(wl["fields"]["alpha2"] - 0.5).argmin()] = 1e200
    for k in ("T1", "T2"):
        s.set_field(k, torch.from_numpy(T))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("whole", [0, 1])
@pytest.mark.parametrize("report", [True, False])
@pytest.mark.parametrize("kind", ["1d", "2d", "3d"])
def test_infinite_conductivity(kind, report, whole, precision):
    from oracle import oracle as orc
    wl = workload(kind)
    tau, _ = oracle_dt(orc, wl)
    fo, _ = run_oracle(orc, wl, tau, 2, passes=2)
    o = StepOpts(dt=tau, passes=2, whole_step=whole)
    s = make_solver(wl, precision)
    for first in range(2):  # without a history, then with one
        if first:
            s.set_workload(wl)
            for _ in range(2):
                assert s.advance(o, report=report)[0] == 0
        print(f"case {kind} report={report} whole={whole} {precision} history={first}", flush=True)
        spoil(s, wl)
        st = s.advance(o, report=report)[0] or s.finish()
        assert st == tlim.E_NUMERIC
        # no pass ran: the fields hold the relaxed start
        T = s.get_field("T1").cpu().numpy()
        assert np.isfinite(T).all() and T.max() > 9e199
    s.set_workload(wl)
    for _ in range(2):
        assert s.advance(o, report=report)[0] == 0
    assert s.finish() == 0
    for k in ("T1", "alpha2"):
        assert rel_err(s.get_field(k).cpu().numpy(), fo[k]) <= TOL[precision], k
    s.close()


def test_viscous_bound_without_mass():
    wl = W.bubbles3d(16, nbubbles=2, shape=(16, 12, 8))
    s = make_solver(wl)
    u = s.get_field("u").cpu().numpy()
    for k in ("m1", "m2"):
        m = wl["fields"][k].copy()
        m.flat[7] = 0.0
        s.set_field(k, torch.from_numpy(m))
    st, rep = s.advance(StepOpts(dt=1e-3, passes=1, do_viscous=1))
    assert st == tlim.E_NUMERIC
    assert np.array_equal(s.get_field("u").cpu().numpy(), u)
    s.close()


@pytest.mark.parametrize("lam", [1e300, float("inf"), float("nan")])
def test_given_bounds(lam):
    wl = W.bubbles3d(16, nbubbles=2, shape=(16, 12, 8))
    s = make_solver(wl)
    T = s.get_field("T1")
    with pytest.raises(TlimError) as e:
        s.advance(StepOpts(dt=1.0, passes=1, frozen_lambda=[lam]))
    assert e.value.status == tlim.E_ARG
    with pytest.raises(TlimError) as e:
        s.advance(StepOpts(dt=1.0, passes=1, do_viscous=1, frozen_visc=[1.0, lam, 1.0]))
    assert e.value.status == tlim.E_ARG
    assert torch.equal(s.get_field("T1"), T)
    n = ctypes.c_size_t()
    arr = (ctypes.c_double * 1)(lam)
    oc = StepOpts(dt=1.0, passes=1).c()
    assert tlim.load_library().tlim_adjoint_workspace_bytes(s._ctx, ctypes.byref(oc), 1, arr,
                                                             ctypes.byref(n)) == tlim.E_ARG
    s.close()
