"""Unequal p_inf on 1D and 2D grids without sources: the alpha2 update that
ends a pass rides with the next pass's coefficients, the last pass's has a
launch of its own, and the reductions come from the stages.  Passes 1 to 4,
grids around a strip of 62 x 4 cells, walls, both face means and laws, a
tolerance that stops the passes early, and steps whose prediction misses.
Two or three steps against the oracle at the usual bars (FP64 1e-12, FP32 form
1e-5); lambda_G of every pass to 1e-12 (FP64)."""
import numpy as np
import pytest

from paper_2106_00282_amd import workloads as W
from paper_2106_00282_amd.tlim import StepOpts
from _cases import make_solver, oracle_dt, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _workload(nx, ny, walls, spitzer, factor):
    wl = W.levelset2d(max(nx, ny))
    ph = [dict(gamma=4.4, pinf=1.0, cv=0.5, q=0.0, k0=1.0, T0=1.0, npow=1.0, mu=0.0),
          dict(gamma=1.4, pinf=0.0, cv=1.0, q=0.0, k0=0.05, T0=1.0, npow=1.0, mu=0.0)]
    wl["phases"] = W.spitzer_phases(ph) if spitzer else ph
    wl["n"] = (nx, ny, 1)
    wl["h"] = (1.0 / max(nx, ny),) * 2 + (1.0,)
    wl["fields"] = {k: np.ascontiguousarray(v[:, :ny, :nx]) for k, v in wl["fields"].items()}
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls) + (W.PERIODIC,)
    wl["dt_factor"] = factor
    return wl


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,walls,face,spitzer,passes", [(200, 1, (1, 0), 0, False, 3), (62, 4, (0, 0), 0, False, 2),
                                                             (63, 33, (1, 1), 1, False, 4), (61, 37, (0, 1), 0, True, 3),
                                                             (124, 101, (1, 0), 0, False, 1), (250, 130, (0, 0), 1, True, 2)])
def test_update_with_coefficients(nx, ny, walls, face, spitzer, passes, precision):
    from oracle import oracle as orc
    wl = _workload(nx, ny, walls, spitzer, 20.0)
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 3, passes=passes, face_mean=face)
    print(f"case {nx}x{ny} {walls} face={face} {precision} P={[r['P'] for r in ro]}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 3, passes=passes, precision=precision, face_mean=face)
    for a, b in zip(rg, ro):
        assert a["P"] == b["P"]
        if precision == "fp64":
            assert np.allclose(a["lambda_G"], b["lambda_G"], rtol=1e-12, atol=0.0)
            assert np.allclose(a["err"], b["err"], rtol=1e-9, atol=1e-12)
    tol = 1e-12 if precision == "fp64" else 1e-5
    errs = {k: rel_err(fg[k], fo[k]) for k in ("T1", "alpha2")}
    assert max(errs.values()) <= tol, errs
    s.close()


def test_update_stops_at_tolerance():
    from oracle import oracle as orc
    wl = _workload(70, 45, (0, 1), False, 5.0)
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=8, picard_tol=1e-3)
    fg, rg, s = run_gpu(wl, tau, 2, passes=8, picard_tol=1e-3)
    assert [r["passes_run"] for r in rg] == [r["passes_run"] for r in ro]
    assert all(1 < r["passes_run"] < 8 for r in rg)
    for k in ("T1", "alpha2"):
        assert rel_err(fg[k], fo[k]) <= 1e-12, k
    s.close()


def test_update_rolls_back():
    from oracle import oracle as orc
    wl = _workload(96, 80, (0, 0), False, 20.0)
    tau, _ = oracle_dt(orc, wl)
    g = orc.make_grid(wl["n"], wl["h"], wl["bc"])
    fo = {k: v.copy() for k, v in wl["fields"].items()}
    s = make_solver(wl)
    ph = [dict(p) for p in wl["phases"]]
    missed = []
    for scale in (1.0, 1.0, 1.0, 4.0, 4.0):
        for k in range(2):
            ph[k]["k0"] = wl["phases"][k]["k0"] * scale
            s.set_phase(k, ph[k])
        orc.step(g, ph, orc.StepOpts(tau=tau, passes=3), fo)
        st, rep = s.advance(StepOpts(dt=tau, passes=3))
        assert st == 0
        missed.append(bool(rep["mispredicted"]))
    assert any(missed)
    for k in ("T1", "alpha2"):
        assert rel_err(s.get_field(k).cpu().numpy(), fo[k]) <= 1e-12, k
    s.close()
