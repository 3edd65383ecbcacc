"""GPU parity of the 1D stages that run a whole pass in one launch.

A wave owns 256 cells and writes the inner 256 - 2K (K up to 48 stages), so
the lengths below sit around whole numbers of segments, below one segment,
and at grids shorter than the halo (periodic: several wraps).  Passes of few
stages and of more than one launch's.  Bars as everywhere: FP64 1e-12, FP32
form 1e-5 per field against the FP64 oracle (max-norm, relative).

The second test compares with the one-stage kernels, which a grid of two equal
rows takes: its y-differences are exactly 0 and the operations are the same,
so the fields agree bit for bit."""
import numpy as np
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# The bar below scales with the dt factor, which is too little at 1500: the
# one-stage kernels miss it on the same inputs too (FP64 1.36e-11 against
# 7.5e-12; the FP32 form ends in bad cells).
BEYOND = pytest.mark.xfail(reason="bar not met by the one-stage kernels either: FP64 1.36e-11, FP32 bad cells")


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,wall,face,factor", [(2, 0, 0, 50.0), (3, 1, 0, 200.0), (31, 0, 1, 300.0), (210, 1, 0, 100.0),
                                                (211, 0, 0, 100.0), (255, 1, 1, 20.0), (1024, 1, 0, 100.0),
                                                pytest.param(1900, 0, 0, 1500.0, marks=BEYOND), (5001, 1, 0, 1.5)])
def test_line_stages(n, wall, face, factor, precision):
    from oracle import oracle as orc
    wl = W.heat1d(n)
    rng = np.random.Generator(np.random.PCG64(n))
    wl["fields"]["T1"] = np.ascontiguousarray(wl["fields"]["T1"] * np.exp(0.1 * rng.standard_normal((1, 1, n))))
    wl["fields"]["T2"] = wl["fields"]["T1"].copy()
    wl["bc"] = (W.ADIABATIC if wall else W.PERIODIC,) + (W.PERIODIC,) * 2
    for p in wl["phases"]:
        p["npow"] = 2.0
    wl["dt_factor"] = factor
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=2, face_mean=face)
    print(f"case {n} wall={wall} face={face} {precision} P={[r['P'] for r in ro]}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 2, passes=2, precision=precision, frozen=[r["lambda_G"] for r in ro], face_mean=face)
    assert [r["P"] for r in rg] == [r["P"] for r in ro]
    tol = 1e-12 if precision == "fp64" else 1e-5
    # the final explicit stage amplifies white rounding by tau lambda (400 at a
    # dt factor of 200, where the bars above are stated)
    tol *= max(1.0, factor / 200.0)
    errs = {k: rel_err(fg[k], fo[k]) for k in ("T1", "alpha2")}
    for k, e in errs.items():
        assert e <= tol, (k, e, errs)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,wall,face,factor", [(2, 0, 0, 50.0), (2, 1, 0, 50.0), (3, 0, 1, 200.0), (31, 1, 0, 300.0),
                                                (162, 0, 0, 300.0), (255, 1, 1, 20.0), (1900, 0, 0, 600.0),
                                                (1901, 1, 0, 600.0), (5001, 0, 1, 1.5)])
def test_line_bits(n, wall, face, factor, precision):
    from oracle import oracle as orc
    base = W.heat1d(n)
    rng = np.random.Generator(np.random.PCG64(n))
    T = base["fields"]["T1"] * np.exp(0.1 * rng.standard_normal((1, 1, n)))
    for p in base["phases"]:
        p["npow"] = 2.0
    base["bc"] = (W.ADIABATIC if wall else W.PERIODIC,) + (W.PERIODIC,) * 2
    base["dt_factor"] = factor
    out = []
    for rows in (1, 2):
        wl = dict(base, n=(n, rows, 1), h=(base["h"][0], 1e100, 1.0))
        wl["fields"] = {k: np.ascontiguousarray(np.repeat(v, rows, axis=1)) for k, v in base["fields"].items()}
        wl["fields"]["T1"] = np.ascontiguousarray(np.repeat(T, rows, axis=1))
        wl["fields"]["T2"] = wl["fields"]["T1"].copy()
        if rows == 1:
            tau, lam = oracle_dt(orc, wl)
        fg, rg, s = run_gpu(wl, tau, 2, passes=2, precision=precision, frozen=[[lam, lam]] * 2, face_mean=face)
        print(f"case {n}x{rows} wall={wall} face={face} {precision} P={rg[0]['P']}", flush=True)
        out.append((fg["T1"][:, :1], [r["P"] for r in rg]))
        s.close()
    assert out[0][1] == out[1][1]
    assert np.isfinite(out[0][0]).all() and np.array_equal(out[0][0], out[1][0])
