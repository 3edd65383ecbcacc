"""1D passes of more stages than one launch takes, against the oracle.

Bars, from the arithmetic: every stage rounds its result by half an ulp of the
largest T, and the final explicit stage passes such a rounding on with at most
tau lambda_G, so FP64 differs by at most (2P - 1) tau lambda_G 2^-53 on either
side.  The FP32 form runs a smooth state under the bar of the shorter passes,
1e-5 at tau lambda_G = 400, in proportion to tau lambda_G."""
import numpy as np
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle
from test_stage_plan import LINE, stage_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,wall,face", [(1900, 0, 0), (1024, 1, 0), (301, 0, 1), (40, 1, 1)])
def test_passes_of_two_launches(n, wall, face, precision):
    from oracle import oracle as orc
    wl = W.heat1d(n)
    if precision == "fp64":
        rng = np.random.Generator(np.random.PCG64(n))
        wl["fields"]["T1"] = np.ascontiguousarray(wl["fields"]["T1"] * np.exp(0.1 * rng.standard_normal((1, 1, n))))
        wl["fields"]["T2"] = wl["fields"]["T1"].copy()
    wl["bc"] = (W.ADIABATIC if wall else W.PERIODIC,) + (W.PERIODIC,) * 2
    for p in wl["phases"]:
        p["npow"] = 2.0
    wl["dt_factor"] = 650.0
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=2, face_mean=face)
    print(f"case {n} wall={wall} face={face} {precision} P={[r['P'] for r in ro]}", flush=True)
    stages = max(2 * P - 1 for r in ro for P in r["P"])
    tl = max(tau * x for r in ro for x in r["lambda_G"])
    plan = stage_plan((n,), precision, face, count=stages, bc=wl["bc"])
    assert plan.kernel == LINE and plan.stages < stages
    fg, rg, s = run_gpu(wl, tau, 2, passes=2, precision=precision, frozen=[r["lambda_G"] for r in ro], face_mean=face)
    assert [r["P"] for r in rg] == [r["P"] for r in ro]
    tol = 2 * stages * tl * 2.0 ** -53 if precision == "fp64" else 1e-5 * tl / 400
    for k in ("T1", "alpha2"):
        assert rel_err(fg[k], fo[k]) <= tol, k
    s.close()
