"""The viscous part's strip kernels (62 columns by 4 rows, marching 4 to 16
planes): coefficients, bounds and the FP32 form's source at sizes below, at and
beyond a strip, in 1D to 3D, walls and periodic, both face means, with and
without heating.  Two steps against the oracle (FP64 1e-12, FP32 form 1e-5);
the components' bounds to 1e-13."""
import numpy as np
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,walls,face,heat", [((63, 1, 1), (1, 0, 0), 0, 0), ((40, 3, 1), (0, 1, 0), 1, 1),
                                                   ((62, 4, 5), (0, 0, 1), 0, 1), ((61, 5, 4), (1, 0, 0), 1, 0),
                                                   ((125, 33, 17), (0, 1, 0), 0, 1), ((3, 66, 33), (1, 1, 1), 0, 0),
                                                   ((124, 2, 2), (0, 0, 0), 0, 1)])
def test_visc_strips(shape, walls, face, heat, precision):
    from oracle import oracle as orc
    wl = W.bubbles3d(max(shape), shape=shape)
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    for c in "uvw":  # a flow that the heating can see
        wl["fields"][c] = np.ascontiguousarray(10.0 * wl["fields"][c])
    wl["dt_factor"] = 20.0
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=1, viscous=True, face_mean=face, visc_heating=heat)
    print(f"case {shape} walls={walls} face={face} heat={heat} {precision} {[r['visc_P'] for r in ro]}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 2, passes=1, viscous=True, precision=precision, face_mean=face, visc_heating=heat)
    for a, b in zip(rg, ro):
        assert list(a["visc_P"]) == list(b["visc_P"]) and a["P"] == b["P"]
        for x, y in zip(a["visc_lambda_G"], b["visc_lambda_G"]):
            assert abs(x - y) <= 1e-13 * abs(y)
    tol = 1e-12 if precision == "fp64" else 1e-5
    errs = {k: rel_err(fg[k], fo[k]) for k in ("T1", "alpha2", "u", "v", "w") if np.abs(fo[k]).max() > 0}
    assert max(errs.values()) <= tol, errs
    s.close()
