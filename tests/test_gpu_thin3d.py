"""3D grids of few y rows, whose stages run one per launch: parity with the
oracle over walls and periodic axes, both face means, with the viscous part
(FP64 1e-12, FP32 form 1e-5 per field, max-norm, relative)."""
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle
from test_stage_plan import MARCH, stage_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,walls,face", [((700, 1, 700), (0, 0, 1), 0), ((701, 2, 699), (1, 1, 0), 1),
                                              ((64, 1, 4097), (1, 0, 0), 0), ((5, 1, 20000), (0, 1, 1), 1)])
def test_thin_grids(shape, walls, face, precision):
    from oracle import oracle as orc
    wl = W.bubbles3d(max(shape[0], shape[2]) // 8, nbubbles=6, shape=shape)
    wl["h"] = (1.0 / shape[0],) * 3
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    assert stage_plan(shape, precision, face, bc=wl["bc"]).kernel == MARCH
    wl["dt_factor"] = 90.0
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 1, passes=2, face_mean=face)
    print(f"case {shape} walls={walls} face={face} {precision} P={[r['P'] for r in ro]}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 1, passes=2, precision=precision, frozen=[r["lambda_G"] for r in ro], face_mean=face)
    assert [r["P"] for r in rg] == [r["P"] for r in ro]
    tol = 1e-12 if precision == "fp64" else 1e-5
    for k in ("T1", "alpha2", "u", "v", "w"):
        assert rel_err(fg[k], fo[k]) <= tol, k
    s.close()
