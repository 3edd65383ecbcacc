"""3D grids of few y rows, whose stages run one per launch: parity with the
oracle over walls and periodic axes, both face means, with the viscous part
(FP64 1e-12, FP32 form 1e-5 per field, max-norm, relative)."""
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle
from test_stage_plan import MARCH, reverse_plan, stage_plan

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


@pytest.mark.parametrize("shape,walls", [((700, 1, 700), (1, 0, 0)), ((65, 2, 4099), (0, 1, 1)), ((5, 1, 20000), (0, 0, 0))])
def test_thin_grids_adjoint(shape, walls):
    """The gradient of two steps against the oracle's adjoint, with the steps of
    the interval recomputed each or kept (the same bits)."""
    import numpy as np
    import torch
    from oracle import oracle as orc
    from paper_2106_00282_amd.tlim import StepOpts
    from _cases import make_solver
    wl = W.interface3d(max(shape[0], shape[2]) // 8, shape=shape)
    wl["h"] = (1.0 / shape[0],) * 3
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    assert reverse_plan(shape) == MARCH
    tau, _ = oracle_dt(orc, wl)
    s = make_solver(wl)
    opts = StepOpts(dt=tau, passes=2)
    ckpt, lam = s.forward_checkpointed(opts, 2, 2)
    seed = np.random.default_rng(3).standard_normal(ckpt.shape[1:])
    dT0, dk0 = s.adjoint(opts, 2, 2, ckpt, lam, torch.from_numpy(seed), keep_interval=False)
    s._adj_ws = None
    kept, dk1 = s.adjoint(opts, 2, 2, ckpt, lam, torch.from_numpy(seed), keep_interval=True)
    assert torch.equal(kept, dT0)
    g = orc.make_grid(wl["n"], wl["h"], wl["bc"])
    f = wl["fields"]
    oT, ok = orc.heat_adjoint(g, wl["phases"], orc.StepOpts(tau=tau, passes=2), 2, np.array(lam), f["alpha2"], f["m1"],
                              f["m2"], f["T1"], seed)[:2]
    assert rel_err(dT0.cpu().numpy(), oT) <= 1e-12
    for dk in (dk0, dk1):  # (sums by atomics: not bit for bit)
        assert max(abs(dk[k] - ok[k]) for k in range(2)) <= 1e-10 * max(abs(x) for x in ok)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("ny,wall,face,spitzer", [(1, 0, 0, False), (1, 1, 1, True), (2, 0, 1, False), (2, 1, 0, False),
                                                  (3, 0, 0, True), (4, 0, 0, False), (4, 1, 1, False), (5, 0, 1, False),
                                                  (6, 0, 0, False), (7, 1, 0, False)])
def test_coefficients_of_few_rows(ny, wall, face, spitzer, precision):
    """Workgroups of one to three waves build the coefficients (lambda_G of the
    first pass to 1e-13)."""
    import numpy as np
    from oracle import oracle as orc
    shape = (63, ny, 19)
    wl = W.bubbles3d(63, shape=shape)
    if spitzer:
        wl["phases"] = W.spitzer_phases(wl["phases"])
    for c in "uvw":
        wl["fields"].pop(c, None)
    wl["bc"] = (W.PERIODIC, W.ADIABATIC if wall else W.PERIODIC, W.PERIODIC)
    wl["fields"]["T2"] = np.ascontiguousarray(1.2 * wl["fields"]["T1"])
    wl["dt_factor"] = 20.0
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=2, viscous=False, face_mean=face)
    print(f"case {shape} wall={wall} face={face} spitzer={spitzer} {precision}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 2, passes=2, viscous=False, precision=precision, face_mean=face)
    assert abs(rg[0]["lambda_G"][0] - ro[0]["lambda_G"][0]) <= 1e-13 * ro[0]["lambda_G"][0]
    assert [r["P"] for r in rg] == [r["P"] for r in ro]
    tol = 1e-12 if precision == "fp64" else 1e-5
    for k in ("T1", "alpha2"):
        assert rel_err(fg[k], fo[k]) <= tol, k
    s.close()
