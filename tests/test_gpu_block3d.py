"""GPU parity of the 3D kernels that advance several LIM stages per launch.

A workgroup writes the inner 64 - 2K by rows - 2K cells of its column (K = 2 or
3 stages in double, up to 4 in float; 10 to 56 rows) and walks a chunk of planes
with K planes more on either side; the shapes below have sides near such tiles
(58 and 60 x cells, 18 and 28 rows), leave small remainders, are thinner than
the halo, or are a single plane chunk (every kernel's own tile edges are in
test_gpu_block3d_edges.py).  dt factors give passes whose stage counts leave every
remainder.  Bars as everywhere: FP64 1e-12, FP32 form 1e-5 per field against the
FP64 oracle (max-norm, relative)."""
import numpy as np
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

CASES = [  # shape, walls (x, y, z), face mean, dt factor
    ((58, 18, 5), (0, 0, 0), 0, 200.0),
    ((59, 19, 2), (1, 0, 1), 0, 40.0),
    ((60, 28, 7), (0, 1, 0), 1, 90.0),
    ((61, 58, 3), (1, 1, 1), 0, 15.0),
    ((117, 37, 13), (0, 0, 1), 1, 5.0),
    ((2, 3, 4), (0, 0, 0), 0, 60.0),
    ((5, 2, 2), (1, 0, 0), 0, 120.0),
    ((7, 61, 29), (0, 1, 1), 0, 2.0),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,walls,face,factor", CASES)
def test_blocked_stages_3d(shape, walls, face, factor, precision):
    from oracle import oracle as orc
    wl = W.bubbles3d(max(shape), nbubbles=6, shape=shape)
    wl["h"] = (1.0 / shape[0], 1.0 / shape[0], 1.0 / shape[0])
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    wl["dt_factor"] = factor
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=2, face_mean=face)
    print(f"case {shape} walls={walls} face={face} {precision} P={[r['P'] for r in ro]}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 2, passes=2, precision=precision, frozen=[r["lambda_G"] for r in ro], face_mean=face)
    assert [r["P"] for r in rg] == [r["P"] for r in ro]
    tol = 1e-12 if precision == "fp64" else 1e-5
    errs = {k: rel_err(fg[k], fo[k]) for k in ("T1", "alpha2", "u", "v", "w")}
    for k, e in errs.items():
        assert e <= tol, (k, e, errs)
    s.close()


@pytest.mark.parametrize("shape,walls", [((59, 29, 6), (1, 0, 0)), ((6, 19, 61), (0, 1, 1))])
def test_blocked_recompute_keeps_every_stage(shape, walls):
    """The adjoint's recomputation through the blocked kernel (every stage
    kept) against the oracle's adjoint."""
    from oracle import oracle as orc
    from paper_2106_00282_amd.tlim import StepOpts
    from _cases import make_solver
    import torch
    wl = W.interface3d(max(shape), shape=shape)
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    tau, _ = oracle_dt(orc, wl)
    s = make_solver(wl)
    opts = StepOpts(dt=tau, passes=2)
    ckpt, lam = s.forward_checkpointed(opts, 2, 2)
    seed = np.random.default_rng(3).standard_normal(ckpt.shape[1:])
    dT0, dk0 = s.adjoint(opts, 2, 2, ckpt, lam, torch.from_numpy(seed))
    g = orc.make_grid(wl["n"], wl["h"], wl["bc"])
    f = wl["fields"]
    oT, ok = orc.heat_adjoint(g, wl["phases"], orc.StepOpts(tau=tau, passes=2), 2, np.array(lam), f["alpha2"], f["m1"], f["m2"],
                              f["T1"], seed)[:2]
    assert rel_err(dT0.cpu().numpy(), oT) <= 1e-12
    assert max(abs(dk0[k] - ok[k]) for k in range(2)) <= 1e-10 * max(abs(x) for x in ok)
    s.close()
