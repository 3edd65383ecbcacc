"""The blocked 3D launches at the edges of their own tiles: a launch of K stages
writes the inner 64 - 2K x cells and rows - 2K of the rows that the library
names for it (float K = 4: 56 x 32, harmonic 56 x 16; float K = 3: 58 x 42;
double K = 3: 58 x 18, harmonic 58 x 10; the adjoint's reverse pairs 60 x 12).
Exactly one tile, one cell more, and one cell less in each direction, over
periodic axes and walls.  FP64 1e-12, FP32 form 1e-5 (max-norm, relative)."""
import numpy as np
import pytest
import torch

from paper_2106_00282_amd import workloads as W
from paper_2106_00282_amd.tlim import StepOpts
from _cases import make_solver, oracle_dt, rel_err, run_gpu, run_oracle
from test_stage_plan import BLOCKED_MARCH, reverse_plan, stage_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 1), (0, 1, 0)])
@pytest.mark.parametrize("dx,dy", [(0, 0), (1, 1), (-1, 0), (0, -1)])
@pytest.mark.parametrize("precision,face,K,tile", [("fp32", 0, 4, (56, 32)), ("fp32", 1, 4, (56, 16)), ("fp32", 0, 3, (58, 42)),
                                                   ("fp64", 0, 3, (58, 18)), ("fp64", 1, 3, (58, 10)),
                                                   ("fp64", 0, 2, (60, 28)), ("fp64", 1, 2, (60, 20))])
def test_stages_at_tile_edges(precision, face, K, tile, dx, dy, walls):
    from oracle import oracle as orc
    shape = (tile[0] + dx, tile[1] + dy, 9)
    p = stage_plan(shape, precision, face, count=K)
    assert (p.kernel, p.stages) == (BLOCKED_MARCH, K)
    assert (p.tile_x - 2 * K, p.tile_y - 2 * K) == tile
    wl = W.bubbles3d(max(shape), nbubbles=4, shape=shape)
    for c in "uvw":
        wl["fields"].pop(c, None)
    wl["h"] = (1.0 / shape[0],) * 3
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    lam = oracle_dt(orc, dict(wl, dt_factor=1.0))[1]
    # double: 3 stages (one launch) or 5 (3 + 2); float, after the first stage
    # and before the final one: 7 (4 + 3) or 5 (3 + 2)
    P = {("fp64", 3): 2, ("fp64", 2): 3, ("fp32", 4): 5, ("fp32", 3): 4}[precision, K]
    tau = ((4.0 / np.pi * (P - 0.5)) ** 2 - 1.0) / lam
    frozen = [[lam]]
    fo, ro = run_oracle(orc, wl, tau, 1, passes=1, viscous=False, face_mean=face, frozen=frozen)
    assert ro[0]["P"] == [P]
    print(f"case {shape} walls={walls} face={face} {precision} K={K} P={P}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 1, passes=1, viscous=False, precision=precision, frozen=frozen, face_mean=face)
    assert rg[0]["P"] == [P]
    tol = 1e-12 if precision == "fp64" else 1e-5
    for k in ("T1", "alpha2"):
        assert rel_err(fg[k], fo[k]) <= tol, k
    s.close()


@pytest.mark.parametrize("shape,walls", [((60, 12, 7), (0, 0, 0)), ((61, 13, 5), (1, 1, 0)), ((60, 12, 9), (1, 1, 1)),
                                         ((59, 25, 6), (0, 1, 0)), ((62, 30, 4), (0, 0, 1))])
def test_reverse_stages_at_tile_edges(shape, walls):
    from oracle import oracle as orc
    assert reverse_plan(shape) == BLOCKED_MARCH
    wl = W.interface3d(max(shape), shape=shape)
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls)
    tau, _ = oracle_dt(orc, wl)
    s = make_solver(wl)
    opts = StepOpts(dt=tau, passes=2)
    ckpt, lam = s.forward_checkpointed(opts, 2, 2)
    seed = np.random.default_rng(5).standard_normal(ckpt.shape[1:])
    dT0, dk0 = s.adjoint(opts, 2, 2, ckpt, lam, torch.from_numpy(seed))
    g = orc.make_grid(wl["n"], wl["h"], wl["bc"])
    f = wl["fields"]
    oT, ok = orc.heat_adjoint(g, wl["phases"], orc.StepOpts(tau=tau, passes=2), 2, np.array(lam), f["alpha2"], f["m1"],
                              f["m2"], f["T1"], seed)[:2]
    assert rel_err(dT0.cpu().numpy(), oT) <= 1e-12
    assert max(abs(dk0[k] - ok[k]) for k in range(2)) <= 1e-10 * max(abs(x) for x in ok)
    s.close()
