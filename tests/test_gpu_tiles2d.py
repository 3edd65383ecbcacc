"""GPU parity of the blocked 2D stages over the tile shapes a launch can take.

The shape (128 x 64, 64 x 128, 64 x 64 or 64 x 32 extended cells) and the number of
stages per launch follow from the grid, so the grids below lead to each of
them, with walls and periodic wraps, odd widths (no pairs across the wrap),
one more cell than a whole number of tiles, harmonic faces, and passes of
many and of few stages.  Bars as everywhere: FP64 1e-12, FP32 form 1e-5 per
field against the FP64 oracle (max-norm, relative)."""
import pytest

from paper_2106_00282_amd import workloads as W
from _cases import oracle_dt, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

CASES = [  # nx, ny, walls (x, y), face mean, dt factor, Spitzer-Harm law
    (38, 47, (1, 1), 0, 237.0, False),
    (129, 32, (0, 1), 1, 60.0, False),
    (2, 40, (1, 0), 0, 90.0, False),
    (93, 185, (0, 0), 0, 300.0, True),
    (400, 330, (1, 0), 0, 3.0, False),
    (657, 491, (0, 0), 1, 120.0, False),
    (800, 700, (0, 1), 0, 200.0, True),
    (1025, 700, (0, 0), 0, 200.0, False),
    (1025, 700, (1, 1), 0, 200.0, False),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,walls,face,factor,spitzer", CASES)
def test_tile_shapes_2d(nx, ny, walls, face, factor, spitzer, precision):
    from oracle import oracle as orc
    wl = (W.levelset2d_spitzer if spitzer else W.levelset2d)(max(nx, ny))
    wl["n"] = (nx, ny, 1)
    wl["h"] = (1.0 / max(nx, ny),) * 2 + (1.0,)
    wl["fields"] = {k: v[:, :ny, :nx].copy() for k, v in wl["fields"].items()}
    wl["bc"] = tuple(W.ADIABATIC if w else W.PERIODIC for w in walls) + (W.PERIODIC,)
    wl["dt_factor"] = factor
    tau, _ = oracle_dt(orc, wl)
    fo, ro = run_oracle(orc, wl, tau, 2, passes=2, face_mean=face)
    print(f"case {nx}x{ny} walls={walls} face={face} {precision} P={[r['P'] for r in ro]}", flush=True)
    fg, rg, s = run_gpu(wl, tau, 2, passes=2, precision=precision, frozen=[r["lambda_G"] for r in ro], face_mean=face)
    assert [r["P"] for r in rg] == [r["P"] for r in ro]
    tol = 1e-12 if precision == "fp64" else 1e-5
    errs = {k: rel_err(fg[k], fo[k]) for k in ("T1", "alpha2")}
    for k, e in errs.items():
        assert e <= tol, (k, e, errs)
    s.close()
