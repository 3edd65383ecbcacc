"""What the final stage's flux form keeps: T^n plus differences of T, so a uniform
temperature in pure phases stays as it is, bit for bit, and the heat
sum C T of any state changes by the rounding of single cells only.

The bar of the sum: a step rounds a cell's T by some ulps of it (32 allowed), in
either direction alike, so the mean over N cells moves by 32 2^-53 / sqrt(N) per
step at most (half a step's ulp common to all cells is 2^-53)."""
import math

import numpy as np
import pytest

from paper_2106_00282_amd import workloads as W
from paper_2106_00282_amd.tlim import StepOpts
from _cases import make_solver
from test_stage_plan import BLOCKED_MARCH, LINE, TILES, stage_plan

pytestmark = pytest.mark.gpu

GRIDS = [((1024, 1024), (TILES, 128, 64)), ((1025, 700), (TILES, 64, 128)), ((400, 400), (TILES, 64, 64)),
         ((140, 140), (TILES, 64, 32)), ((96, 64, 33), (BLOCKED_MARCH, 64, 24)), ((5000,), (LINE, 256, 1))]


def pure(n):
    """Two pure phases with a straight interface."""
    wl = W.levelset2d(8)
    n = tuple(n) + (1,) * (3 - len(n))
    a = np.zeros(n[::-1])
    a[..., : n[0] // 3] = 1.0
    rho = (wl["fields"]["m1"] / (1.0 - wl["fields"]["alpha2"])).flat[0], (wl["fields"]["m2"] / wl["fields"]["alpha2"]).flat[0]
    wl["n"], wl["h"], wl["bc"] = n, (1.0 / n[0],) * 3, (W.PERIODIC,) * 3
    wl["fields"] = dict(alpha2=a, m1=(1.0 - a) * rho[0], m2=a * rho[1])
    return wl


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,plan", GRIDS)
def test_uniform_temperature_stays(n, plan, precision):
    p = stage_plan(n)
    assert (p.kernel, p.tile_x, p.tile_y) == plan
    wl = pure(n)
    rng = np.random.default_rng(7)
    s = None
    for T in rng.uniform(0.5, 2.0, 8):
        wl["fields"]["T1"] = np.full_like(wl["fields"]["alpha2"], T)
        wl["fields"]["T2"] = wl["fields"]["T1"]
        if s is None:
            s = make_solver(wl, precision)
        s.set_workload(wl)
        dt = 200.0 * 2.0 / s.spectral_bound()
        for _ in range(5):
            assert s.advance(StepOpts(dt=dt, passes=2, whole_step=2), report=False)[0] == 0
        assert s.finish() == 0
        got = s.get_field("T1").cpu().numpy()
        print(f"case {n} {precision} T={T!r} {np.unique(got)[:3]}", flush=True)
        assert (got == T).all()
    s.close()


@pytest.mark.parametrize("n,plan", GRIDS)
def test_heat_is_kept_to_rounding(n, plan):
    wl = pure(n)
    N, steps = wl["fields"]["alpha2"].size, 8
    # one heat capacity everywhere: the heat is the sum of T
    cv = [p["cv"] for p in wl["phases"]]
    a = wl["fields"]["alpha2"]
    wl["fields"]["m1"], wl["fields"]["m2"] = (1.0 - a) / cv[0], a / cv[1]
    s = None
    for seed in range(4):
        rng = np.random.default_rng(seed)
        wl["fields"]["T1"] = rng.uniform(1.0, 1.9, a.shape)
        wl["fields"]["T2"] = wl["fields"]["T1"]
        if s is None:
            s = make_solver(wl)
        s.set_workload(wl)
        dt = 200.0 * 2.0 / s.spectral_bound()
        for _ in range(steps):
            assert s.advance(StepOpts(dt=dt, passes=2, whole_step=2), report=False)[0] == 0
        assert s.finish() == 0
        h0 = math.fsum(wl["fields"]["T1"].ravel())
        h1 = math.fsum(s.get_field("T1").cpu().numpy().ravel())
        print(f"case heat {n} seed={seed} {h1 / h0 - 1.0:.2e} {(h1 - h0) / h0:.2e}", flush=True)
        assert abs(h1 - h0) <= steps * 32 * 2.0 ** -53 / math.sqrt(N) * h0
    s.close()
