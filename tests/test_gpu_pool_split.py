"""The serving pool's two forms of a step, the fused tiles and the two launches that a lightly loaded
pool takes, against a simulation that runs the fused launch: the per-node arithmetic is the same, so
the results agree bit for bit.  Ragged boxes at the edges of the 32 x 8 tiles, every kind of request
(periodic, walls and gravity, tabulated equation of state, BGK and MRT), replays of an even and of an
odd number of steps, requests that end within a replay, and a load that passes from one form to the
other while it drains."""
import numpy as np
import pytest

from eos_tables import vdw_table
from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm

pytestmark = pytest.mark.gpu

MRT = dict(collision=lbm.LBM_COLLISION_MRT, s_e=1.19, s_eps=1.4, s_q=1.2, s_m=1.98)


def _case(scene, shape, kw):
    params = I.physics(**kw)
    if scene == "boil":
        return I.pool_boiling_3d(shape=shape, params=params, gravity=1e-4)
    case = I.droplet_3d(shape=shape, radius=4.0, params=params, velocity=(0.07, -0.04, 0.03))
    if scene == "table":
        case["params"] = dict(params, eos_table=vdw_table())
    return case


def _fused(case, steps):
    with lbm.Sim(19, case["params"], case["rho0"], case["u0"], case["T0"], storage_bytes=4) as s:
        s.set_launch(0, 0)
        s.step(steps)
        return s.moments()


def _pool(cases, steps, spr):
    with lbm.Pool(1 << 31, max_slots=12, steps_per_run=spr) as pool:
        tickets = [pool.submit(c["params"], c["rho0"], c["u0"], c["T0"], n) for c, n in zip(cases, steps)]
        for _ in range((max(steps) + spr - 1) // spr):
            pool.run()
        assert all(pool.poll(t) == (True, lbm.LBM_OK) for t in tickets)
        return [pool.collect(t)[0] for t in tickets]


def _check(cases, steps, spr):
    for case, n, got in zip(cases, steps, _pool(cases, steps, spr)):
        want = _fused(case, n)
        for k in want:
            assert np.array_equal(got[k], want[k]), (case["rho0"].shape, n, k)


@pytest.mark.parametrize("spr", [1, 3, 4])
def test_light_load_of_every_kind(spr):
    cases = [_case("drop", (9, 17, 33), {}), _case("boil", (12, 8, 31), {}), _case("table", (7, 9, 32), {}),
             _case("drop", (16, 15, 34), dict(tau=0.8)), _case("drop", (8, 7, 65), dict(tau=0.8, **MRT)),
             _case("boil", (11, 16, 9), dict(tau=0.8, **MRT)), _case("table", (5, 23, 12), dict(tau=0.8, **MRT)),
             _case("boil", (2, 25, 64), dict(tau=0.7))]
    print("light pool, %d steps per replay" % spr, flush=True)
    _check(cases, [7, 12, 5, 9, 11, 8, 10, 6], spr)


def test_load_passing_from_the_fused_form_to_two_launches():
    cases = [_case("drop", (128, 128, 128), {}), _case("drop", (128, 128, 127), {}), _case("drop", (33, 48, 65), {})]
    print("draining pool", flush=True)
    _check(cases, [4, 4, 15], 4)


def _tall(scene, nz, kw, ny=9):
    """A box of 33 x ny nodes a plane, 2 x ceil(ny / 8) tiles."""
    return _case(scene, (nz, ny, 33), kw)


def test_every_kind_on_chunks_of_two():
    """Twelve requests, 828 or 840 tiles of each kind, more than a launch has workgroups: chunks of 2 planes,
    workgroups that go on to a second tile of another request, requests that end within a replay."""
    kinds = [("drop", {}), ("boil", {}), ("table", {}), ("drop", dict(tau=0.8, **MRT)), ("boil", dict(tau=0.8, **MRT)),
             ("table", dict(tau=0.8, **MRT))]
    cases = [_tall(scene, nz, kw) for nz in (127, 80) for scene, kw in kinds]
    cases[6] = _tall("drop", 83, dict(tau=0.8))
    print("pool of every kind, chunks of 2", flush=True)
    _check(cases, [7, 9, 5, 8, 6, 10, 9, 4, 7, 5, 8, 3], 4)


def test_one_kind_on_chunks_of_four():
    """Twelve requests of 15180 tiles: chunks of 4 planes, with up to three left over."""
    cases = [_tall("drop", nz, kw, ny=33) for nz, kw in zip((125, 126, 127, 128) * 3, ({}, {}, dict(tau=0.8)) * 4)]
    print("pool, chunks of 4", flush=True)
    _check(cases, [3, 5, 4, 6, 5, 3, 4, 5, 6, 3, 4, 5], 3)


@pytest.mark.parametrize("kind", ["walls", "table", "mrt"])
def test_other_kinds_on_chunks_of_four(kind):
    scene = {"walls": "boil", "table": "table", "mrt": "drop"}[kind]
    kw = dict(tau=0.8, **MRT) if kind == "mrt" else {}
    cases = [_tall(scene, nz, kw, ny=33) for nz in (125, 126, 127, 128) * 3]
    print("pool, chunks of 4, %s" % kind, flush=True)
    _check(cases, [3, 5, 4, 6, 5, 3, 4, 5, 6, 3, 4, 5], 3)
