"""The two-launch D3Q19 step (moments, then force and collision), which small and ragged boxes take
by default, against the fused launch on the same box: the per-node arithmetic is the same, so the
populations agree bit for bit.  Boxes at the edges of its 32 x 8 tiles and z chunks of 1, 2 and 4
planes, every collision, walls and body force, the tabulated equation of state, both storages."""
import numpy as np
import pytest

from eos_tables import vdw_table
from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm

pytestmark = pytest.mark.gpu

MRT = dict(collision=lbm.LBM_COLLISION_MRT, s_e=1.19, s_eps=1.4, s_q=1.2, s_m=1.98)
KINDS = {"tau1": {}, "tau": dict(tau=0.8), "mrt": dict(tau=0.8, **MRT)}


def _case(scene, shape, kind):
    params = I.physics(**KINDS[kind])
    if scene == "boil":
        case = I.pool_boiling_3d(shape=shape, params=params, gravity=1e-4)
        case["u0"][0] += 0.05
        return case
    case = I.droplet_3d(shape=shape, radius=5.0, params=params, velocity=(0.07, -0.04, 0.03))
    if scene == "table":
        case["params"] = dict(params, eos_table=vdw_table())
    return case


def _both(case, storage, steps):
    args = (case["Q"], case["params"], case["rho0"], case["u0"], case["T0"])
    with lbm.Sim(*args, storage_bytes=storage) as a, lbm.Sim(*args, storage_bytes=storage) as b:
        b.set_launch(0, 0)          # the fused launch
        for s in (a, b):
            s.step(steps)
        ta, tb = a.step_reduce(1), b.step_reduce(1)
        assert a.checkpoint() == b.checkpoint()
    # the totals sum the same stored values in another order (bound as for the fused totals)
    assert np.abs(ta[:4] - tb[:4]).max() <= 1e-12 * abs(tb[0])
    assert abs(ta[4] - tb[4]) <= 1e-12 * abs(tb[4])


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("scene,kind", [("drop", "tau1"), ("drop", "tau"), ("drop", "mrt"), ("boil", "tau1"),
                                        ("boil", "mrt"), ("table", "tau1"), ("table", "tau")])
def test_two_launches_match_the_fused_step_bitwise(scene, kind, storage):
    for shape in ((2, 9, 33), (3, 8, 32), (5, 7, 65), (1, 1, 50), (28, 36, 40), (7, 1, 31)):
        if scene == "boil" and shape[0] < 2:
            continue
        print("two launches: %s %s %s %dB" % (scene, kind, shape, storage), flush=True)
        _both(_case(scene, shape, kind), storage, 7)


@pytest.mark.parametrize("scene,shape", [("drop", (41, 52, 75)), ("boil", (97, 150, 200)),
                                         ("drop", (73, 130, 201))])
def test_two_launches_on_longer_chunks(scene, shape):
    """Chunks of 2 planes (odd height), and of 4 with one plane left over."""
    print("two launches: %s %s" % (scene, shape), flush=True)
    _both(_case(scene, shape, "tau1"), 4, 3)


# Chunks of 2 planes (788 and 524 tiles) and of 4 (6158 and 4102), at heights that leave one and three planes over, in
# boxes whose steps run as two launches with every collision, with totals too (checked on the CPU).
CHUNKED = [(4, (197, 9, 33)), (4, (3079, 8, 33)), (8, (131, 9, 33)), (8, (2051, 8, 63))]


@pytest.mark.parametrize("storage,shape", CHUNKED)
@pytest.mark.parametrize("scene,kind", [("drop", "tau1"), ("drop", "tau"), ("drop", "mrt"), ("boil", "tau1"), ("boil", "tau"),
                                        ("boil", "mrt"), ("table", "tau1"), ("table", "tau"), ("table", "mrt")])
def test_every_form_on_chunks_of_two_and_four(scene, kind, storage, shape):
    print("two launches on chunks: %s %s %s %dB" % (scene, kind, shape, storage), flush=True)
    _both(_case(scene, shape, kind), storage, 3)


TERMS = {"none": 0, "work": I.WORK, "conduction": I.CONDUCTION, "latent": I.LATENT, "pseudoforce": I.PSEUDOFORCE,
         "latent at T0": I.LATENT | I.BAROTROPIC, "barotropic": I.ALL_TERMS | I.BAROTROPIC}


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("terms", sorted(TERMS))
def test_single_terms_and_temperatures_beyond_the_band(terms, storage):
    """Each term by itself and the barotropic pressure, on a drop in a gas that is below the latent band's range
    on one side and supercritical on the other."""
    shape = (11, 18, 47)
    case = I.droplet_3d(shape=shape, radius=4.0, params=I.physics(flags=TERMS[terms], T0_baro=0.85),
                        velocity=(0.03, -0.02, 0.01))
    x = np.arange(shape[2])
    case["T0"][:] = np.where(x < 8, 0.38, np.where(x > 38, 1.2, case["T0"]))
    case["rho0"][:, :, (x < 8) | (x > 38)] = 0.05
    print("two launches: %s %dB" % (terms, storage), flush=True)
    _both(case, storage, 4)
