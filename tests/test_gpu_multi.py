"""Several D2Q9 steps per launch, which small boxes take by default, against the fused single-step
launch on the same box: the same per-node arithmetic with the populations rounded to the storage
type after every step, so the populations agree bit for bit, whatever the number of steps leaves
for the last launch.  Rows and columns of one node, boxes narrower than a tile's halo, ragged
tiles, the largest box, both storages, every collision, body force, the tabulated EOS."""
import numpy as np
import pytest

from eos_tables import vdw_table
from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm

pytestmark = pytest.mark.gpu

MRT = dict(collision=lbm.LBM_COLLISION_MRT, s_e=1.19, s_eps=1.4, s_q=1.2, s_m=1.98)
KINDS = {"tau1": {}, "tau": dict(tau=0.8), "mrt": dict(tau=0.8, **MRT), "gravity": dict(gravity=(1e-5, -2e-5, 0.0)),
         "table": dict(eos_table=vdw_table())}


def _box(ny, nx, kind):
    n = max(nx, ny, 8)
    c = I.slab_2d(n=n, width=n // 3, params=I.physics(**KINDS[kind]))
    u = c["u0"][:, :, :ny, :nx].copy()
    u[0] += 0.06
    u[1] -= 0.03
    return c["params"], c["rho0"][:, :ny, :nx].copy(), u, c["T0"][:, :ny, :nx].copy()


def _compare(args, storage, counts):
    with lbm.Sim(9, *args, storage_bytes=storage) as a, lbm.Sim(9, *args, storage_bytes=storage) as b:
        b.set_launch(0, 0)
        for n in counts:
            a.step(n)
            b.step(n)
            assert a.step_count == b.step_count
            assert a.checkpoint() == b.checkpoint(), n


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_several_steps_per_launch_match_single_steps_bitwise(kind, storage):
    for ny, nx in ((1, 300), (300, 1), (1, 1), (3, 5), (2, 64), (45, 70), (17, 129)):
        print("several steps per launch: %s %dx%d %dB" % (kind, nx, ny, storage), flush=True)
        _compare(_box(ny, nx, kind), storage, (1, 2, 23))


@pytest.mark.parametrize("ny,nx", [(128, 128), (256, 256), (1, 5003)])
def test_several_steps_per_launch_on_larger_boxes(ny, nx):
    print("several steps per launch: %dx%d" % (nx, ny), flush=True)
    _compare(_box(ny, nx, "tau1"), 8, (5, 12))


def test_a_node_that_leaves_the_domain_is_reported():
    """A step count inside one launch: the error word is set by whichever step the node leaves in."""
    params, rho, u, T = _box(40, 40, "tau1")
    params = dict(params, tau=0.501)
    u[0] += 0.3
    with lbm.Sim(9, params, rho, u, T, storage_bytes=8) as s:
        with pytest.raises(lbm.LbmError) as e:
            s.step(400)
        assert e.value.status == lbm.LBM_EUNSTABLE


TERMS = {"none": 0, "work": I.WORK, "conduction": I.CONDUCTION, "latent": I.LATENT, "pseudoforce": I.PSEUDOFORCE,
         "latent at T0": I.LATENT | I.BAROTROPIC, "barotropic": I.ALL_TERMS | I.BAROTROPIC}


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("terms", sorted(TERMS))
def test_single_terms_and_temperatures_beyond_the_band(terms, storage):
    """Each term by itself and the barotropic pressure, with gas below the latent band's range on one side and
    supercritical on the other."""
    params, rho, u, T = _box(45, 70, "tau1")
    params = dict(params, flags=TERMS[terms], T0_baro=0.85)
    x = np.arange(70)
    T[:] = np.where(x < 10, 0.38, np.where(x > 60, 1.2, T))
    rho[:, :, (x < 10) | (x > 60)] = 0.05
    print("several steps per launch: %s %dB" % (terms, storage), flush=True)
    _compare((params, rho, u, T), storage, (1, 2, 7))
