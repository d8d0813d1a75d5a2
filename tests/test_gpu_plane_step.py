"""The forms of the D2Q9 step on its default tiles (two, three or four tiles per CU, chosen by the number
of tiles) against the 64 x 8 tiles, which have one form: the per-node arithmetic is the same, so the
populations agree bit for bit.  Boxes on both sides of the lines where the form changes (512, 768, 1024 and
2048 tiles), ragged in x and y, every collision, body force and the tabulated equation of state,
both storages."""
import numpy as np
import pytest

from eos_tables import vdw_table
from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm

pytestmark = pytest.mark.gpu

KINDS = {"tau1": {}, "tau": dict(tau=0.8),
         "mrt": dict(tau=0.8, collision=lbm.LBM_COLLISION_MRT, s_e=1.19, s_eps=1.4, s_q=1.2, s_m=1.98)}


def _step(sim, n):
    """Status of n steps (a state that leaves the EOS domain has to do so in every form)."""
    try:
        sim.step(n)
    except lbm.LbmError as e:
        return e.status
    return lbm.LBM_OK


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("nx,ny", [(512, 256), (513, 255), (512, 385), (511, 377), (512, 512), (512, 513), (1025, 491)])
def test_forms_match_bitwise(nx, ny, kind, storage):
    params = I.physics(**KINDS[kind])
    rng = np.random.default_rng(nx * ny)
    y = np.arange(ny)[None, :, None]
    rho0 = np.where((y > ny // 4) & (y < ny // 2), 1.9, 0.25) * (1 + 0.01 * rng.uniform(-1, 1, (1, ny, nx)))
    u0 = 0.02 * rng.uniform(-1, 1, (3, 1, ny, nx))
    u0[2] = 0.0
    T0 = np.full((1, ny, nx), 0.85)
    for extra in ({}, dict(gravity=(1e-5, -2e-5, 0.0)), dict(eos_table=vdw_table())):
        print("plane step: %dx%d %s %dB %s" % (nx, ny, kind, storage, sorted(extra)), flush=True)
        with lbm.Sim(9, dict(params, **extra), rho0, u0, T0, storage_bytes=storage) as a, \
                lbm.Sim(9, dict(params, **extra), rho0, u0, T0, storage_bytes=storage) as b:
            a.set_launch(0, 0)
            b.set_launch(2, 0)
            assert _step(a, 3) == _step(b, 3)
            assert a.checkpoint() == b.checkpoint()


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("n", [390, 500, 560])
def test_forms_match_bitwise_with_a_table(n, kind, storage):
    case = I.slab_2d(n=n, width=120, params=I.physics(**KINDS[kind]))
    params = dict(case["params"], eos_table=vdw_table())
    args = (9, params, case["rho0"], case["u0"], case["T0"])
    print("plane step: slab %d^2 table %s %dB" % (n, kind, storage), flush=True)
    with lbm.Sim(*args, storage_bytes=storage) as a, lbm.Sim(*args, storage_bytes=storage) as b:
        a.set_launch(0, 0)
        b.set_launch(2, 0)
        assert _step(a, 3) == _step(b, 3) == lbm.LBM_OK
        assert a.checkpoint() == b.checkpoint()


@pytest.mark.parametrize("storage", [4, 8])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("nx,ny", [(512, 256), (513, 255), (512, 385), (511, 377), (512, 513), (1025, 491)])
def test_forms_match_bitwise_with_a_table_at_the_lines(nx, ny, kind, storage):
    """The table on a slab that stays in its domain, on the boxes at the lines where the form changes."""
    n = max(nx, ny)
    case = I.slab_2d(n=n, width=n // 3, params=I.physics(**KINDS[kind]))
    args = (9, dict(case["params"], eos_table=vdw_table()), case["rho0"][:, :ny, :nx].copy(),
            case["u0"][:, :, :ny, :nx].copy(), case["T0"][:, :ny, :nx].copy())
    print("plane step: slab %dx%d table %s %dB" % (nx, ny, kind, storage), flush=True)
    with lbm.Sim(*args, storage_bytes=storage) as a, lbm.Sim(*args, storage_bytes=storage) as b:
        a.set_launch(0, 0)
        b.set_launch(2, 0)
        assert _step(a, 3) == _step(b, 3) == lbm.LBM_OK
        same = a.checkpoint() == b.checkpoint()
        assert same
