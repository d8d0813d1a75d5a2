"""The checks of the initial fields run on several threads over long boxes: the lowest faulty node is
the one that is reported, wherever it lies, with the message of its own fault."""
import numpy as np
import pytest

from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm


@pytest.mark.parametrize("node", [0, 1, 16383, 16384, 32767, 32768, 131071, 131072, 262142])
def test_lowest_faulty_node_is_reported(node):
    shape = (64, 64, 64)
    case = I.droplet_3d(shape=shape, radius=10.0, params=I.physics())
    rho0, u0, T0 = (np.array(case[k]) for k in ("rho0", "u0", "T0"))
    u0[1].flat[node] = np.nan
    T0.flat[node + 1:] = -1.0
    with pytest.raises(lbm.LbmError) as e:
        lbm.Sim(19, case["params"], rho0, u0, T0, storage_bytes=4)
    assert e.value.status == lbm.LBM_EINVAL and "node %d: non-finite velocity" % node in str(e.value)
