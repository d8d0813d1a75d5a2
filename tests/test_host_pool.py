"""The serving pool's host code with a HIP runtime that computes nothing (hostrun.py): which form of the step a load
of requests takes, in which order its launches run, and what the pool holds."""
import pytest

import hostrun

KINDS = """
from eos_tables import vdw_table
MRT = dict(tau=0.8, collision=1, s_e=1.19, s_eps=1.4, s_q=1.2, s_m=1.98)

def request(pool, kind, e):
    kw = dict(MRT) if kind.endswith("m") else {}
    if kind[0] == "b":
        kw["gravity"] = (0.0, 0.0, -1e-5)
    if kind[0] == "t":
        kw["eos_table"] = vdw_table()
    sh = (e, e, e)
    t = pool.submit(I.physics(**kw), np.full(sh, 0.2), np.zeros((3,) + sh), np.full(sh, 0.85), 1000)
    assert t is not None
"""


def _launches_of_a_run(load):
    return hostrun.run(KINDS + """
pool = lbm.Pool(6 << 30, max_slots=16, steps_per_run=1)
for kind, e in %r:
    request(pool, kind, e)
launches()
pool.run()
result([k for k, *_ in launches()])
""" % (load,))


@pytest.mark.parametrize("load,split", [
    # two launches 1.2 to 10 times as fast
    ([("b", 32), ("bm", 32)], True), ([("p", 64), ("b", 64)], True), ([("p", 96), ("b", 96)], True),
    ([(k, 48) for k in ("p", "b", "t", "pm", "bm", "tm")], True), ([(k, 96) for k in ("p", "b", "t", "pm")], True),
    # fused 3 to 15% faster
    ([(k, 120) for k in ("p", "b", "t", "pm")], False), ([("p", 96), ("b", 96), ("p", 96), ("b", 96)], False),
    ([("p", 128), ("b", 128)], False),
])
def test_form_of_loads_of_several_kinds(load, split):
    kernels = _launches_of_a_run(load)
    steps = [k for k in kernels if k in ("k_pool_moments", "k_pool_collide", "k_pool_step")]
    kinds = len(set(k for k, _ in load))
    if not split:
        assert steps == ["k_pool_step"] * kinds
    else:
        assert steps.count("k_pool_collide") == kinds and "k_pool_step" not in steps
        # every collision comes right behind the moments of its class (periodic, walls, table)
        classes = len(set(k[0] for k, _ in load))
        assert steps.count("k_pool_moments") == classes and steps[0] == "k_pool_moments"
        assert "k_pool_momentsk_pool_moments" not in "".join(steps)


def test_what_a_pool_holds_and_its_fallback_without_room_for_the_workspace():
    """Creation is one device allocation: the budget, staging for the largest request, and a workspace of an eighth of
    the budget; without room for the workspace the same pool runs fused steps, without room for the rest creation
    fails and leaves nothing; destruction gives everything back."""
    got = hostrun.run(KINDS + """
budget, out = 1 << 30, {}
def form():   # (the fused graph of periodic requests is captured at creation)
    launches()
    pool.run()
    return ([k for k, *_ in launches()] or ["k_pool_step"])[0]

m0 = fake.fake_mallocs()
pool = lbm.Pool(budget, max_slots=16, steps_per_run=1)
out["mallocs"], out["held"] = fake.fake_mallocs() - m0, fake.fake_held()
request(pool, "p", 32)
out["form"] = form()
pool.close()
out["left"] = fake.fake_held()
for name, room in (("tight", out["held"] - budget // 8), ("short", out["held"] - budget // 8 - 4096)):
    fake.fake_capacity(room)
    try:
        pool = lbm.Pool(budget, max_slots=16, steps_per_run=1)
        request(pool, "p", 32)
        out[name] = [form(), fake.fake_held() <= room]
        pool.close()
    except lbm.LbmError as e:
        out[name] = e.status
    out[name + " left"] = fake.fake_held()
result(out)
""")
    staging = (5 + 8) * 8 * 128 ** 3
    assert got["mallocs"] == 1
    assert (1 << 30) * 9 // 8 + staging <= got["held"] <= (1 << 30) * 9 // 8 + staging + (1 << 20)
    assert got["form"] == "k_pool_moments" and got["left"] == 0
    assert got["tight"] == ["k_pool_step", True] and got["tight left"] == 0
    assert got["short"] == -2 and got["short left"] == 0
