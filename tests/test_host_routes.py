"""Which launches the library's host code makes, with a HIP runtime that computes nothing in the place of the
device's (hostrun.py): the number and order of launches and the buffers they go between."""
import pytest

import hostrun


@pytest.mark.parametrize("shape,several", [("(1, 1, 1000)", True), ("(1, 1, 7)", True), ("(1, 128, 128)", True),
                                           ("(1, 200, 256)", True), ("(1, 300, 310)", False)])
@pytest.mark.parametrize("storage", [4, 8])
def test_the_buffer_of_the_state_follows_the_step_count(shape, several, storage):
    """Several D2Q9 steps per launch: n steps go through as many launches as leave the state in the buffer that n
    single launches would, whatever n is."""
    got = hostrun.run("""
s = case(9, %s, %d)
launches()
out = []
for n in list(range(1, 70)) + [200, 1001]:
    s.step_async(n)
    steps = launches()
    # fields of the state, read from the buffer that holds it
    lbm.lbm_moments_device(s.handle, 256, None, None, None)
    where = launches()
    out.append([n, len(steps), steps[0][0], where[0][0], steps[0][2], steps[-1][3], where[0][2]])
result(out)
""" % (shape, storage))
    for n, count, form, moments, src, dst, where in got:
        assert (form, moments) == ("k_multi_step", "k_moments_a")
        assert count % 2 == n % 2 and count <= n
        assert dst == where and (src == where) == (n % 2 == 0)
    assert (max(n / count for n, count, *_ in got) > 1) == several


MRT = "collision=1, s_e=1.19, s_eps=1.4, s_q=1.2, s_m=1.98, "


@pytest.mark.parametrize("shape,storage,kind,form", [
    # the fused form was 8 to 16% faster
    ("(128, 128, 128)", 4, "tau=0.8", "k_step"), ("(64, 256, 256)", 4, "tau=0.8", "k_step"),
    ("(256, 200, 64)", 4, MRT + "tau=0.8", "k_step"), ("(112, 112, 112)", 4, MRT + "tau=0.8", "k_step"),
    # 4 to 7%
    ("(256, 200, 64)", 8, "tau=0.8", "k_step"), ("(64, 256, 256)", 8, "tau=0.8", "k_step"),
    ("(300, 96, 96)", 8, "tau=0.8", "k_step"), ("(200, 200, 200)", 4, "tau=0.8", "k_step"),
    # two launches 9 to 25%
    ("(64, 64, 64)", 4, "tau=0.8", "k_split_moments"), ("(80, 80, 80)", 4, MRT + "tau=0.8", "k_split_moments"),
    ("(100, 100, 100)", 8, "tau=0.8", "k_split_moments"), ("(128, 128, 128)", 8, MRT + "tau=1.0", "k_split_moments"),
    # tau = 1 and FP64 MRT throughout
    ("(128, 128, 128)", 4, "tau=1.0", "k_split_moments"), ("(64, 256, 256)", 4, "tau=1.0", "k_split_moments"),
    ("(64, 256, 256)", 8, "tau=1.0", "k_split_moments"), ("(64, 256, 256)", 8, MRT + "tau=0.8", "k_split_moments"),
    # states of 4 GB, and planes
    ("(400, 300, 240)", 4, "tau=1.0", "k_step"), ("(1, 300, 240)", 4, "tau=1.0", "k_step"),
])
def test_the_step_with_totals_takes_the_faster_form(shape, storage, kind, form):
    """The form of lbm_step_reduce's last step against what was measured; and a simulation that takes the fused form
    there holds no scratch for the other."""
    q = 9 if shape.startswith("(1,") else 19
    got = hostrun.run("""
s = case(%d, %s, %d, %s)
held = fake.fake_held()
launches()
s.step_reduce(1)
result([[k for k, *_ in launches()], fake.fake_held() - held])
""" % (q, shape, storage, kind))
    kernels, grown = got
    assert kernels[0] == form
    if form == "k_step":
        assert kernels[:2] == ["k_step", "k_sum_partials"]
        assert grown <= 8 * (5 * 8192 + 8)
    else:
        assert kernels[:3] == ["k_split_moments", "k_split_collide", "k_sum_partials"]


@pytest.mark.parametrize("shape,storage,form", [
    # single steps were 3 to 11% faster
    ("(1, 320, 320)", 8, "k_step"), ("(1, 200, 500)", 8, "k_step"), ("(1, 316, 310)", 8, "k_step"),
    ("(1, 208, 480)", 8, "k_step"), ("(1, 450, 220)", 8, "k_step"), ("(1, 360, 360)", 8, "k_step"),
    ("(1, 360, 360)", 4, "k_step"),
    # the other form 5 to 21%
    ("(1, 300, 300)", 8, "k_multi_step"), ("(1, 320, 304)", 8, "k_multi_step"), ("(1, 2400, 40)", 8, "k_multi_step"),
    ("(1, 320, 320)", 4, "k_multi_step"), ("(1, 350, 350)", 4, "k_multi_step"),
])
def test_plane_steps_take_the_faster_form(shape, storage, form):
    got = hostrun.run("""
s = case(9, %s, %d)
launches()
s.step_async(2)
result([k for k, *_ in launches()])
""" % (shape, storage))
    assert len(set(got)) == 1 and got[0].startswith(form)   # (k_step, or k_step_waves)
