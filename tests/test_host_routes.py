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


MEMORY = """
def held(Q, shape, storage, **kw):
    # bytes beyond the footprint after creation, then what moments on the host, moments on the device and a step with
    # totals add
    s = case(Q, shape, storage, **kw)
    out = [fake.fake_held() - lbm.lbm_footprint_bytes(s.params)]
    for use in (s.moments, lambda: lbm.lbm_moments_device(s.handle, 256, 512, 768, 1024), lambda: s.step_reduce(1)):
        before = fake.fake_held()
        use()
        out.append(fake.fake_held() - before)
    s.close()
    return out + [fake.fake_held()]
"""


@pytest.mark.parametrize("q,shape,storage,kw,split", [
    (9, (1, 1, 1000), 8, "", 0), (9, (1, 128, 128), 8, "", 0), (9, (1, 600, 600), 4, "", 0),
    (19, (32, 32, 32), 4, "", 36), (19, (75, 52, 41), 8, "tau=0.8", 56), (19, (128, 128, 128), 4, "tau=0.8", 0),
])
def test_device_memory_of_a_simulation(q, shape, storage, kw, split):
    """Beside its footprint a simulation holds some rounding (none to speak of for a small state) and, where its steps
    are two launches, their workspace; moments add 16 bytes per node where there is no workspace."""
    n = shape[0] * shape[1] * shape[2]
    pitch = -(-shape[2] * storage // 128) * 128 // storage
    extra, host, device, totals, left = hostrun.run(MEMORY + "result(held(%d, %r, %d, %s))" % (q, shape, storage, kw))
    state = 4 * q * storage * n
    work = split * pitch * shape[0] * shape[1]
    assert work <= extra <= work + (65536 if state < 16 << 20 else 4 << 20) + 40 * (1024 + 8)
    assert host == 0
    assert device == (0 if split else 16 * n)
    assert totals <= 8 * (5 * 8192 + 8)
    assert left == 0


def test_steps_without_room_for_the_workspace():
    """No room for the workspace at creation: the fused step; none for the step with totals: its fused form, and the
    runtime is asked once only."""
    got = hostrun.run("""
out = []
for shape, kw in (((32, 32, 32), {}), ((128, 128, 128), {})):
    s = case(19, shape, 4, **kw)
    held = fake.fake_held()
    need = 36 * shape[0] * shape[1] * shape[2]
    s.close()
    # the box whose steps are two launches has its workspace inside what it holds, the other not
    fake.fake_capacity(held + 4096 - (need if shape[0] == 32 else 0) + 8 * (5 * 8192 + 8))
    s = case(19, shape, 4, **kw)
    launches()
    s.step_async(1)
    forms = [launches()[0][0]]
    calls = []
    for i in range(3):
        m = fake.fake_mallocs()
        s.step_reduce(1)
        calls.append(fake.fake_mallocs() - m)
    forms += [k for k, *_ in launches()][:2]
    s.moments()
    out.append([forms, calls])
    s.close()
    fake.fake_capacity((1 << 64) - 1)
result(out)
""")
    for forms, calls in got:
        assert forms == ["k_step", "k_step", "k_sum_partials"]
        assert calls == [2, 0, 0]     # the workspace refused, the totals' partial sums


def test_moments_clear_the_buffer_they_pass_through():
    """lbm_moments takes the population buffer of the next step for its fields, and clears it."""
    got = hostrun.run("""
out = []
for args in ((9, (1, 20, 31), 4), (19, (5, 9, 33), 8)):
    s = case(*args)
    for steps in (1, 2):
        launches()
        s.step_async(steps)
        last = launches()[-1]
        s.moments()
        seen = launches()
        out.append([last[3], seen[0][2], [x for x in seen if x[0] == "memset"],
                    (lbm.lbm_footprint_bytes(s.params) - 16 * 4096 - 64) // 2])
    s.close()
result(out)
""")
    for state, read, cleared, size in got:
        assert read == state
        assert len(cleared) == 1 and cleared[0][1] == size and cleared[0][2] != state


@pytest.mark.parametrize("kind", ["tau=1.0", "tau=0.8", MRT + "tau=0.8"])
@pytest.mark.parametrize("storage,shape,tiles,chunk", [(4, (197, 9, 33), 4, 2), (4, (3079, 8, 33), 2, 4),
                                                       (8, (131, 9, 33), 4, 2), (8, (2051, 8, 63), 2, 4)])
def test_boxes_whose_two_launches_march_through_chunks(storage, shape, tiles, chunk, kind):
    """The boxes of the GPU test of chunks run what it is there for."""
    got = hostrun.run("""
s = case(19, %r, %d, %s)
launches()
s.step_async(1)
s.step_reduce(1)
result([x[:2] for x in launches()])
""" % (shape, storage, kind))
    collide = ["k_split_collide", tiles * -(-shape[0] // chunk)]
    assert [x[0] for x in got] == ["k_split_moments", "k_split_collide"] * 2 + ["k_sum_partials"]
    assert got[1] == got[3] == collide
