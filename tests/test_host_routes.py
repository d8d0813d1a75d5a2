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
