"""Which kernels a call launches, on the HIP runtime without a device.

A call takes a combined launch only where that was measured to be the faster
one; both routes give the same results (tests on the GPU).
"""
from test_host_memory_cpu import fake, pytestmark  # noqa: F401


def test_spline_adjoint_takes_one_launch_for_narrow_cells_only(fake):  # noqa: F811
    code = """
f = Fake()
def nodes(n, step):
    return np.append(np.arange(0, n - 1, step), n - 1.0) * 10.0
for nz, nx, sz, sx in ((300, 1700, 10, 10), (300, 1700, 10, 64), (2000, 2500, 64, 10), (100, 200, 64, 64), (100, 200, 30, 200),
                       (300, 1700, 250, 250), (2000, 2500, 10, 64), (2000, 2500, 250, 250), (2000, 300, 64, 64),
                       (2000, 2500, 1000, 250), (500, 2500, 30, 200)):
    before = f.launched("k_spline_adjoint1")
    assert f.spline(nz, nx, nodes(nz, sz), nodes(nx, sx), True) == 0
    print(f.launched("k_spline_adjoint1") - before)
# one wide cell among narrow ones
before = f.launched("k_spline_adjoint1")
assert f.spline(2000, 2500, np.append(nodes(500, 10), 20000.0), nodes(2500, 64), True) == 0
print(f.launched("k_spline_adjoint1") - before)
"""
    assert fake(code) == ["1"] * 5 + ["0"] * 7


def test_lbfgs_direction_of_long_vectors_takes_the_recursion(fake):  # noqa: F811
    code = """
f = Fake()
for n, k in ((5985, 1), (5985, 15), (3000000, 1), (6000000, 2), (6000000, 15), (3000001, 1), (6000001, 2), (31000000, 15),
             (5985, 16)):
    before = f.launched("k_lbfgs_gram")
    assert f.lbfgs(n, k) == 0
    print(f.launched("k_lbfgs_gram") - before)
"""
    assert fake(code) == ["1"] * 5 + ["0"] * 4
