"""The FP64 Sternheimer solver that keeps p in LDS and r, A p in registers, on
grids at the edges of what it takes: smallest planes, most planes per thread,
full LDS, one and many column groups, a last plane that only some groups have,
and the first grids beyond each limit (which the marching solver takes)."""
import numpy as np
import pytest

from test_gpu_cocg_shapes import P, _check  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [(7, 9, 15), (7, 8, 16), (13, 9, 20), (12, 24, 32), (13, 24, 32), (24, 16, 24), (11, 17, 44),
                               (19, 12, 15)])
def test_resident_solver_shapes(P, n):  # noqa: F811
    _check(P, n, "fp64", False)


def test_resident_solves_do_not_depend_on_the_batch(P):  # noqa: F811
    n, n_occ = (13, 9, 20), 3
    N = int(np.prod(n))
    L = tuple(0.45 * v for v in n)
    rng = np.random.default_rng(3)
    psi = np.linalg.qr(rng.standard_normal((N, n_occ)))[0].T / np.sqrt(0.45 ** 3)
    h = P.Handle(n, L, rng.uniform(-2, 0, N), psi, np.array([-0.9, -0.6, -0.4]), stern_tol=1e-9)
    u = torch.from_numpy(rng.standard_normal((40, N)))
    every = h.chi0_apply(0.3, u)[0]
    for k in (0, 17, 39):
        assert torch.equal(every[k], h.chi0_apply(0.3, u[k:k + 1])[0][0])
    h.close()
