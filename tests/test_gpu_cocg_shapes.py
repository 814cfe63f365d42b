"""The Sternheimer solvers on grids at the edges of their LDS pitches, tile
modes and rounds of planes, plain and preconditioned, with and without
nonlocal projectors."""
import numpy as np
import pytest

import oracle as O
import synthcell as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_2609_16408_amd as P
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    P.lib()
    return P


def _check(P, n, precision, precond, atoms=0, n_occ=2):
    """chi0 against the oracle: every orbital's solution is within
    (tol_gpu + tol_oracle) ||b|| / omega of the oracle's (the operator is normal
    with its spectrum at least omega away from zero), so chi0 u is within
    4 sum_n ||psi_n||_inf of that."""
    rng = np.random.default_rng(sum(n) + atoms)
    L = tuple(0.45 * v for v in n)
    N = int(np.prod(n))
    dV = 0.45 ** 3
    pos = rng.uniform(0, 1, (max(1, atoms), 3)) * np.array(L)
    v = sc.gaussian_vloc(n, L, pos)
    psi = np.linalg.qr(rng.standard_normal((N, n_occ)))[0].T / np.sqrt(dV)
    eps = np.array([-0.9, -0.4])[:n_occ]
    proj = sc.projector_balls(n, L, pos, seed=7, rc=1.3) if atoms else None
    tol = 1e-10 if precision == "fp64" else 1e-8
    omega = 0.4
    h = P.Handle(n, L, v, psi, eps, precision=precision, stern_tol=tol, precond=precond, proj=proj)
    u = rng.standard_normal((3, N))
    y, st = h.chi0_apply(omega, torch.from_numpy(u))
    assert st["n_noconv"] == 0 and st["n_breakdown"] == 0
    x, _ = h.sternheimer_solve(omega, torch.from_numpy(u[:1]))
    h.close()
    ham = O.Hamiltonian(n, L, v, proj=proj)
    for k in range(n_occ):
        xk = x[0, k].cpu().numpy()
        b = -psi[k] * u[0]
        r = np.linalg.norm(b - (ham.apply(xk) - (eps[k] + 1j * omega) * xk))
        assert r <= 1.01 * tol * np.linalg.norm(b), (n, k, r / np.linalg.norm(b))
    for b in range(3):
        ref = O.chi0_apply(ham, psi, eps, u[b], omega, tol=1e-11)
        bound = 4 * sum(np.abs(psi[k]).max() * (tol + 1e-11) * np.linalg.norm(psi[k] * u[b]) / omega for k in range(n_occ))
        assert np.abs(y[b].cpu().numpy() - ref).max() <= bound, n


# pitches 56 / 64 / 128 change after n_z = 44 and 52; whole planes, one and two
# halo slots per thread; x lengths on either side of the unrolled march
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("n", [(9, 7, 44), (14, 8, 45), (13, 7, 52), (7, 12, 53), (8, 24, 45), (7, 14, 60), (17, 24, 33),
                               (16, 9, 7)])
def test_plain_solver_shapes(P, n, precision):
    _check(P, n, precision, False)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("n", [(7, 8, 9), (17, 16, 15), (33, 17, 16), (16, 33, 20), (48, 18, 33), (15, 7, 49)])
def test_preconditioned_solver_shapes(P, n, precision):
    _check(P, n, precision, True)


@pytest.mark.parametrize("precond", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("n", [(12, 17, 14), (9, 24, 46)])
def test_solvers_with_projectors(P, n, precision, precond):
    _check(P, n, precision, precond, atoms=3)
