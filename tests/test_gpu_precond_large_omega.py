"""Mixed-precision preconditioned solves that converge in a few iterations
(frequencies far above the potential), where a solve reaches the FP32 rounding
of its solution between two looks at the true residual."""
import math

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


@pytest.mark.parametrize("tol", [1e-6, 1e-8, 1e-10, 1e-12])
@pytest.mark.parametrize("omega", [20.0, 49.36, 107.0, 400.0])
@pytest.mark.parametrize("n,n_occ", [((7, 8, 9), 2), ((17, 16, 15), 3), ((14, 24, 24), 4)])
def test_fast_preconditioned_solves_converge_in_fp32(P, n, n_occ, omega, tol):
    rng = np.random.default_rng(sum(n))
    N = int(np.prod(n))
    L = tuple(0.45 * v for v in n)
    v = sc.gaussian_vloc(n, L, rng.uniform(0, 1, (3, 3)) * np.array(L))
    psi = np.linalg.qr(rng.standard_normal((N, n_occ)))[0].T / math.sqrt(0.45 ** 3)
    eps = np.linspace(-0.9, -0.3, n_occ)
    u = rng.standard_normal((8, N))
    h = P.Handle(n, L, v, psi, eps, precision="fp32_refine", stern_tol=tol, precond=True)
    x, st = h.sternheimer_solve(omega, torch.from_numpy(u))
    h.close()
    assert st["n_noconv"] == 0 and st["n_breakdown"] == 0 and st["n_fp64_fallback"] == 0
    # A M^-1 = 1 + D M^-1 with D the diagonal V - eps - Re sigma and |M| >= omega: each
    # iteration reduces the residual by q at least.  Each of the at most four stretches
    # between true residuals (FP32 carries a stretch by 6 digits or so, a stretch has
    # at least four iterations) may lose what it gained beyond that
    re = np.maximum(v.mean() - eps, 0.25)
    q = max(np.abs(v - e - s).max() for e, s in zip(eps, re)) / omega
    assert st["cocg_iters_max"] <= 4 * max(4, math.ceil(math.log(tol) / math.log(min(q, 0.5))))
    ham = O.Hamiltonian(n, L, v)
    x = x.cpu().numpy()
    for b in range(u.shape[0]):
        for k in range(n_occ):
            rhs = -psi[k] * u[b]
            r = rhs - (ham.apply(x[b, k]) - (eps[k] + 1j * omega) * x[b, k])
            assert np.linalg.norm(r) <= 1.01 * tol * np.linalg.norm(rhs), (b, k)
