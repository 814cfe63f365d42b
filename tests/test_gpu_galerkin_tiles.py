"""The Galerkin guess at the edges of its tiles and chunks.  On a free cell
(V = 0) the real Fourier modes are exact eigenvectors, and a smooth u keeps
psi_n u inside the span of the given modes: the guess then solves every
Sternheimer system and COCG takes no iteration."""
import numpy as np
import pytest

import synthcell as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_2609_16408_amd as P
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    P.lib()
    return P


def _modes(n, L, count):
    """The `count` lowest real eigenvectors of -1/2 Lap_h (unit norm) and their energies."""
    ax, en = [], []
    for d in range(3):
        i = np.arange(n[d])
        one = [0] * 3
        V = [np.ones(n[d])]
        k = [0]
        for m in range(1, n[d] // 2 + 1):
            V.append(np.cos(2 * np.pi * m * i / n[d]))
            k.append(m)
            if 2 * m < n[d]:
                V.append(np.sin(2 * np.pi * m * i / n[d]))
                k.append(m)
        ax.append(np.array([v / np.linalg.norm(v) for v in V]))
        sym = sc.kinetic_symbol(n, L)
        e = []
        for m in k:
            one = [0, 0, 0]
            one[d] = m
            e.append(sym[tuple(one)])
        en.append(np.array(e))
    E = en[0][:, None, None] + en[1][None, :, None] + en[2][None, None, :]
    low = np.argsort(E, axis=None, kind="stable")[:count]
    a, b, c = np.unravel_index(low, E.shape)
    psi = np.einsum("si,sj,sk->sijk", ax[0][a], ax[1][b], ax[2][c]).reshape(count, -1)
    return psi, E.reshape(-1)[low]


@pytest.mark.parametrize("n,n_occ,n_extra,smooth", [((7, 8, 9), 17, 486, True), ((7, 8, 9), 33, 470, True),
                                                    ((9, 8, 10), 16, 700, True), ((12, 12, 14), 1, 0, False),
                                                    ((12, 13, 14), 17, 16, False), ((7, 7, 7), 2, 13, False),
                                                    ((11, 12, 13), 48, 65, False)])
def test_guess_solves_systems_inside_its_span(P, n, n_occ, n_extra, smooth):
    L = tuple(0.5 * v for v in n)
    dV = 0.5 ** 3
    N = int(np.prod(n))
    psi, eps = _modes(n, L, n_occ + n_extra)
    psi = psi / np.sqrt(dV)
    omega = 0.7
    extra = (psi[n_occ:], eps[n_occ:]) if n_extra else None
    h = P.Handle(n, L, np.zeros(N), psi[:n_occ], eps[:n_occ], stern_tol=1e-8, extra=extra)
    u = np.ones((2, N))
    if smooth:
        g = np.meshgrid(*[np.arange(v) / v for v in n], indexing="ij")
        u[0] += 0.5 * np.cos(2 * np.pi * g[0]).reshape(-1) - 0.3 * np.sin(2 * np.pi * g[2]).reshape(-1)
        u[1] = np.cos(2 * np.pi * (g[1] + 0.1)).reshape(-1)
    x, st = h.sternheimer_solve(omega, torch.from_numpy(u))
    h.close()
    assert st["cocg_iters_total"] == 0 and st["n_noconv"] == 0
    x = x.cpu().numpy()
    for v in range(2):
        for k in range(n_occ):
            c = dV * psi @ (-psi[k] * u[v])
            ref = (c / (eps - eps[k] - 1j * omega)) @ psi
            # two contractions, over N points and over the states
            tol = 4 * (N + n_occ + n_extra) * 2.0 ** -53 / omega
            assert np.linalg.norm(x[v, k] - ref) <= tol * np.linalg.norm(psi[k] * u[v]) * np.sqrt(n_occ + n_extra), (v, k)
