"""Fused separable transforms at the edges of their tiles and of their range
(dimensions 16 / 17, 80 / 81 and 128, one past it on the per-axis kernels),
with one and with two planes per workgroup."""
import ctypes

import numpy as np
import pytest

import synthcell as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def P():
    import paper_2609_16408_amd as P
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    P.lib()
    return P


@pytest.mark.parametrize("n,nvec", [((16, 17, 128), 1), ((7, 80, 81), 3), ((33, 80, 80), 32), ((128, 9, 15), 2),
                                    ((24, 16, 48), 43), ((129, 8, 9), 1), ((8, 129, 7), 2), ((9, 7, 130), 1)])
def test_kinetic_plan_matches_the_fft(P, n, nvec):
    L = tuple(0.43 * v for v in n)
    N = int(np.prod(n))
    rng = np.random.default_rng(sum(n) + nvec)
    x = rng.standard_normal((nvec, 2, N))
    sig = 0.3 + 0.05 * np.arange(nvec) - 1j * (0.02 + 0.3 * np.arange(nvec))
    f = np.fft.fftn((x[:, 0] + 1j * x[:, 1]).reshape(nvec, *n), axes=(1, 2, 3))
    ref = np.fft.ifftn(f / (sc.kinetic_symbol(n, L) + sig[:, None, None, None]), axes=(1, 2, 3)).reshape(nvec, N)
    plan = ctypes.c_void_p()
    nn, LL = np.array(n, dtype=np.int32), np.array(L)
    sr, si = np.ascontiguousarray(sig.real), np.ascontiguousarray(sig.imag)
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    lib = P.lib()
    assert lib.rpa_kinetic_precond_create(nn.ctypes.data, LL.ctypes.data, s, ctypes.byref(plan)) == P.RPA_OK
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty_like(xd)
    assert lib.rpa_kinetic_precond_apply(plan, nvec, sr.ctypes.data, si.ctypes.data, ctypes.c_void_p(xd.data_ptr()),
                                         ctypes.c_void_p(yd.data_ptr()), s) == P.RPA_OK
    y = yd.cpu().numpy()
    lib.rpa_kinetic_precond_destroy(plan)
    y = y[:, 0] + 1j * y[:, 1]
    # six orthogonal contractions of length n_d, each within n_d eps of the
    # vector's norm, before a diagonal of norm 1 / Re(sigma) <= 1 / 0.3; basis and
    # symbol entries carry a few eps of their own
    tol = 6 * (max(n) + 8) * EPS / 0.3
    for b in range(nvec):
        assert np.linalg.norm(y[b] - ref[b]) <= tol * np.linalg.norm(x[b]), (n, b)


@pytest.mark.parametrize("kind", ["trilinear", "tricubic", "fourier"])
@pytest.mark.parametrize("n,g,n_omega", [((8, 12, 10), 2, 1), ((34, 36, 32), 2, 64), ((34, 36, 32), 2, 65),
                                         ((72, 18, 33), 3, 8)])
def test_energy_sums_the_interpolated_fields(P, kind, n, g, n_omega):
    N = int(np.prod(n))
    rng = np.random.default_rng(N + n_omega)
    h = P.Handle(n, tuple(0.43 * v for v in n), np.zeros(N), rng.standard_normal((1, N)), np.array([-0.5]))
    w = rng.uniform(0.1, 3.0, n_omega)
    c = torch.from_numpy(rng.standard_normal((n_omega, N // g ** 3))).cuda()
    fine = h.interpolate(kind, g, c).cpu().numpy()
    e_c, e_fine = h.energy_from_coarse(w, g, kind, c)
    ref = w @ fine
    dV = 0.43 ** 3
    # at most n_omega + 2 max(n) / g + 2 rounded terms on either side; the
    # interpolants' per-axis row sums of |weights| stay below 4
    bound = 2 * (n_omega + 2 * max(n) / g + 8) * EPS * 4 ** 3 * (np.abs(w) @ np.abs(c.cpu().numpy()).max(axis=1))
    assert np.abs(e_fine.cpu().numpy() * 2 * np.pi * dV - ref).max() <= bound
    assert abs(e_c * 2 * np.pi - ref.sum()) <= N * bound
    e_c2, none = h.energy_from_coarse(w, g, kind, c, want_fine=False)
    assert none is None and e_c2 == e_c
    h.close()
