"""FP64 per-axis transforms with the even/odd split (3-D, and 2-D beyond the
LDS-resident kernels) through the slab inverse, against the inverse formed from
the oracle's 1-D pencils with SciPy's symmetric-definite eigensolver.  The
tolerance is the repository's FP64 parity bound, 1e-10 of the largest entry."""
import numpy as np
import pytest
import scipy.linalg as sl

from oracle.spacetime import Problem, time_matrices, space_matrices_1d

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _axis(v, m):
    """m along every spatial axis of v (slab, time, ...)."""
    for a in range(2, v.ndim):
        v = np.moveaxis(np.tensordot(v, m, axes=([a], [1])), -1, a)
    return v


def _slab_inverse(prob, r):
    M, K = space_matrices_1d(prob.n_elem, prob.degree)
    mu, U = sl.eigh(K, M)
    Kt, Mt = time_matrices(0.0, prob.tau, prob.n_elem_t, prob.degree, prob.sigma)
    m = mu
    for _ in range(prob.dim - 1):
        m = np.add.outer(m, mu)
    A = Kt + m.reshape(-1)[:, None, None] * Mt
    h = _axis(r, U.T)
    s, nt = h.shape[:2]
    h = np.moveaxis(h.reshape(s, nt, -1), -1, 0)                   # mode, slab, time
    z = np.linalg.solve(A[:, None], h[..., None])[..., 0]
    return _axis(np.moveaxis(z, 0, -1).reshape(r.shape), U)


# halves below, at and above one tile of 16 columns, remainders of one column
# (33, 34, 65, 129, 130, 257, 258) and of several, odd and even n, one to five
# column tiles per panel, several panels, few and many lines
@pytest.mark.parametrize("dim,n,degree,n_slabs,n_elem_t", [
    (3, 1, 1, 2, 1), (3, 2, 2, 3, 1), (3, 3, 1, 2, 2), (3, 15, 2, 2, 1), (3, 16, 3, 1, 1), (3, 17, 2, 3, 1),
    (3, 31, 1, 2, 1), (3, 32, 2, 20, 2), (3, 33, 2, 2, 1), (3, 34, 4, 1, 1), (3, 35, 3, 1, 1), (3, 49, 2, 1, 1),
    (2, 97, 2, 3, 1), (2, 98, 4, 1, 2), (2, 112, 1, 40, 1), (2, 128, 2, 40, 1), (2, 129, 3, 2, 1), (2, 130, 4, 2, 1),
    (2, 131, 2, 1, 1), (2, 160, 2, 30, 1), (2, 161, 2, 2, 1), (2, 162, 3, 30, 1), (2, 193, 2, 2, 1),
    (2, 256, 2, 20, 1), (2, 257, 3, 20, 1), (2, 258, 4, 1, 2), (2, 300, 2, 1, 1),
])
def test_slab_inverse_and_update(dim, n, degree, n_slabs, n_elem_t):
    _check(dim, n, degree, n_slabs, n_elem_t)


# both axes of an image at once: halves below, at and above the tiles of 16
# rows and columns, odd and even n, one image to more than the card holds, odd
# counts of images
@pytest.mark.parametrize("n,degree,n_slabs,n_elem_t", [
    (1, 1, 1, 1), (2, 2, 1, 1), (3, 1, 2, 1), (4, 2, 3, 2), (15, 2, 2, 1), (16, 2, 16, 2), (17, 3, 1, 2), (20, 2, 700, 1),
    (29, 1, 3, 2), (31, 2, 1, 1), (32, 2, 9, 1), (33, 3, 5, 1), (34, 4, 1, 2), (35, 2, 3, 1), (36, 1, 2, 2), (40, 2, 24, 2),
    (47, 1, 3, 1), (61, 3, 7, 2), (62, 4, 2, 1), (63, 2, 3, 1), (64, 2, 300, 1), (65, 3, 260, 2), (66, 4, 3, 1), (67, 2, 1, 1),
    (79, 1, 3, 2), (80, 2, 2, 1), (81, 3, 1, 1), (94, 2, 2, 1), (95, 1, 2, 1), (96, 2, 130, 1),
])
def test_slab_inverse_and_update_images(n, degree, n_slabs, n_elem_t):
    _check(2, n, degree, n_slabs, n_elem_t)


def _check(dim, n, degree, n_slabs, n_elem_t):
    import paper_1802_09277_amd as sth
    prob = Problem(dim, n + 2 - degree, degree, n_slabs, n_elem_t)
    assert prob.n == n
    shape = (n_slabs, prob.N_t) + (n,) * dim
    r = np.random.default_rng(n).standard_normal(shape)
    want = _slab_inverse(prob, r)
    s = sth.Solver(dim, prob.n_elem, degree, n_slabs, n_elem_t)
    rd = torch.from_numpy(r).reshape(-1).cuda()
    z = s.block_solve(rd, s.new_vector())
    err = np.abs(z.cpu().numpy().reshape(shape) - want).max() / np.abs(want).max()
    # the update epilogue: one damped step from u = 0 leaves omega A^{-1} f, a
    # second from there adds omega A^{-1} (f - L u)
    u = s.smooth(rd, s.new_vector(), steps=1)
    erru = np.abs(u.cpu().numpy().reshape(shape) - 0.5 * want).max() / np.abs(want).max()
    res = s.residual(rd, u, s.new_vector())
    step = _slab_inverse(prob, res.cpu().numpy().reshape(shape))
    u2 = s.smooth(rd, u.clone(), steps=1)
    want2 = u.cpu().numpy().reshape(shape) + 0.5 * step
    err2 = np.abs(u2.cpu().numpy().reshape(shape) - want2).max() / np.abs(want2).max()
    print(f"  dim={dim} n={n}: slab inverse {err:.1e}, from zero {erru:.1e}, update {err2:.1e}")
    assert err <= 1e-10 and erru <= 1e-10 and err2 <= 1e-10
    s.close()


@pytest.mark.parametrize("n_elem,degree", [(6, 2), (9, 2), (32, 3), (5, 4), (2, 1), (3, 1)])
def test_modes_even_then_odd(n_elem, degree):
    """ceil(n/2) even modes, then n/2 odd ones, for odd n as well."""
    import paper_1802_09277_amd as sth
    F = sth.host_factors(level=0, dim=2, n_elem=n_elem, degree=degree, n_slabs=2, n_elem_t=1)
    U, h = F["U"], (len(F["mu"]) + 1) // 2
    tol = 1e-13 * np.abs(U).max()
    assert np.abs(U[::-1, :h] - U[:, :h]).max() <= tol
    assert U.shape[1] == h or np.abs(U[::-1, h:] + U[:, h:]).max() <= tol
