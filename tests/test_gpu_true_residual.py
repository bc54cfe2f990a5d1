"""A solve that reports convergence leaves a vector whose own residual, formed
from it, meets the tolerance: from guesses far larger than the solution, and
for smooth loads, whose solutions are the largest for their size, at small
tolerances (SHAPES' meshes: rounding of the coefficients leaves 2e-13 to 6e-12
there, so the eigenbasis iteration, which stops on its own iterate, is asked
for 1e-10 and the coefficient iteration for 1e-12)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# four, three and one levels; odd n; per-axis transforms and whole images; 3-D
SHAPES = [(2, 128, 2, 64, 1, 8), (2, 60, 3, 48, 2, 12), (2, 126, 2, 16, 1, 16), (2, 99, 1, 24, 1, 3), (3, 16, 2, 32, 2, 8)]
FINE = [(2, 250, 1, 64, 1, 16), (2, 256, 2, 32, 1, 8), (2, 256, 4, 16, 2, 4), (3, 24, 2, 16, 1, 4)]


def _solver(shape, basis):
    import paper_1802_09277_amd as sth
    dim, n_elem, degree, n_slabs, n_elem_t, coarse = shape
    return sth.Solver(dim, n_elem, degree, n_slabs, n_elem_t, basis=basis, coarse_slabs=coarse)


def _relres(s, f, u):
    return float(s.residual(f, u, s.new_vector()).norm() / f.norm())


@pytest.mark.parametrize("basis", ["eigen", "nodal"])
@pytest.mark.parametrize("shape", SHAPES)
def test_from_a_large_guess(shape, basis):
    print(f"[gpu-true-residual] guess {shape} {basis}", flush=True)
    s = _solver(shape, basis)
    f = s.load_rhs(W.manufactured_modes(s.dim), s.new_vector())
    g = torch.from_numpy(np.random.default_rng(1).standard_normal(s.vector_len)).cuda()
    for scale in (1.0, 100.0):
        for rtol in (1e-8, 1e-10):
            u = g * scale
            it, rr, code = s.solve(f, u, rtol=rtol, maxit=80, check=False)
            true = _relres(s, f, u)
            print(f"  scale {scale} rtol {rtol}: {it} cycles, reported {rr:.2e}, true {true:.2e}")
            assert code == 0 and true <= rtol
    # a guess that meets the tolerance stays as it is
    v = u.clone()
    it, _, _ = s.solve(f, v, rtol=1e-9, maxit=80)
    assert it == 0 and torch.equal(u, v)


@pytest.mark.parametrize("basis,rtols", [("eigen", (1e-8, 1e-10)), ("nodal", (1e-8, 1e-10, 1e-12))])
@pytest.mark.parametrize("shape", FINE)
def test_smooth_load(shape, basis, rtols):
    print(f"[gpu-true-residual] load {shape} {basis}", flush=True)
    s = _solver(shape, basis)
    f = s.load_rhs(W.manufactured_modes(s.dim), s.new_vector())
    for rtol in rtols:
        u = s.new_vector()
        it, rr, code = s.solve(f, u, rtol=rtol, maxit=80, check=False)
        true = _relres(s, f, u)
        print(f"  rtol {rtol}: {it} cycles, reported {rr:.2e}, true {true:.2e}")
        assert code == 0 and true <= rtol
        if basis == "nodal":                # (exact norms are reported)
            assert abs(rr - true) <= 1e-2 * true


def test_rough_load_in_batches():
    """Quartic splines and a rough right-hand side: the mode-weighted bound of
    the residual norm is negative, the eigenvalues of M_1 bound it, and a solve
    takes a few batches with an exact norm near the end instead of one batch and
    one exact norm for every cycle."""
    s = _solver((2, 20, 4, 64, 1, 16), "nodal")
    f = torch.from_numpy(np.random.default_rng(2).standard_normal(s.vector_len)).cuda()
    u = s.new_vector()
    s.solve(f, u, rtol=1e-8)
    s.timing(1 << 11 | 1 << 13)
    it, _, _ = s.solve(f, u.zero_(), rtol=1e-8)
    batches = s.timing_report("eig_cycle_close")["launches"]
    norms = s.timing_report("resnorm")["launches"]
    s.timing(0)
    print(f"  {it} cycles, {batches} batches, {norms} exact norms")
    assert it >= 9 and norms <= 5 and batches <= 8
