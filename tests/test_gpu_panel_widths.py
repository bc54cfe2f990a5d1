"""Reduced-precision per-axis transforms whose matrix is cut into 3, 5 or 7
panels (padded widths 96 in 3-D, 160, 192 and 224): every tile of the data goes
through every panel once.  Slab inverses against the FP64 one, to the bounds of
the other reduced-precision slab inverses; solves end at their tolerance, and
both give the same bits again."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# few tiles and more than one for each wave of the card, full and ragged widths
SHAPES = [
    (2, 160, 2, 1, 1), (2, 150, 2, 40, 1), (2, 192, 2, 3, 1), (2, 181, 1, 100, 1), (2, 224, 2, 2, 1), (2, 210, 3, 30, 1),
    (3, 96, 2, 1, 1), (3, 90, 1, 3, 1), (3, 160, 1, 1, 1), (3, 192, 1, 1, 1),
]


@pytest.mark.parametrize("prec,bound", [("fp32", 1e-4), ("bf16x3", 1e-3)])
@pytest.mark.parametrize("shape", SHAPES)
def test_slab_inverse(shape, prec, bound):
    import paper_1802_09277_amd as sth
    print(f"[gpu-panel-widths] {shape} {prec}", flush=True)
    a, b = sth.Solver(*shape), sth.Solver(*shape, prec=prec)
    r = torch.from_numpy(np.random.default_rng(1).standard_normal(a.vector_len)).cuda()
    want, z, again = a.new_vector(), b.new_vector(), b.new_vector()
    a.block_solve(r, want)
    # the work vectors hold the results of other data first
    b.block_solve(r * 3.0 + 1.0, z)
    b.block_solve(r, z)
    err = float((z - want).abs().max() / want.abs().max())
    b.block_solve(r * -2.0, again)
    b.block_solve(r, again)
    print(f"  error {err:.1e}")
    assert err < bound and torch.equal(z, again)


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("shape", [(2, 160, 2, 16, 1), (2, 190, 2, 8, 1), (2, 222, 2, 8, 1), (3, 90, 1, 4, 1)])
def test_solve(shape, prec):
    import paper_1802_09277_amd as sth
    print(f"[gpu-panel-widths] solve {shape} {prec}", flush=True)
    s = sth.Solver(*shape, prec=prec, basis="eigen", coarse_slabs=2)
    f, u, v = s.load_rhs(W.random_modes(5, shape[0]), s.new_vector()), s.new_vector(), s.new_vector()
    it, _, _ = s.solve(f, u, rtol=1e-8, maxit=60)
    again, _, _ = s.solve(f, v, rtol=1e-8, maxit=60)
    res = s.residual(f, u, s.new_vector())
    assert float(res.norm() / f.norm()) <= 1e-8 * (1.0 + 1e-6)
    assert it == again and torch.equal(u, v)
