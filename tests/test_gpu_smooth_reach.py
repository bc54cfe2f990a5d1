"""Several smoothing steps at once are local in time: infinities and NaN of the
right-hand side or the iterate reach the slabs that the same steps reach one by
one, and the slabs before and beyond keep their values."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one slab to a lane, more than one, the line not filling its lanes; N_t 2..6
@pytest.mark.parametrize("shape", [(2, 9, 1, 40, 1), (2, 6, 2, 64, 1), (2, 12, 2, 150, 2), (3, 5, 3, 300, 2), (2, 5, 4, 70, 2)])
def test_reach_of_a_nan(shape):
    import paper_1802_09277_amd as sth
    print(f"[gpu-smooth-reach] {shape}", flush=True)
    s = sth.Solver(*shape)
    rng = np.random.default_rng(3)
    slab = s.vector_len // shape[3]
    for where in ("f", "u"):
        for at, bad in ((0, np.nan), (7, np.inf), (shape[3] - 1, np.nan), (shape[3] // 2, -np.inf)):
            f, u = rng.standard_normal(s.vector_len), rng.standard_normal(s.vector_len)
            (f if where == "f" else u)[at * slab + 3] = bad
            f, u = torch.from_numpy(f).cuda(), torch.from_numpy(u).cuda()
            for steps in (2, 3, 5):
                one, many = u.clone(), u.clone()
                for _ in range(steps):
                    s.smooth(f, one, steps=1)
                s.smooth(f, many, steps=steps)
                a, b = one.cpu().numpy(), many.cpu().numpy()
                assert np.array_equal(np.isfinite(a), np.isfinite(b))
                ok = np.isfinite(a)
                assert np.abs(a[ok] - b[ok]).max() <= 1e-11 * np.abs(a[ok]).max()
