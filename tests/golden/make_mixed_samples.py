"""Writes sampled results of the library's own reduced-precision forms (needs a
GPU), for a test that they stay what they are.

    python tests/golden/make_mixed_samples.py

The mixed-precision solves end with the noise of their reduced-precision
transforms still in u, at the size of the tolerance (BF16x3: 1e-9 to 1e-8 of
the solution), so a change of the order of a transform, of the eigenvectors or
of the place where a vector is rounded moves a result by more than the FP64
kernels' 1e-10, though it is as accurate as before.  The file holds, for each
configuration below, the cycle count, the largest entry and 64 entries of the
solution (or of the slab inverse of the load vector), relative tolerance 1e-8,
random modes seed 5.  Written at commit e676eeb.
"""
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
PATH = os.path.join(HERE, "mixed_samples.txt")

# (call, dim, n_elem, degree, n_slabs, n_elem_t, coarse_slabs, precision)
CONFIGS = [
    # one axis at a time, widths padded to 112, 144 and 208
    ("solve", 2, 110, 2, 16, 1, 4, "bf16x3"), ("solve", 2, 143, 3, 8, 1, 2, "bf16x3"),
    ("solve", 2, 208, 2, 4, 1, 2, "bf16x3"),
    # odd numbers of functions per axis
    ("solve", 2, 107, 2, 8, 2, 128, "fp32"), ("solve", 2, 128, 3, 24, 1, 6, "bf16x3"),
    ("solve", 2, 125, 2, 16, 2, 128, "bf16x3"), ("solve", 2, 12, 3, 10, 2, 128, "bf16x3"),
    ("solve", 2, 21, 2, 24, 1, 128, "bf16x3"), ("solve", 3, 16, 3, 8, 2, 128, "bf16x3"),
    ("solve", 3, 18, 3, 16, 3, 4, "fp32"), ("block_solve", 2, 36, 1, 6, 2, 128, "bf16x3"),
    ("block_solve", 3, 9, 2, 4, 1, 128, "fp32"),
    # float eigenbasis vectors
    ("solve", 3, 16, 3, 8, 2, 4, "bf16x3"), ("solve", 2, 116, 4, 8, 1, 4, "bf16x3"),
    ("solve", 2, 90, 4, 8, 1, 4, "bf16x3"), ("solve", 2, 25, 3, 8, 2, 4, "bf16x3"),
    ("solve", 2, 92, 2, 160, 1, 40, "bf16x3"), ("solve", 3, 16, 2, 16, 2, 4, "bf16x3"),
    ("solve", 2, 128, 2, 64, 1, 16, "bf16x3"), ("solve", 3, 16, 2, 16, 2, 4, "fp32"),
    ("solve", 2, 64, 2, 64, 1, 16, "fp32"), ("solve", 2, 62, 4, 64, 1, 16, "fp32"),
    ("solve", 3, 27, 3, 24, 2, 4, "fp32"), ("solve", 2, 31, 3, 64, 2, 16, "fp32"),
]


def result(config):
    """The cycle count (0 for a slab inverse) and the whole result."""
    import paper_1802_09277_amd as sth
    import workloads as W
    call, dim, n_elem, degree, n_slabs, n_elem_t, coarse, prec = config
    basis = "eigen" if call == "solve" else "nodal"
    s = sth.Solver(dim, n_elem, degree, n_slabs, n_elem_t, prec=prec, basis=basis, coarse_slabs=coarse)
    f, u, it = s.load_rhs(W.random_modes(5, dim), s.new_vector()), s.new_vector(), 0
    if call == "solve":
        it, _, code = s.solve(f, u, rtol=1e-8, maxit=100, check=False)
        assert code == 0
    else:
        s.block_solve(f, u)
    u = u.cpu().numpy()
    s.close()
    return it, u


def places(n):
    return np.random.default_rng(n).integers(0, n, 64)


def read():
    with open(PATH) as fh:
        rows = [ln.split() for ln in fh if not ln.startswith("#")]
    return {int(r[0]): (int(r[1]), float(r[2]), np.array(r[3:], dtype=np.float64)) for r in rows}


def main():
    with open(PATH, "w") as fh:
        fh.write("# results of the reduced-precision forms, written by make_mixed_samples.py at commit e676eeb\n")
        fh.write("# columns: index of the configuration, cycles, largest entry, 64 entries\n")
        for i, c in enumerate(CONFIGS):
            print(i, c, flush=True)
            it, u = result(c)
            fh.write(f"{i} {it} {np.abs(u).max():.17e} " + " ".join(f"{v:.17e}" for v in u[places(u.size)]) + "\n")


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    main()
