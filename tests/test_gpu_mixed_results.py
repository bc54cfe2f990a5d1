"""The reduced-precision forms against their own earlier results (sampled in
golden/mixed_samples.txt): same cycle counts, and the repository's FP64 parity
bound, 1e-10 of the largest entry, because every operation in which the noise
of the reduced-precision transforms arises is unchanged and the others are FP64."""
import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden"))
import make_mixed_samples as G  # noqa: E402


@pytest.mark.parametrize("i", range(len(G.CONFIGS)))
def test_results_are_kept(i):
    print(f"[gpu-mixed-results] {G.CONFIGS[i]}", flush=True)
    cycles, largest, want = G.read()[i]
    it, u = G.result(G.CONFIGS[i])
    err = np.abs(u[G.places(u.size)] - want).max() / largest
    print(f"  {it} cycles, error {err:.1e}")
    assert it == cycles and err <= 1e-10
