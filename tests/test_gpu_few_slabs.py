"""Few slabs on many modes: a wave that holds one mode's time line is nearly
empty there, so eigenbasis solves go level by level, with the cycle counts and
results of the coefficient iteration; and a server whose budget is too small
for the tables of cycles on chip, but not for the passes, still takes a request."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (shape, whether the solve goes level by level): two to four levels and one,
# on either side of the rule, padded and whole rows of modes
SHAPES = [
    ((3, 32, 2, 8, 2, 1), True), ((3, 40, 1, 16, 1, 2), True), ((2, 130, 2, 16, 2, 2), True), ((2, 254, 3, 4, 1, 1), True),
    ((2, 60, 2, 8, 2, 1), False), ((3, 12, 2, 8, 2, 1), False), ((2, 130, 2, 160, 2, 20), False),
    ((3, 64, 2, 2, 1, 128), True), ((2, 100, 2, 2, 1, 128), False), ((2, 258, 1, 16, 1, 128), False),
]


@pytest.mark.parametrize("shape,levels", SHAPES)
def test_route_and_result(shape, levels):
    import paper_1802_09277_amd as sth
    print(f"[gpu-few-slabs] {shape}", flush=True)
    dim, n_elem, degree, n_slabs, n_elem_t, coarse = shape
    e, s = (sth.Solver(dim, n_elem, degree, n_slabs, n_elem_t, basis=b, coarse_slabs=coarse) for b in ("eigen", "nodal"))
    f = s.load_rhs(W.random_modes(7, dim), s.new_vector())
    u, v = s.new_vector(), s.new_vector()
    e.timing(1 << 13)
    it, _, _ = e.solve(f, u, rtol=1e-8, maxit=60)
    launches = e.timing_report("eig_cycle_close")["launches"]
    e.timing(0)
    iv, _, _ = s.solve(f, v, rtol=1e-8, maxit=60)
    if e.num_levels > 1:                # one launch a cycle, or a few batches of several
        assert (launches >= it) if levels else (launches <= it // 2)
    else:
        assert (launches == 0) == levels
    assert it == iv and float((u - v).abs().max()) <= 1e-10 * float(v.abs().max())


def test_budget_without_the_tables():
    import paper_1802_09277_amd as sth
    problem = dict(dim=3, n_elem=20, degree=3, n_slabs=4, n_elem_t=2, basis="nodal", coarse_slabs=2)
    n = sth.problem_vector_len(**problem)
    with_tables = sth.workspace_bytes(**problem) + 16 * n
    u, v = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
    srv = sth.Server(with_tables, 1)
    a = srv.wait(srv.submit(W.random_modes(3, 3), u, rtol=1e-10, maxit=60, **problem))
    srv.close()
    srv = sth.Server(with_tables - 1, 1)
    b = srv.wait(srv.submit(W.random_modes(3, 3), v, rtol=1e-10, maxit=60, **problem))
    srv.close()
    torch.cuda.synchronize()
    assert a["status"] == b["status"] == 0 and a["iters"] == b["iters"]
    assert a["footprint_bytes"] == with_tables and b["footprint_bytes"] < with_tables
    assert float((u - v).abs().max()) <= 1e-10 * float(u.abs().max())
