"""Graph replay and speculation of cycles taken one by one: the routes that
batches of cycles do not take (five levels, N_t = 7, tolerances below 1e-12,
reduced precision with float vectors) and the coefficient iteration's single
cycles.  Replays, with eager work between them, and eager launches, speculative
or not, give the same bits."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {
    "five_levels": (dict(dim=2, n_elem=12, degree=2, n_slabs=64, n_elem_t=1, coarse_slabs=4, basis="eigen"), 1e-9),
    "five_levels_3d": (dict(dim=3, n_elem=6, degree=2, n_slabs=32, n_elem_t=2, coarse_slabs=2, basis="eigen"), 1e-9),
    "nt7": (dict(dim=2, n_elem=16, degree=3, n_slabs=16, n_elem_t=4, coarse_slabs=4, basis="eigen"), 1e-9),
    "small_rtol": (dict(dim=2, n_elem=20, degree=2, n_slabs=32, n_elem_t=1, coarse_slabs=8, basis="eigen"), 1e-13),
    "per_axis": (dict(dim=2, n_elem=99, degree=2, n_slabs=64, n_elem_t=1, coarse_slabs=4, basis="eigen"), 1e-9),
    "bf16x3": (dict(dim=2, n_elem=20, degree=2, n_slabs=32, n_elem_t=1, coarse_slabs=8, basis="eigen", prec="bf16x3"), 1e-8),
    "fp32_cubic": (dict(dim=2, n_elem=20, degree=3, n_slabs=32, n_elem_t=2, coarse_slabs=8, basis="eigen", prec="fp32"), 1e-8),
    "coefficients": (dict(dim=2, n_elem=20, degree=2, n_slabs=32, n_elem_t=1, coarse_slabs=8), 1e-13),
    "coefficients_five": (dict(dim=2, n_elem=12, degree=2, n_slabs=64, n_elem_t=1, coarse_slabs=4), 1e-9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_replay_and_speculation(name):
    import paper_1802_09277_amd as sth
    shape, rtol = CASES[name]
    print(f"[gpu-replay] {name} {shape}", flush=True)
    s = sth.Solver(**shape)
    f = s.load_rhs(W.random_modes(8, s.dim), s.new_vector())
    g = s.load_rhs(W.random_modes(9, s.dim), s.new_vector())
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    u, want = s.new_vector(), {}
    for spec, graphs in ((False, False), (True, False), (True, True), (True, True), (False, True), (False, True), (True, True)):
        s.speculate(spec)
        s.use_graphs(graphs)
        for rhs in (0, 1):
            with torch.cuda.stream(stream):
                out = s.solve((f, g)[rhs], u.zero_(), rtol=rtol, maxit=24, stream=stream, check=False)
                got = (out, u.clone())
                # eager work and a synchronization between the replays
                s.residual(f, u, s.new_vector(), stream=stream)
            stream.synchronize()
            first = want.setdefault(rhs, got)
            assert got[0] == first[0] and torch.equal(got[1], first[1])
        # a residual of another vector, on the default stream
        torch.cuda.synchronize()
    s.speculate(True)
    s.use_graphs(False)
    assert want[0][0][0] >= 8
    if rtol >= 1e-9:
        r = s.residual(f, want[0][1], s.new_vector())
        assert float(r.norm() / f.norm()) <= rtol * (1 + 1e-6)


def test_served_replays():
    """The same through the serving loop, setups that replay and setups that do not."""
    import paper_1802_09277_amd as sth
    results = {}
    for graphs in (False, True):
        srv = sth.Server(8 << 30, 3)
        srv.use_graphs(graphs)
        for turn in range(3):
            outs, tickets = [], []
            for name, (shape, rtol) in CASES.items():
                n = sth.problem_vector_len(**{k: v for k, v in shape.items() if k not in ("basis", "coarse_slabs", "prec")})
                u = torch.zeros(n, dtype=torch.float64, device="cuda")
                outs.append(u)
                tickets.append(srv.submit(W.random_modes(8, shape["dim"]), u, rtol=max(rtol, 1e-11), maxit=40, **shape))
            stats = [srv.wait(t) for t in tickets]
            torch.cuda.synchronize()
            for name, u, st in zip(CASES, outs, stats):
                first = results.setdefault(name, (st["iters"], u))
                assert st["status"] == 0 and st["iters"] == first[0] and torch.equal(u, first[1])
        srv.close()
