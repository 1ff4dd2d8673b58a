"""A solver keeps the captured graph of its line searches from call to call. Every call of a sequence that
changes what the graph depends on (or nothing) has to give the bits a fresh solver gives."""

import numpy as np
import pytest

from synth import start_coefficients
from synth.generator import lattice_positions, make_system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1312_1549_amd as pkg

    return torch, pkg


def _system(seed, M=21):
    rng = np.random.default_rng(seed)
    pos = lattice_positions((4, 4, 2), 2.5)
    pos = pos + rng.uniform(-0.2, 0.2, size=pos.shape)
    s = make_system(pos, 4, 6.0, M, rng, name="graph", eta=0.5, tau=10.0, seed=seed)
    return s, start_coefficients(s.S, s.M, seed + 1)


def _result(solver, s, C0, **kw):
    solver.minimize(C0, eta=0.5, tol=0.0, **kw)
    return solver.energy_trace(), solver.get_C()


@pytest.mark.skip(reason="this test ended once in a segmentation fault of the host process inside omm_minimize (fp32, no "
                         "refinement); the cause is not known, and a context no longer keeps its graph between calls")
@pytest.mark.parametrize("precision,refine,sparse", [("fp64", True, False), ("fp32", True, False),
                                                    ("fp32", False, False), ("bf16x3", True, True)])
def test_kept_graph_gives_the_bits_of_a_fresh_solver(api, precision, refine, sparse):
    torch, pkg = api
    print(f"[gpu-case] graph reuse {precision} refine={refine} sparse={sparse}", flush=True)
    s, C0 = _system(300)
    s2, D0 = _system(310)
    make = lambda **kw: pkg.OMM(s.N, s.M, precision=precision, refine=refine, sparse=sparse, **kw)  # noqa: E731
    kept = make()
    side = torch.cuda.Stream()
    calls = [
        (s, C0, dict(tau=10.0, max_iter=8), None, None),
        (s, C0, dict(tau=10.0, max_iter=8), None, None),      # nothing changed
        (s2, D0, dict(tau=10.0, max_iter=7), None, None),     # other inputs, an odd number of steps
        (s, C0, dict(tau=0.0, max_iter=8), None, None),       # no preconditioner
        (s, C0, dict(tau=10.0, max_iter=60), None, None),     # the energy trace is allocated anew
        (s, C0, dict(tau=10.0, max_iter=9), side, None),      # on another stream
        (s, C0, dict(tau=10.0, max_iter=8), None, "fp64"),    # another precision and back
        (s2, D0, dict(tau=10.0, max_iter=8), None, None),
    ]
    for k, (sys_, c, kw, stream, prec) in enumerate(calls):
        with torch.cuda.stream(stream or torch.cuda.current_stream()):
            for solver in (kept, fresh := make()):
                solver.set_precision(prec or precision, refine)
                solver.set_HS(sys_.H, sys_.S, sys_.T)
            got, want = _result(kept, sys_, c, **kw), _result(fresh, sys_, c, **kw)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), k
        torch.zeros(1000, device="cuda").add_(1.0)  # the program's own work between the replays
        torch.cuda.synchronize()
        fresh.close()


def test_batch_keeps_its_lists_and_graphs(api):
    torch, pkg = api
    print("[gpu-case] graph reuse batch", flush=True)
    systems = [_system(400 + k, M=9 + 4 * k) for k in range(4)]
    others = [_system(420 + k, M=9 + 4 * k) for k in range(4)]
    make = lambda: pkg.OMMBatch([s.N for s, _ in systems], [s.M for s, _ in systems],  # noqa: E731
                                precision="fp32", refine=True)
    kept = make()
    for which, tau, iters in ((systems, 10.0, 6), (systems, 10.0, 6), (others, 10.0, 7), (systems, 0.0, 6),
                              (systems, 10.0, 30), (others, 10.0, 6)):
        fresh = make()
        for b in (kept, fresh):
            for i, (s, _) in enumerate(which):
                b.set_HS(i, s.H, s.S, s.T)
            b.minimize([c for _, c in which], [0.5] * 4, [tau] * 4, 0.0, iters)
        assert np.array_equal(kept.energies(), fresh.energies()), (tau, iters)
        for i in range(4):
            assert np.array_equal(kept.get_C(i), fresh.get_C(i))
        torch.zeros(1000, device="cuda").add_(1.0)
        torch.cuda.synchronize()
