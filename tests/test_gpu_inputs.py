"""Device inputs of one context: the fused check (finite, symmetric, changed or not) and store."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1312_1549_amd import OMM
    from paper_1312_1549_amd.omm import OMMError

    return torch, OMM, OMMError


def _spd(n, seed):
    A = 0.1 / np.sqrt(n) * np.random.default_rng(seed).standard_normal((n, n))
    return 0.5 * (A + A.T) + np.eye(n)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 65])
def test_device_inputs_are_checked_and_kept(api, n):
    """A bad entry anywhere (each of H, S, T; first, last and middle pairs) is refused with the error
    of the first bad matrix, and the inputs of before stay in force; symmetric to 1e-10 is accepted
    and stored symmetrized; only a change of S or T drops the preconditioner."""
    torch, OMM, OMMError = api
    print(f"[gpu-case] device inputs n={n}", flush=True)
    H, S, T = (_spd(n, k) for k in range(3))
    dev = lambda A: torch.from_numpy(A.copy()).cuda()  # noqa: E731
    C0 = np.full((1, n), 1e-2)
    solver = OMM(n, 1, precision="fp64")
    solver.set_HS(dev(H), dev(S), dev(T))
    run = lambda: (solver.minimize(C0, eta=2.0, tau=5.0, tol=0.0, max_iter=2), solver.energy())[1]  # noqa: E731
    E0 = run()
    P0 = solver.preconditioner()
    pairs = {(0, n - 1), (n - 1, 0), (n // 2, 0), (n - 1, n // 2), (0, 0)}
    for which in range(3):
        for i, j in pairs:
            for value, error in ((np.nan, "OMM_E_NONFINITE"), (np.inf, "OMM_E_NONFINITE"), (9.0, "OMM_E_ASYMMETRIC")):
                if error == "OMM_E_ASYMMETRIC" and i == j:
                    continue
                mats = [H.copy(), S.copy(), T.copy()]
                mats[which][i, j] = value
                with pytest.raises(OMMError, match=error):
                    solver.set_HS(*(dev(m) for m in mats))
    assert run() == E0 and np.array_equal(solver.preconditioner(), P0)
    # the first bad matrix is the one reported
    bad = H.copy()
    bad[0, 0] = np.nan
    badT = T.copy()
    badT[n - 1, n - 1] = np.inf
    with pytest.raises(OMMError, match="H has a non-finite"):
        solver.set_HS(dev(bad), dev(S), dev(badT))
    # within the tolerance: the average of the pair is stored
    if n > 1:
        near = S.copy()
        near[0, n - 1] += 4e-11
        solver.set_HS(dev(H), dev(near), dev(T))
        run()
        want = near.copy()
        want[0, n - 1] = want[n - 1, 0] = 0.5 * (near[0, n - 1] + near[n - 1, 0])
        inv = np.linalg.inv(want + T / 5.0)
        assert np.max(np.abs(solver.preconditioner() - inv)) <= 1e4 * n * np.finfo(float).eps * np.abs(inv).max() * np.linalg.cond(want)
    # a changed T alone, in one element, rebuilds the preconditioner; a changed H does not
    solver.set_HS(dev(H), dev(S), dev(T))
    run()
    assert np.array_equal(solver.preconditioner(), P0)
    T2 = T.copy()
    T2[n - 1, n - 1] = np.nextafter(T[n - 1, n - 1], 2.0) + 0.25
    solver.set_HS(dev(H + np.eye(n)), dev(S), dev(T2))
    run()
    inv = np.linalg.inv(S + T2 / 5.0)
    assert np.max(np.abs(solver.preconditioner() - inv)) <= 1e4 * n * np.finfo(float).eps * np.abs(inv).max() * np.linalg.cond(S + T2 / 5.0)
    solver.set_HS(dev(H), dev(S), None)
    assert solver.minimize(C0, eta=2.0, tau=0.0, tol=0.0, max_iter=2) in (0, 1)


@pytest.mark.parametrize("n", [1, 33, 65])
def test_what_new_device_inputs_keep_and_drop(api, n):
    """A new H alone keeps the preconditioner (it can be read before the next minimization); a new S, a new T
    or a dropped T drops it. Without T the results are those of a solver that never had one, and a
    finite tau is refused."""
    torch, OMM, OMMError = api
    print(f"[gpu-case] kept and dropped n={n}", flush=True)
    H, S, T = (_spd(n, k) for k in range(3))
    dev = lambda A: torch.from_numpy(A.copy()).cuda()  # noqa: E731
    C0 = np.full((1, n), 1e-2)
    solver = OMM(n, 1, precision="fp64")
    solver.set_HS(dev(H), dev(S), dev(T))
    solver.minimize(C0, eta=2.0, tau=5.0, tol=0.0, max_iter=2)
    P0 = solver.preconditioner()
    solver.set_HS(dev(H + np.eye(n)), dev(S), dev(T))
    assert np.array_equal(solver.preconditioner(), P0)
    dS, dT = S.copy(), T.copy()
    dS[n - 1, n - 1] = np.nextafter(S[n - 1, n - 1], 2.0)
    dT[0, 0] = np.nextafter(T[0, 0], 2.0)
    for args in ((H, dS, T), (H, S, dT), (H, S, None)):
        solver.set_HS(dev(H), dev(S), dev(T))
        solver.minimize(C0, eta=2.0, tau=5.0, tol=0.0, max_iter=2)
        assert np.array_equal(solver.preconditioner(), P0)
        solver.set_HS(*(None if A is None else dev(A) for A in args))
        with pytest.raises(OMMError, match="OMM_E_STATE"):
            solver.preconditioner()
    # (H, S, None) is in: tau needs T
    with pytest.raises(OMMError, match="OMM_E_ARG"):
        solver.minimize(C0, eta=2.0, tau=5.0, tol=0.0, max_iter=2)
    fresh = OMM(n, 1, precision="fp64")
    fresh.set_HS(dev(H), dev(S), None)
    for o in (solver, fresh):
        o.minimize(C0, eta=2.0, tau=np.inf, tol=0.0, max_iter=3)
    assert np.array_equal(solver.energy_trace(), fresh.energy_trace())
    assert np.array_equal(solver.get_C(), fresh.get_C())
