"""The line minimum and the updates in one launch (up to 704 Wannier functions: 256 blocks of partial
sums) and in separate launches beyond."""

import numpy as np
import pytest

from oracle import omm as oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,rtol", [("fp64", 1e-11), ("bf16x3", 1e-3)])
@pytest.mark.parametrize("n,m", [(40, 31), (40, 32), (40, 33), (71, 64), (720, 704), (721, 704), (720, 705)])
def test_line_update_follows_oracle(n, m, precision, rtol):
    """Energies of a few line searches on both sides of the 32-wide tiles and of the 704 limit, for even
    and odd row lengths. FP64 to rounding; the BF16 scheme perturbs each search direction by its bf16
    rounding (2^-9), which moves the energies of the first line searches by less than 1e-3."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1312_1549_amd import OMM

    print(f"[gpu-case] line update n={n} m={m} {precision}", flush=True)
    rng = np.random.default_rng(n + m)
    A = rng.standard_normal((n, n)) / np.sqrt(n)
    S = np.eye(n) + 0.05 * (A + A.T)
    B = rng.standard_normal((n, n)) / np.sqrt(n)
    H = 0.5 * (B + B.T) + np.diag(rng.uniform(-1.0, 0.0, n))
    C0 = rng.standard_normal((m, n)) * (0.2 / (np.sqrt(n) + np.sqrt(m)))
    solver = OMM(n, m, precision=precision, resync=100)
    solver.set_HS(H, S, S)
    solver.minimize(C0, eta=3.0, tau=10.0, tol=0.0, max_iter=4)
    ref = oracle.minimize(H, S, S, C0, 3.0, 10.0, 0.0, 4)
    scale = np.max(np.abs(ref.energies))
    np.testing.assert_allclose(solver.energy_trace(), ref.energies, rtol=0, atol=rtol * scale)
    # HW and SW are those of the returned C, and exactly symmetric
    C = solver.get_C()
    HW, SW = solver.subspace()
    assert np.array_equal(HW, HW.T) and np.array_equal(SW, SW.T)
    tol = 1e-10 if precision == "fp64" else 1e-9  # bf16x3: recomputed in FP64 at the end of the call
    assert np.max(np.abs(C @ S @ C.T - SW)) <= tol * max(1.0, np.abs(SW).max())
    assert np.max(np.abs(C @ (H - 3.0 * S) @ C.T - HW)) <= tol * max(1.0, np.abs(HW).max())
