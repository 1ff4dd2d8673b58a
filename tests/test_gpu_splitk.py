"""Split-K partials of the BF16 products: row lengths of every remainder modulo the four columns a
thread of the reduction takes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1028, 1029, 1030, 1031])
@pytest.mark.parametrize("m", [40, 41])
def test_split_products_match_unsplit(n, m, monkeypatch):
    """Without the autotuner products of this size split K over workgroups (a few 64 x 64 tiles, K >= 1024);
    pinned to tile 1 they do not. Both add the same FP32 accumulations of bf16 products in another
    order: K / 32 = 33 steps of at most 2^-24 relative each move an energy by less than 1e-5 of
    the largest, over three line searches."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1312_1549_amd import OMM

    print(f"[gpu-case] split-K n={n} m={m}", flush=True)
    rng = np.random.default_rng(n + m)
    A = rng.standard_normal((n, n)) / np.sqrt(n)
    S = np.eye(n) + 0.05 * (A + A.T)
    B = rng.standard_normal((n, n)) / np.sqrt(n)
    H = 0.5 * (B + B.T)
    C0 = rng.standard_normal((m, n)) * (0.2 / np.sqrt(n))
    monkeypatch.setenv("OMM_AUTOTUNE", "0")
    out = []
    for tile in (None, "1"):
        if tile:
            monkeypatch.setenv("OMM_TILE", tile)
        solver = OMM(n, m, precision="bf16x3", resync=100)
        solver.set_HS(H, S, None)
        solver.minimize(C0, eta=3.0, tau=float("inf"), tol=0.0, max_iter=3)
        out.append(solver.energy_trace())
        solver.close()
    np.testing.assert_allclose(out[0], out[1], rtol=0, atol=1e-5 * np.max(np.abs(out[1])))
