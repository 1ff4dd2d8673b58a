"""The small FP64 / FP32 GEMM tiles (16x32 to 64x96, each wave taking every fourth K step): every tile
shape pinned with OMM_TILE, at sizes that leave partial tiles, partial K steps, odd extents of the
r-contiguous operands and fewer K steps than waves."""

import sys

import numpy as np
import pytest

from oracle import omm as oracle
from synth import start_coefficients
from synth.generator import lattice_positions, make_system

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def OMM():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1312_1549_amd import OMM

    return OMM


def _system(dims, orbs, M, seed):
    rng = np.random.default_rng(seed)
    pos = lattice_positions(dims, 2.5)
    pos = pos + rng.uniform(-0.2, 0.2, size=pos.shape)
    s = make_system(pos, orbs, 6.0, M, rng, name="tiles", eta=0.5, tau=10.0, seed=seed)
    return s, start_coefficients(s.S, s.M, seed + 1)


# N, M: one K step and less; odd and even; tile extents and one more (16, 32, 48, 64, 96)
SIZES = [((2, 1, 1), 4, 1), ((3, 3, 1), 1, 2), ((4, 4, 1), 1, 5), ((7, 7, 1), 1, 16),
         ((4, 3, 2), 4, 17), ((5, 5, 1), 5, 33), ((8, 3, 2), 4, 49), ((5, 5, 2), 4, 65),
         ((7, 4, 4), 3, 97)]


@pytest.mark.parametrize("tile", [None, 7, 8, 9, 10, 11, 12])
@pytest.mark.parametrize("dims,orbs,M", SIZES)
def test_small_tiles_against_oracle(OMM, dims, orbs, M, tile, monkeypatch):
    """FP64: the energies of a few line searches follow the oracle; the density matrix and dE/dS equal
    the products of the returned C and subspace matrices within the rounding of their sums."""
    import torch

    s, C0 = _system(dims, orbs, M, 70 + M)
    if tile is None:
        monkeypatch.delenv("OMM_TILE", raising=False)
    else:
        monkeypatch.setenv("OMM_TILE", str(tile))
    print(f"[gpu-case] small tile {tile} N={s.N} M={M} fp64", flush=True)
    sys.stdout.flush()
    solver = OMM(s.N, s.M, precision="fp64")
    solver.set_HS(s.H, s.S, s.T)
    solver.minimize(C0, eta=0.5, tau=10.0, tol=0.0, max_iter=4)
    ref = oracle.minimize(s.H, s.S, s.T, C0, 0.5, 10.0, 0.0, 4)
    np.testing.assert_allclose(solver.energy_trace(), ref.energies, rtol=1e-11, atol=0)
    C = solver.get_C()
    HW, SW = solver.subspace()
    rho = solver.density()
    dH = torch.empty((s.N, s.N), dtype=torch.float64, device="cuda")
    dS = torch.empty_like(dH)
    solver.backward(0.75, dH, dS)
    # two sums of M terms each (Y C, then C^T Z), every term rounded once and every partial sum once
    bound = lambda Y: 4.0 * (2 * M + 8) * EPS * (np.abs(C).T @ (np.abs(Y) @ np.abs(C)))  # noqa: E731
    Y = 2.0 * np.eye(M) - SW
    b_rho = bound(2.0 * np.eye(M) + np.abs(SW))
    exact = 2.0 * C.T @ (Y @ C)
    assert np.all(np.abs(rho - exact) <= b_rho)
    assert np.array_equal(rho, rho.T)
    assert np.all(np.abs(dH.cpu().numpy() - 0.75 * exact) <= b_rho)
    exact_dS = -0.75 * (2.0 * C.T @ (HW @ C) + 0.5 * exact)
    assert np.all(np.abs(dS.cpu().numpy() - exact_dS) <= bound(HW) + b_rho)


@pytest.mark.parametrize("tile", [None, 7, 8, 9, 10, 11, 12])
@pytest.mark.parametrize("dims,orbs,M", SIZES[2::3])
def test_small_tiles_fp32(OMM, dims, orbs, M, tile, monkeypatch):
    """FP32 products: relative errors of 1e-7 per product, a few hundred terms and four line searches
    stay below 1e-5 of the energy."""
    s, C0 = _system(dims, orbs, M, 90 + M)
    if tile is None:
        monkeypatch.delenv("OMM_TILE", raising=False)
    else:
        monkeypatch.setenv("OMM_TILE", str(tile))
    print(f"[gpu-case] small tile {tile} N={s.N} M={M} fp32", flush=True)
    sys.stdout.flush()
    solver = OMM(s.N, s.M, precision="fp32", refine=False)
    solver.set_HS(s.H, s.S, s.T)
    solver.minimize(C0, eta=0.5, tau=10.0, tol=0.0, max_iter=4)
    ref = oracle.minimize(s.H, s.S, s.T, C0, 0.5, 10.0, 0.0, 4)
    scale = np.max(np.abs(ref.energies))
    np.testing.assert_allclose(solver.energy_trace(), ref.energies, rtol=0, atol=1e-5 * scale)


def test_grouped_small_tiles_match_single_systems(OMM):
    """Grouped launches (tile lists of uneven systems) against the same systems one by one."""
    from paper_1312_1549_amd import OMMBatch

    systems = [_system(d, o, m, 110 + m) for d, o, m in SIZES]
    print("[gpu-case] grouped small tiles", flush=True)
    batch = OMMBatch([s.N for s, _ in systems], [s.M for s, _ in systems], precision="fp64")
    for i, (s, _) in enumerate(systems):
        batch.set_HS(i, s.H, s.S, s.T)
    n = len(systems)
    batch.minimize([c for _, c in systems], [0.5] * n, [10.0] * n, 0.0, 4)
    E = batch.energies()
    for i, (s, C0) in enumerate(systems):
        ref = oracle.minimize(s.H, s.S, s.T, C0, 0.5, 10.0, 0.0, 4)
        assert abs(E[i] - ref.energies[-1]) <= 1e-11 * np.max(np.abs(ref.energies))
