"""Workloads of the orbital minimization on one GPU, each driven through the public entry points.

Four kinds of work, as a program that uses the solver meets them:

* ``scf``: one self-consistent step at a fixed geometry. A new Hamiltonian with the S and T of the
  step before goes in, a fixed number of CG line searches runs from the coefficients at hand, and
  the density matrix comes out (``set_HS``, ``minimize``, ``density``). With ``geometries`` = 2
  the pass is two steps of a molecular-dynamics run: S and T change with the atoms, so every
  step also builds its own preconditioner (or Cholesky factor).
* ``forces``: the derivatives of the minimum energy with respect to H and S (``backward``).
* ``batch``: many independent systems of uneven size in grouped launches (``OMMBatch``).
* ``kpoint``: a complex Hermitian problem (``OMMComplex``).

The number of line searches is fixed (tol = 0), so that a pass is the same work every time.
Results are returned in the digits of the arithmetic that made them: FP64 results as they are,
those of FP32 products in float32, and those of the BF16 scheme, whose search directions are
rounded to bf16, in bfloat16 (its energies are Python floats).
"""

import math

import numpy as np
import torch

from paper_1312_1549_amd import OMM, OMMBatch, OMMComplex

DEVICE = "cuda"
RESULT = {"fp64": torch.float64, "fp32": torch.float32, "bf16x3": torch.bfloat16}


def listed():
    return [
        # 32 atoms of four orbitals, the smallest workload of the benchmark: a serial chain of tiny
        # products and reductions, so latency and the number of launches count
        dict(name="scf-128-fp64", kind="scf", N=128, M=24, orbs=4, precision="fp64", iters=20,
             flavour="dense", sparse=False, geometries=1),
        # an odd size between the benchmark's first two, in molecular dynamics: every step inverts
        # its own preconditioner and needs only a few line searches from the last step's C
        dict(name="dynamics-717-fp64", kind="scf", N=717, M=131, orbs=4, precision="fp64", iters=10,
             flavour="dense", sparse=False, geometries=2),
        # the 512-atom workload (N = 2048) in FP64: the reference precision
        dict(name="scf-2048-fp64", kind="scf", N=2048, M=384, orbs=4, precision="fp64", iters=20,
             flavour="dense", sparse=False, geometries=1),
        # the same in the BF16 scheme with FP64 state: one resynchronization period
        dict(name="scf-2048-bf16", kind="scf", N=2048, M=384, orbs=4, precision="bf16x3", iters=80,
             flavour="dense", sparse=False, geometries=1),
        # Cholesky-reduced flavour on a ragged size, in dynamics: factorization, reduction of H
        # and a few line searches per geometry
        dict(name="dynamics-2301-cholesky", kind="scf", N=2301, M=413, orbs=13, precision="fp64",
             iters=10, flavour="cholesky", sparse=False, geometries=2),
        # the 1024-atom workload (N = 4096) with FP32 products
        dict(name="scf-4096-fp32", kind="scf", N=4096, M=768, orbs=4, precision="fp32", iters=20,
             flavour="dense", sparse=False, geometries=1),
        # backward pass of the differentiable energy on the 1024-atom workload
        dict(name="forces-4096", kind="forces", N=4096, M=768, orbs=4, precision="fp64", iters=3),
        # 500 atoms of 13 orbitals with block-sparse operator products
        dict(name="scf-6500-sparse", kind="scf", N=6500, M=1000, orbs=13, precision="bf16x3",
             iters=80, flavour="dense", sparse=True, geometries=1),
        # the headline workload: 1000 atoms of 13 orbitals, one period of 80 line searches
        dict(name="scf-13000-bf16", kind="scf", N=13000, M=2000, orbs=13, precision="bf16x3",
             iters=80, flavour="dense", sparse=False, geometries=1),
        # 32 systems of 64 to 256 atoms, FP32 grouped phase and FP64 grouped phase
        dict(name="batch-32", kind="batch", systems=32, min_atoms=64, max_atoms=256, iters=10),
        # one k-point of a 128-atom cell (its real embedding is 1024 x 192)
        dict(name="kpoint-512-fp64", kind="kpoint", N=512, M=96, orbs=4, precision="fp64", iters=20),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scf", "scf", "scf", "scf", "forces", "batch", "kpoint"])
    if kind == "batch":
        lo = rng.randint(16, 96)
        return dict(kind=kind, systems=rng.randint(4, 40), min_atoms=lo,
                    max_atoms=rng.randint(lo, 288), iters=rng.randint(5, 15))
    orbs = rng.choice([1, 4, 4, 9, 13])
    if kind == "forces":
        N = _log_uniform(rng, 200, 6000)
        return dict(kind=kind, N=N, M=_occupied(rng, N), orbs=orbs, precision="fp64",
                    iters=rng.randint(1, 3))
    if kind == "kpoint":
        N = _log_uniform(rng, 48, 1000)
        return dict(kind=kind, N=N, M=_occupied(rng, N), orbs=orbs, precision="fp64",
                    iters=rng.randint(10, 20))
    precision = rng.choice(["fp64", "fp64", "fp32", "bf16x3", "bf16x3"])
    N = _log_uniform(rng, *((400, 8000) if precision == "bf16x3" else (100, 4500)))
    flavour = rng.choice(["dense", "dense", "dense", "cholesky"])
    return dict(kind=kind, N=N, M=_occupied(rng, N), orbs=orbs, precision=precision,
                iters=80 if precision == "bf16x3" else rng.randint(5, 20), flavour=flavour,
                sparse=precision == "bf16x3" and flavour == "dense" and rng.random() < 0.3,
                geometries=1 if rng.random() < 0.7 or N > 3000 else 2)


def _occupied(rng, N):
    return max(1, int(N * rng.uniform(0.12, 0.2)))


# ---- inputs: the finite-range model of synth/generator.py, drawn on the GPU ----------------------
def _box(atoms):
    k = 1
    while k ** 3 < atoms:
        k += 1
    d = [k, k, k]
    for ax in (2, 1, 0):
        if (d[0] * d[1] * d[2]) // d[ax] * (d[ax] - 1) >= atoms:
            d[ax] -= 1
    return d


def _lowest(A, steps=48):
    """Lowest and highest eigenvalue of a Hermitian A, by Lanczos with full reorthogonalization."""
    n = A.shape[0]
    steps = min(steps, n)
    V = torch.zeros((steps, n), dtype=A.dtype, device=A.device)
    v = torch.cos(torch.arange(n, dtype=torch.float64, device=A.device) ** 2).to(A.dtype)
    K = torch.zeros((steps, steps), dtype=torch.float64, device=A.device)
    for k in range(steps):
        V[k] = v / torch.linalg.vector_norm(v)
        v = A @ V[k]
        K[k, k] = torch.real(torch.vdot(V[k], v))
        for _ in range(2):
            v = v - V[: k + 1].T @ (V[: k + 1].conj() @ v)
        if k + 1 < steps:
            K[k, k + 1] = K[k + 1, k] = torch.linalg.vector_norm(v)
    w = torch.linalg.eigvalsh(torch.nan_to_num(K).cpu())
    return float(w[0]), float(w[-1])


def _matrices(N, orbs, seed, phase=None):
    """H, S, T (real, or Hermitian with one Bloch phase per atom pair when `phase` is given) and an
    upper bound of S's spectrum."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    f64 = dict(dtype=torch.float64, device=DEVICE)
    atoms = -(-N // orbs)
    a, rc = (3.0, 8.0) if orbs > 4 else (2.5, 6.0)
    nx, ny, _ = _box(atoms)
    i = torch.arange(atoms, device=DEVICE)
    pos = torch.stack([i % nx, (i // nx) % ny, i // (nx * ny)], 1).to(torch.float64) * a
    pos = pos + 0.4 * torch.rand(pos.shape, generator=g, **f64) - 0.2
    at = torch.arange(N, device=DEVICE) // orbs
    r_at = torch.cdist(pos, pos, compute_mode="donot_use_mm_for_euclid_dist")
    r = r_at[at][:, at]
    A = torch.exp(-r / 1.5)
    A *= 0.5 + 0.5 * torch.rand((N, N), generator=g, **f64)
    A *= torch.randint(0, 2, (N, N), generator=g, device=DEVICE) * 2 - 1
    A *= (r <= rc) & (at[:, None] != at[None, :])
    A = torch.triu(A, 1)
    if phase is not None:
        dx = pos[:, 0][at]
        A = A * torch.polar(torch.ones_like(r), phase * (dx[None, :] - dx[:, None]))
    A = A + A.mH
    lo, hi = _lowest(A)
    shift = max(0.0, math.ceil((0.1 - (1.0 + lo * 1.02)) * 1024) / 1024)
    T = A * (1.5 - 0.25 * r * r)
    T.diagonal().fill_(1.5 * (1.0 + shift))
    A.diagonal().fill_(1.0 + shift)
    H = T.clone()
    H.diagonal().sub_(torch.rand(N, generator=g, **f64))
    return H.contiguous(), A.contiguous(), T.contiguous(), 1.0 + shift + hi * 1.02


def _start(M, N, bound, seed, dtype=torch.float64):
    """C0 = sigma Z, scaled so that the largest eigenvalue of C0 S C0^H stays below 1/4."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    Z = torch.randn((M, N), generator=g, dtype=dtype, device=DEVICE)
    return Z * min(0.01, 0.5 / ((math.sqrt(N) + math.sqrt(M)) * 1.05 * math.sqrt(bound)))


def _perturbed(H, seed, amplitude=1e-3):
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    U = torch.triu(torch.randn(H.shape, generator=g, dtype=torch.float64, device=DEVICE))
    return H + amplitude * (U + torch.triu(U, 1).T)


def _eta(case):
    return 0.0 if case["orbs"] > 4 else 0.5


TAU = 10.0


def _inputs(case, seed):
    """Per geometry: (H, S, T, C0)."""
    out = []
    for k in range(case.get("geometries", 1)):
        H, S, T, bound = _matrices(case["N"], case["orbs"], 1000 * seed + 10 * k)
        out.append((H, S, T, _start(case["M"], case["N"], bound, 1000 * seed + 10 * k + 1)))
    return out


def _batch_sizes(case, seed):
    """Atoms of every system: fixed by the case, so that another seed is the same amount of work."""
    n, lo, hi = case["systems"], case["min_atoms"], case["max_atoms"]
    return [lo + ((hi - lo) * ((k * 37) % n)) // max(1, n - 1) for k in range(n)]


def prepare(case, seed):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        if case["kind"] == "batch":
            atoms = _batch_sizes(case, seed)
            Ns = [4 * a for a in atoms]
            Ms = [max(1, round(3 * n / 16)) for n in Ns]
            b = OMMBatch(Ns, Ms, precision="fp32", refine=True)
            C0s = []
            for i, (n, m) in enumerate(zip(Ns, Ms)):
                H, S, T, bound = _matrices(n, 4, 1000 * seed + 2 * i)
                b.set_HS(i, H, S, T)
                C0s.append(_start(m, n, bound, 1000 * seed + 2 * i + 1).cpu().numpy())
            return dict(case=case, stream=stream, solver=b, C0s=C0s)
        N, M = case["N"], case["M"]
        if case["kind"] == "kpoint":
            H, S, T, bound = _matrices(N, case["orbs"], 1000 * seed, phase=0.3)
            solver = OMMComplex(N, M, precision=case["precision"])
            solver.set_HS(H.cpu().numpy(), S.cpu().numpy(), T.cpu().numpy())
            C0 = _start(M, N, bound, 1000 * seed + 1, torch.complex128).cpu().numpy()
            return dict(case=case, stream=stream, solver=solver, C0=C0)
        steps = _inputs(case, seed)
        solver = OMM(N, M, precision=case["precision"], refine=case["precision"] == "bf16x3",
                     flavour=case.get("flavour", "dense"), sparse=case.get("sparse", False))
        solver.set_HS(*steps[0][:3])
        state = dict(case=case, stream=stream, solver=solver,
                     steps=[(_perturbed(H, 1000 * seed + 7) if len(steps) == 1 else H, S, T, C0)
                            for H, S, T, C0 in steps],
                     out=[torch.empty((N, N), dtype=torch.float64, device=DEVICE) for _ in range(2)])
        if case["kind"] == "forces":
            H, S, T, C0 = steps[0]
            solver.minimize(C0, eta=_eta(case), tau=TAU, tol=0.0, max_iter=case["iters"])
        return state


def run(state):
    case, solver = state["case"], state["solver"]
    with torch.cuda.stream(state["stream"]):
        if case["kind"] == "batch":
            n = len(state["C0s"])
            solver.minimize(state["C0s"], [0.5] * n, [TAU] * n, 0.0, case["iters"])
            return dict(energies=solver.energies().astype(np.float32),
                        C=[solver.get_C(i).astype(np.float32) for i in range(n)])
        if case["kind"] == "kpoint":
            solver.minimize(state["C0"], eta=_eta(case), tau=TAU, tol=0.0, max_iter=case["iters"])
            return dict(trace=solver.energy_trace(), rho=solver.density())
        if case["kind"] == "forces":
            dH, dS = state["out"]
            solver.backward(1.0, dH, dS)
            return dict(dH=dH, dS=dS)
        answer = {}
        for k, (H, S, T, C0) in enumerate(state["steps"]):
            solver.set_HS(H, S, T)
            solver.minimize(C0, eta=_eta(case), tau=TAU, tol=0.0, max_iter=case["iters"])
            rho = solver.density(out=state["out"][k])
            answer["energy%d" % k] = solver.energy()
            answer["rho%d" % k] = rho.to(RESULT[case["precision"]])
            if case["precision"] == "fp64":
                answer["trace%d" % k] = solver.energy_trace()
        return answer


# ---- what a pass cannot do without -----------------------------------------------------------
def _solve_flops(N, M, iters, reduced=False, filling=1.0):
    """Initial products and `iters` line searches; symmetric M x M results count by their half."""
    op = 2.0 * M * N * N
    first = (1 if reduced else 2 * filling) * op + 2.0 * M * M * N
    line = (1 if reduced else 2 * filling + 1) * op + 10.0 * M * M * N
    return first + iters * line


def _density_flops(N, M):
    return 2.0 * M * M * N + 1.0 * M * N * N  # (2I - SW) C, then half of a symmetric N x N


def work(case):
    if case["kind"] == "batch":
        sizes = [(4 * a, max(1, round(3 * 4 * a / 16))) for a in _batch_sizes(case, 0)]
        return dict(bytes=sum(24.0 * n * n + 20.0 * m * n for n, m in sizes),
                    flops=sum(2 * _solve_flops(n, m, case["iters"]) for n, m in sizes))
    N, M = case["N"], case["M"]
    if case["kind"] == "kpoint":  # a complex product is four real ones
        return dict(bytes=3 * 16.0 * N * N + 16.0 * M * N + 16.0 * N * N,
                    flops=4 * (_solve_flops(N, M, case["iters"]) + _density_flops(N, M)))
    if case["kind"] == "forces":
        return dict(bytes=8.0 * M * N + 16.0 * M * M + 16.0 * N * N, flops=2 * _density_flops(N, M))
    filling, reduced, setup = 1.0, case["flavour"] == "cholesky", 0.0
    if case["sparse"]:  # orbitals within the cutoff of one orbital
        a, rc = (3.0, 8.0) if case["orbs"] > 4 else (2.5, 6.0)
        filling = min(1.0, 4.19 * (rc / a) ** 3 * case["orbs"] / N)
    if case["geometries"] > 1:  # symmetric inverse; Cholesky: L, L^-1 H L^-T, C L, C~ L^-1
        setup = (4.0 / 3 + 1 / 3.0) * N ** 3 + 4.0 * M * N * N if reduced else 1.0 * N ** 3
    elif reduced:  # H changes with every step
        setup = 4.0 / 3 * N ** 3 + 4.0 * M * N * N
    step = _solve_flops(N, M, case["iters"], reduced, filling) + _density_flops(N, M) + setup
    return dict(bytes=case["geometries"] * (4 * 8.0 * N * N + 8.0 * M * N),
                flops=case["geometries"] * step)


# ---- the same results in plain FP64 torch ----------------------------------------------------
def _line_minimum(a):
    """First local minimum of sum_k a[k] x^k met going downhill from x = 0."""
    if a[1] == 0.0:
        return 0.0
    side = 1.0 if a[1] < 0.0 else -1.0
    roots = np.roots([4 * a[4], 3 * a[3], 2 * a[2], a[1]])
    best = None
    for x in roots[np.abs(roots.imag) < 1e-9 * (1 + np.abs(roots.real))].real:
        for _ in range(3):
            x = x - np.polyval([4 * a[4], 3 * a[3], 2 * a[2], a[1]], x) / np.polyval(
                [12 * a[4], 6 * a[3], 2 * a[2]], x)
        if side * x > 0 and np.polyval([12 * a[4], 6 * a[3], 2 * a[2]], x) > 0:
            best = x if best is None or abs(x) < abs(best) else best
    return best


def _minimized(H, S, T, C, eta, tau, iters):
    """C and the energies after `iters` CG line searches in FP64 (real or complex Hermitian)."""
    Hs = H - eta * S
    K = torch.linalg.cholesky(S + T / tau) if math.isfinite(tau) else torch.linalg.cholesky(S)
    ip = lambda X, Y: float(torch.real(torch.sum(X.conj() * Y)))  # noqa: E731
    tr = lambda X, Y: float(torch.real(torch.sum(X * Y.T)))  # noqa: E731  Tr(X Y)
    HC, SC = C @ Hs, C @ S
    HW, SW = HC @ C.mH, SC @ C.mH
    energy = lambda: 4 * float(torch.real(torch.trace(HW))) - 2 * tr(SW, HW)  # noqa: E731
    E, D, old = [energy()], None, None
    for k in range(iters):
        G = 8 * HC - 4 * (HW @ SC) - 4 * (SW @ HC)
        PG = torch.cholesky_solve(G.mH.contiguous(), K).mH.contiguous()
        if D is None:
            D = -PG
        else:
            D = -PG + (ip(PG, G) - ip(PG, old[0])) / ip(old[1], old[0]) * D
        old = (G, PG)
        HD, SD = D @ Hs, D @ S
        H1, S1, H2, S2 = D @ HC.mH, D @ SC.mH, D @ HD.mH, D @ SD.mH
        t = lambda X: float(torch.real(torch.trace(X)))  # noqa: E731
        a = [4 * t(HW) - 2 * tr(SW, HW),
             8 * t(H1) - 4 * tr(S1, HW) - 4 * tr(SW, H1),
             4 * t(H2) - 2 * tr(S2, HW) - 2 * tr(SW, H2) - 4 * tr(S1, H1) - 4 * ip(S1, H1),
             -4 * tr(S2, H1) - 4 * tr(S1, H2),
             -2 * tr(S2, H2)]
        x = _line_minimum(a)
        C, HC, SC = C + x * D, HC + x * HD, SC + x * SD
        HW = HW + x * (H1 + H1.mH) + x * x * H2
        SW = SW + x * (S1 + S1.mH) + x * x * S2
        E.append(energy())
    return C, HW, SW, E


def _density(C, SW):
    return 2 * C.mH @ (2 * C - SW @ C)


def exact(case, seed):
    if case["kind"] == "batch":
        E, Cs = [], []
        for i, atoms in enumerate(_batch_sizes(case, seed)):
            n, m = 4 * atoms, max(1, round(3 * 4 * atoms / 16))
            H, S, T, bound = _matrices(n, 4, 1000 * seed + 2 * i)
            C0 = _start(m, n, bound, 1000 * seed + 2 * i + 1)
            C, _, _, e = _minimized(H, S, T, C0, 0.5, TAU, case["iters"])
            # the FP64 phase starts afresh (steepest descent) from the FP32 phase's C
            C, _, _, e = _minimized(H, S, T, C, 0.5, TAU, case["iters"])
            E.append(e[-1])
            Cs.append(C)
        return dict(energies=np.array(E), C=Cs)
    if case["kind"] == "kpoint":
        H, S, T, bound = _matrices(case["N"], case["orbs"], 1000 * seed, phase=0.3)
        C0 = _start(case["M"], case["N"], bound, 1000 * seed + 1, torch.complex128)
        C, _, SW, E = _minimized(H, S, T, C0, _eta(case), TAU, case["iters"])
        # rows of C hold conjugated coefficients: rho = 2 C^H (2I - SW) C
        return dict(trace=np.array(E), rho=_density(C, SW))
    answer = {}
    steps = _inputs(case, seed)
    for k, (H, S, T, C0) in enumerate(steps):
        if case["kind"] == "scf" and len(steps) == 1:
            H = _perturbed(H, 1000 * seed + 7)
        tau = math.inf if case.get("flavour") == "cholesky" else TAU
        C, HW, SW, E = _minimized(H, S, T, C0, _eta(case), tau, case["iters"])
        rho = _density(C, SW)
        if case["kind"] == "forces":
            return dict(dH=rho, dS=-2 * C.T @ (HW @ C) - _eta(case) * rho)
        answer["energy%d" % k] = E[-1]
        answer["rho%d" % k] = rho
        if case["precision"] == "fp64":
            answer["trace%d" % k] = np.array(E)
    return answer
