"""The one-launch sides of a V-cycle against a V-cycle written from its
definition on the exported level matrices: one BiCGStab iteration (two
V-cycles), at extents around the tile sizes (24, 32 and 40 cells in 2D, 8 in
3D), odd and even, with explicit rows of every reach, with and without
second-phase unknowns, and at other sweep counts. Bars: FP64 1e-10 of the
iterate (rounding, over one iteration); mixed 1e-4 (FP32 V-cycles)."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spl

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"

CASES = {
    "box 2d 48": lambda: W.manufactured_sine(48),
    "box 2d 97": lambda: W.manufactured_sine(97),
    "box 2d 73": lambda: W.eddington(2, 73, 3.0, seed=1),
    "box 3d 16": lambda: W.eddington(3, 16, 3.0, seed=1),
    "box 3d 17": lambda: W.eddington(3, 17, 9.0, seed=1),
    "box 3d 40": lambda: W.eddington(3, 40, 3.0, seed=1),
    "disks 64": lambda: W.two_disks(64, seed=3),
    "disks 81": lambda: W.two_disks(81, seed=3),
    "disks 200": lambda: W.two_disks(200, seed=3),
    "pin 32": lambda: W.pin_plane(32, seed=2),
    "pin 36": lambda: W.pin_plane(36, seed=2),
}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


def _vcycle(P, pr, nu1, nu2):
    """The V-cycle from zero on the exported matrices, as a function of b."""
    ext, lev = list(pr.n) if np.ndim(pr.n) else [pr.n] * pr.dim, []
    for q in range(P.levels):
        tag, prim, sec = P.level_arrays(q)
        n = ext + [1] * (3 - len(ext))
        cell = np.concatenate([np.arange(len(tag)), sec])
        ijk = (cell % n[0], cell // n[0] % n[1], cell // n[0] // n[1])
        phase = np.concatenate([prim, np.ones(len(sec), prim.dtype)])
        lev.append(dict(A=P.operator(q), cell=cell, ijk=ijk, phase=phase, n=n, col=sum(ijk) & 1, live=phase >= 0))
        ext = [(e + 1) // 2 for e in ext]
    for f, c in zip(lev[:-1], lev[1:]):
        at = {(int(x), int(p)): k for k, (x, p) in enumerate(zip(c["cell"], c["phase"])) if p >= 0}
        par = f["ijk"][0] // 2 + c["n"][0] * (f["ijk"][1] // 2 + c["n"][1] * (f["ijk"][2] // 2))
        rows = np.flatnonzero(f["live"])
        cols = [at[(int(par[r]), int(f["phase"][r]))] for r in rows]
        f["P"] = sp.csr_matrix((np.ones(len(rows)), (rows, cols)), shape=(len(f["cell"]), len(c["cell"])))
    lu = spl.splu(lev[-1]["A"].tocsc())

    def smooth(f, x, b, nu):
        d = f["A"].diagonal()
        for _ in range(nu):
            for colour in (0, 1):
                m = (f["col"] == colour) & f["live"]
                x = x + np.where(m, (b - f["A"] @ x) / d, 0.0)
        return x

    def cycle(b, q=0):
        f = lev[q]
        if q == len(lev) - 1:
            return lu.solve(b)
        x = smooth(f, np.zeros_like(b), b, nu1)
        r = np.where(f["live"], b - f["A"] @ x, 0.0)
        return smooth(f, x + f["P"] @ cycle(f["P"].T @ r / 2 ** pr.dim, q + 1), b, nu2)
    return cycle, lev[0]["A"]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name,nu1,nu2", [(n, 2, 2) for n in sorted(CASES)] +
                         [("disks 81", 1, 2), ("disks 81", 2, 0), ("pin 32", 1, 1), ("box 3d 17", 0, 2)])
def test_one_iteration(ctx, name, nu1, nu2, prec):
    print("tile levels", name, nu1, nu2, prec, flush=True)
    pr = CASES[name]()
    P = ebmg.Problem(ctx, pr, precision=prec, smoother=4, tail=1, krylov=2, nu1=nu1, nu2=nu2)
    M, A = _vcycle(P, pr, nu1 or 2, nu2 or 2)   # (0 stands for the default of two sweeps)
    t = lambda a: torch.tensor(np.ascontiguousarray(a).ravel(), dtype=torch.float64, device=DEV)   # noqa: E731
    phi = torch.zeros(P.N, dtype=torch.float64, device=DEV)
    phi2 = torch.zeros(max(P.N2, 1), dtype=torch.float64, device=DEV)
    P.solve(t(pr.rho), phi, sigma=t(pr.sigma) if pr.sigma is not None else None, phi2=phi2 if P.N2 else None,
            rtol=1e-14, max_cycles=2, check=False)
    x = np.concatenate([phi.cpu().numpy(), phi2.cpu().numpy()[:P.N2]])
    b = P.rhs()
    p = M(b)
    v = A @ p
    alpha = (b @ b) / (b @ v)
    s = b - alpha * v
    z = M(s)
    w = A @ z
    want = alpha * p + (w @ s) / (w @ w) * z
    assert np.linalg.norm(x - want) <= (1e-10 if prec == 0 else 1e-4) * np.linalg.norm(want)
    P.release()


@pytest.mark.parametrize("name", ["box 2d 97", "box 2d 73", "box 3d 17", "box 3d 40"])
def test_one_refinement(ctx, name):
    """Plain refinement in FP64, where a tiled level 0 adds its result to x."""
    print("tile refinement", name, flush=True)
    pr = CASES[name]()
    P = ebmg.Problem(ctx, pr, precision=0, smoother=4, tail=1, krylov=1)
    M, A = _vcycle(P, pr, 2, 2)
    b = P.rhs()
    phi = torch.zeros(P.N, dtype=torch.float64, device=DEV)
    rho = torch.tensor(np.ascontiguousarray(pr.rho).ravel(), dtype=torch.float64, device=DEV)
    x = np.zeros_like(b)
    for cycles in (1, 2):
        x = x + M(b - A @ x)
        _, info = P.solve(rho, phi.zero_(), rtol=1e-14, max_cycles=cycles, check=False)
        assert np.linalg.norm(phi.cpu().numpy() - x) <= 1e-10 * np.linalg.norm(x)
        rel = np.linalg.norm(b - A @ x) / np.linalg.norm(b)
        assert abs(info["rel_residual"] - rel) <= 1e-8 * rel
    P.release()
