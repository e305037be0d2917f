"""Levels of odd extent outside the one-launch V-cycle sides, so that the sweep
kernels themselves meet them: 3D levels above 64^3 and 2D levels above 1024^2,
and smaller ones at three sweeps, under every smoother choice. Boxes whose
solution is a sum of low eigenvectors of the separable operator, the source its
image in extended precision; solved to a relative residual of 1e-10, of which
the error can be the ratio of the largest to the smallest eigenvalue in the sum
times as large (plus half for the rounding of the FP64 residual). Batches of
boxes that coarsen through odd extents, with the bars of the other parity tests
(FP64 1e-10, mixed 1e-8 relative L2)."""
import dataclasses

import numpy as np
import pytest
import scipy.linalg

import workloads as W
from oracle.operator import assemble
from oracle.solvers import rel_residual, solve_splu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


def _box(n, kappa):
    """A plain box of n cells: Poisson with value 0 around (kappa None), or the
    Eddington operator of absorption kappa; its
    source, its solution and the bar of the solution's error."""
    dim, h = len(n), 1.0 / max(n)
    if kappa is None:
        pr = W.Problem(dim, n, h, (0.0,) * dim, [], *W._bc(W.BC_DIRICHLET), name=f"odd-{n}")
        mass, b, end = 0.0, 1.0, 3.0
    else:
        pr = dataclasses.replace(W.eddington_coefficients(dim, max(n), kappa), n=n)
        mass, b, a = kappa, 1.0 / (3.0 * kappa), 1.5 * kappa
        end = 1.0 + a * h / (1.0 + 0.5 * a * h)
    rng = np.random.default_rng(sum(n))
    x, low, top = rng.normal(size=(3,) * dim), mass, mass
    for m in n:
        T = 2.0 * np.eye(m) - np.diag(np.ones(m - 1), 1) - np.diag(np.ones(m - 1), -1)
        T[0, 0] = T[-1, -1] = end
        lam, V = scipy.linalg.eigh(T, subset_by_index=(0, 2))
        x = np.tensordot(x, V, axes=([0], [1]))           # axes cycle to (x, y[, z])
        low, top = low + b / h ** 2 * lam[0], top + b / h ** 2 * lam[2]
    x = np.ascontiguousarray(x.transpose())
    e = x.astype(np.longdouble)
    y = mass * e
    for d in range(dim):
        f = np.moveaxis(e, d, 0)
        g = np.moveaxis(y, d, 0)
        c = np.longdouble(b) / np.longdouble(h) ** 2
        g += 2 * c * f
        g[0] += (end - 2) * c * f[0]
        g[-1] += (end - 2) * c * f[-1]
        g[1:] -= c * f[:-1]
        g[:-1] -= c * f[1:]
    pr.rho = np.ascontiguousarray(y.astype(np.float64))
    return pr, x, 1.5e-10 * top / low


def _solve(ctx, pr, **opts):
    P = ebmg.Problem(ctx, pr, **opts)
    rho = torch.tensor(pr.rho.ravel(), dtype=torch.float64, device=DEV)
    phi = torch.zeros_like(rho)
    torch.cuda.synchronize()
    st, info = P.solve(rho, phi, rtol=1e-10, max_cycles=30, check=False)
    tune = [P.tuning(q)[0] for q in range(P.levels)]
    P.release()
    return st, info, phi.cpu().numpy(), tune


CASES = [((65, 65, 65), None), ((67, 66, 65), 5.0), ((64, 65, 65), None), ((130, 130, 130), 3.0),
         ((1025, 1025), None), ((1031, 1027), 4.0)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("smoother", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("n,kappa", CASES)
def test_sweeps(ctx, n, kappa, smoother, prec):
    print("odd sweeps", n, kappa, smoother, prec, flush=True)
    pr, want, bar = _box(n, kappa)
    st, info, x, tune = _solve(ctx, pr, precision=prec, smoother=smoother, tail=1)
    err = np.linalg.norm(x - want.ravel()) / np.linalg.norm(want)
    print("   cycles", info["cycles"], "error", err, "sweeps", tune, flush=True)
    assert st == ebmg.OK and err <= bar, info


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("smoother", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("n,kappa", [((33, 35, 34), None), ((513, 511), None), ((50, 50, 50), 3.0)])
def test_three_sweeps(ctx, n, kappa, smoother, prec):
    """Three sweeps are more than a tile's halo holds."""
    print("odd, three sweeps", n, kappa, smoother, prec, flush=True)
    pr, want, bar = _box(n, kappa)
    st, info, x, tune = _solve(ctx, pr, precision=prec, smoother=smoother, tail=1, nu1=3, nu2=3)
    err = np.linalg.norm(x - want.ravel()) / np.linalg.norm(want)
    print("   cycles", info["cycles"], "error", err, "sweeps", tune, flush=True)
    assert st == ebmg.OK and err <= bar, info


@pytest.mark.parametrize("tail", [0, 1, 2])
@pytest.mark.parametrize("mode", [ebmg.BATCH_LEVELSYNC, ebmg.BATCH_PERSISTENT])
@pytest.mark.parametrize("prec", [0, 1])
def test_batches(ctx, prec, mode, tail):
    print("odd batch", prec, mode, tail, flush=True)
    probs = [W.two_disks(101, seed=3), W.two_disks(99, seed=1), W.two_disks(130, seed=2), W.two_disks(90, seed=4)]
    B = ebmg.Batch(ctx, probs, precision=prec, batch=mode, tail=tail)
    t = lambda a: torch.tensor(np.ascontiguousarray(a).ravel(), dtype=torch.float64, device=DEV)   # noqa: E731
    phi = [torch.zeros(n, dtype=torch.float64, device=DEV) for n, _ in B.sizes]
    phi2 = [torch.zeros(max(1, m), dtype=torch.float64, device=DEV) for _, m in B.sizes]
    rho, sig = [t(p.rho) for p in probs], [t(p.sigma) for p in probs]
    torch.cuda.synchronize()
    st, infos = B.solve(rho, phi, sigma=sig, phi2=phi2, rtol=1e-12, max_cycles=60, check=False)
    assert st == ebmg.OK, infos
    for p, x, x2, (n, m) in zip(probs, phi, phi2, B.sizes):
        S = assemble(p)
        y = np.concatenate([x.cpu().numpy(), x2.cpu().numpy()[:m]])
        xs = solve_splu(S.A, S.b)
        assert rel_residual(S.A, S.b, y) <= 1.01e-12
        assert np.linalg.norm(y - xs) / np.linalg.norm(xs) <= (1e-8 if prec else 1e-10)
    B.release()
