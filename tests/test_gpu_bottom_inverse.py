"""The dense bottom inverse formed on the device: systems that are one level
(bottom_max_dof at least their size), so that a solve is one application of
the inverse, over the panel widths and the remainders of panels and tiles.
One cycle has to reach 1e-11 relative residual (the inverse of a matrix of
condition below 1e4 leaves a few 1e-13), and the oracle's solution to 1e-10."""
import dataclasses

import numpy as np
import pytest

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


def _t(a):
    return torch.tensor(np.ascontiguousarray(a).ravel(), dtype=torch.float64, device=DEV)


def plain(nx, ny):
    rho = np.random.default_rng(nx).normal(size=(ny, nx))
    return W.Problem(2, (nx, ny), 1.0 / max(nx, ny), (0.0, 0.0), [], [W.BC_DIRICHLET] * 6, [0.0] * 6, [0.0] * 6,
                     [1.0] * 6, rho=rho, name=f"plain-{nx}x{ny}")


# unknowns: 1, 6, 31, 32, 33 | 992, 1024 (one panel row a thread) | 1025, 2048 (two) | 2050, 4096 (four)
PLAIN = [(1, 1), (2, 3), (1, 31), (4, 8), (3, 11), (31, 32), (32, 32), (25, 41), (32, 64), (41, 50), (64, 64)]


@pytest.mark.parametrize("nx,ny", PLAIN)
def test_plain_box(ctx, nx, ny):
    print("bottom inverse", nx, ny, flush=True)
    pr = plain(nx, ny)
    S = assemble(pr)
    xs = solve_splu(S.A, S.b)
    P = ebmg.Problem(ctx, pr, bottom_max_dof=4096)
    assert P.levels == 1
    phi = torch.zeros(P.N, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    st, info = P.solve(_t(pr.rho), phi, rtol=1e-11, max_cycles=1, check=False)
    x = phi.cpu().numpy()
    assert st == ebmg.OK and info["cycles"] == 1
    assert rel_residual(S.A, S.b, x) <= 1e-11
    assert np.linalg.norm(x - xs) <= 1e-10 * np.linalg.norm(xs)
    P.release()


CUT = {"two disks 32": lambda: W.two_disks(32, seed=3), "blade 48": lambda: W.blade_plane(48, seed=1),
       "pin 12": lambda: W.pin_plane(12, seed=1, r_pin=0.12, blob_sigma=(0.06, 0.1), nblob=1),
       "eddington 3d 9": lambda: W.eddington(3, 9, 4.0, seed=2)}


@pytest.mark.parametrize("name", sorted(CUT))
def test_cut_cells(ctx, name):
    """Rows with wide, nonsymmetric stencils, second-phase unknowns and
    identity rows of covered cells."""
    pr = CUT[name]()
    S = assemble(pr)
    xs = solve_splu(S.A, S.b)
    P = ebmg.Problem(ctx, pr, bottom_max_dof=4096, krylov=ebmg.KRYLOV_NONE)
    assert P.levels == 1
    phi = torch.zeros(P.N, dtype=torch.float64, device=DEV)
    phi2 = torch.zeros(max(1, P.N2), dtype=torch.float64, device=DEV)
    sig = _t(pr.sigma) if pr.sigma is not None else None
    torch.cuda.synchronize()
    st, info = P.solve(_t(pr.rho), phi, sigma=sig, phi2=phi2 if P.N2 else None, rtol=1e-11, max_cycles=1,
                       check=False)
    x = np.concatenate([phi.cpu().numpy(), phi2.cpu().numpy()[:P.N2]])
    assert st == ebmg.OK and info["cycles"] == 1
    assert np.linalg.norm(x - xs) <= 1e-10 * np.linalg.norm(xs)
    P.release()


def test_new_coefficients(ctx):
    """The inverse formed again for new coefficients equals a fresh setup's, bitwise."""
    p1, p2 = W.eddington(2, 24, 2.0, seed=1), W.eddington(2, 24, 50.0, seed=2)
    P, Q = ebmg.Problem(ctx, p1, smoother=4, tail=1), ebmg.Problem(ctx, p2, smoother=4, tail=1)
    out = []
    for prob, new in ((P, True), (Q, False)):
        for _ in range(2 if new else 1):
            if new:
                prob.set_coefficients(p1)
                prob.set_coefficients(p2)
            phi = torch.zeros(prob.N, dtype=torch.float64, device=DEV)
            torch.cuda.synchronize()
            prob.solve(_t(p2.rho), phi, rtol=1e-10)
            out.append(phi.cpu().numpy())
    assert all(np.array_equal(out[0], o) for o in out[1:])
    P.release()
    Q.release()


@pytest.mark.parametrize("nx,ny", PLAIN[1:])
def test_plain_box_with_pivots(ctx, nx, ny):
    """A negative mass (above the lowest eigenvalue's) takes the diagonal below
    the off-diagonal sum, so that pivots are searched."""
    print("bottom inverse with pivots", nx, ny, flush=True)
    pr = dataclasses.replace(plain(nx, ny), alpha=1.0, a_gas=-3.0, a_diel=-3.0)
    S = assemble(pr)
    A = abs(S.A)
    assert min(nx, ny) < 8 or (A.sum(axis=1).A1 - 2 * A.diagonal()).max() > 0
    xs = solve_splu(S.A, S.b)
    P = ebmg.Problem(ctx, pr, bottom_max_dof=4096)
    assert P.levels == 1
    phi = torch.zeros(P.N, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    st, info = P.solve(_t(pr.rho), phi, rtol=1e-11, max_cycles=1, check=False)
    assert st == ebmg.OK and info["cycles"] == 1
    assert np.linalg.norm(phi.cpu().numpy() - xs) <= 1e-10 * np.linalg.norm(xs)
    P.release()
