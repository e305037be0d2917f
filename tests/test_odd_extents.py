"""Hierarchies whose extents turn odd above the bottom level: coarsening goes
on to (n + 1) / 2 cells, the last over one fine cell. The hierarchy and its
rebuild for new coefficients on the CPU; solves against the oracle, with the
grid-wide cycle and the one-workgroup engine, on the GPU. Bars as in the other
parity tests (FP64 1e-10, mixed 1e-8 relative L2)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle.operator import assemble
from oracle.solvers import rel_residual, solve_splu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"


def ragged_pin(n):
    """The pin-plane gap cut to an n[0] x n[1] x n[2] box of its lower corner region."""
    full = W.pin_plane(max(n), seed=2)
    objs = [dataclasses.replace(o, sdf=np.ascontiguousarray(o.sdf[:n[2] + 1, :n[1] + 1, :n[0] + 1]))
            for o in full.objects]
    rho = np.ascontiguousarray(full.rho[:n[2], :n[1], :n[0]])
    return dataclasses.replace(full, n=n, objects=objs, rho=rho, bc_kind=[W.BC_DIRICHLET] * 6,
                               bc_value=[0.0] * 6, name=f"ragged-pin-{n}")


CASES = {
    "sine 50 (25 = odd at level 1)": lambda: W.manufactured_sine(50),
    "sine 99 (odd at every level)": lambda: W.manufactured_sine(99),
    "sine 150 (75 = odd at level 1)": lambda: W.manufactured_sine(150),
    "eddington 2d 77": lambda: W.eddington(2, 77, 3.0, seed=1),
    "eddington 3d 21": lambda: W.eddington(3, 21, 9.0, seed=1),
    "two disks 101": lambda: W.two_disks(101, seed=3),
    "two disks 90": lambda: W.two_disks(90, seed=3),
    "two disks 150": lambda: W.two_disks(150, seed=3),
    "pin 21 x 24 x 22": lambda: ragged_pin((21, 24, 22)),
}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


@pytest.mark.parametrize("name", sorted(CASES))
def test_hierarchy_reaches_a_small_bottom(name):
    P = ebmg.Problem(ebmg.Context(-1), CASES[name]())
    # a first odd level of at most 4096 unknowns is the bottom; past one, coarsening goes on
    ext = CASES[name]().n[0]
    assert sum(P.level_size(P.levels - 1)) <= (600 if ext in (99, 150, 77, 21, 101) else 4096)
    for lev in range(P.levels):
        tag, prim, _ = P.level_arrays(lev)
        A = P.operator(lev)
        assert np.all(A.diagonal()[:len(tag)][prim >= 0] > 0)


@pytest.mark.parametrize("dim,n", [(2, 50), (2, 51), (2, 130), (2, 150), (3, 18), (3, 27), (3, 34)])
def test_new_coefficients_equal_new_setup(dim, n):
    """Explicit rows on coarse levels (odd extents) are rebuilt too."""
    c = ebmg.Context(-1)
    p2 = W.eddington(dim, n, 37.0, seed=3)
    P, Q = ebmg.Problem(c, W.eddington(dim, n, 2.0, seed=3)), ebmg.Problem(c, p2)
    P.set_coefficients(p2)
    assert P.levels == Q.levels
    for lev in range(P.levels):
        assert (P.operator(lev) != Q.operator(lev)).nnz == 0


def test_pure_coarse_rows_are_symmetric():
    """A plain box: every level's rows come from one flux per face."""
    P = ebmg.Problem(ebmg.Context(-1), W.manufactured_sine(99))
    for lev in range(P.levels):
        A = P.operator(lev)
        assert abs(A - A.T).max() <= 1e-12 * abs(A).max()


def _solve(P, pr, rtol):
    t = lambda a: torch.tensor(np.ascontiguousarray(a).ravel(), dtype=torch.float64, device=DEV)   # noqa: E731
    phi = torch.zeros(P.N, dtype=torch.float64, device=DEV)
    phi2 = torch.zeros(max(P.N2, 1), dtype=torch.float64, device=DEV)
    sig = t(pr.sigma) if pr.sigma is not None else None
    st, info = P.solve(t(pr.rho), phi, sigma=sig, phi2=phi2 if P.N2 else None, rtol=rtol, max_cycles=60, check=False)
    return st, info, np.concatenate([phi.cpu().numpy(), phi2.cpu().numpy()[:P.N2]])


@pytest.mark.gpu
@pytest.mark.parametrize("tail", [1, 2])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_solve_parity(ctx, name, prec, tail):
    print("odd extents", name, prec, tail, flush=True)
    pr = CASES[name]()
    S = assemble(pr)
    xs = solve_splu(S.A, S.b)
    P = ebmg.Problem(ctx, pr, precision=prec, tail=tail)
    st, info, x = _solve(P, pr, 1e-12)
    assert st == ebmg.OK, info
    assert rel_residual(S.A, S.b, x) <= 1.01e-12
    err = np.linalg.norm(x - xs) / np.linalg.norm(xs)
    print("   levels", P.levels, "cycles", info["cycles"], "error", err, flush=True)
    assert err <= (1e-10 if prec == 0 else 1e-8)
    P.release()


@pytest.mark.gpu
def test_new_coefficients_solve(ctx):
    """A resident odd box re-coefficiented solves as a fresh one, bitwise."""
    p1, p2 = W.eddington(2, 75, 2.0, seed=3), W.eddington(2, 75, 37.0, seed=4)
    for prec in (0, 1):
        P = ebmg.Problem(ctx, p1, precision=prec, smoother=4, tail=1)
        Q = ebmg.Problem(ctx, p2, precision=prec, smoother=4, tail=1)
        _solve(P, p1, 1e-10)
        P.set_coefficients(p2)
        a, b = _solve(P, p2, 1e-10), _solve(Q, p2, 1e-10)
        assert a[0] == b[0] == ebmg.OK and np.array_equal(a[2], b[2])
        P.release()
        Q.release()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [0, 1])
def test_thin_box_keeps_the_krylov_bottom(ctx, prec):
    """A 6 x 2800 strip coarsens once, to 3 x 1400 (fewer than four cells across),
    which is too large for an inverse: BiCGStab on the bottom level."""
    n = (6, 2800)
    h = 1.0 / 2800
    k = [W.BC_DIRICHLET] * 6
    rho = np.random.default_rng(0).normal(size=(n[1], n[0]))
    pr = W.Problem(2, n, h, (0.0, 0.0), [], k, [0.0] * 6, [0.0] * 6, [1.0] * 6, rho=rho, name="strip")
    S = assemble(pr)
    xs = solve_splu(S.A, S.b)
    P = ebmg.Problem(ctx, pr, precision=prec)
    assert P.levels == 2 and P.level_size(1)[0] > 4096
    st, info, x = _solve(P, pr, 1e-12)
    assert st == ebmg.OK
    assert np.linalg.norm(x - xs) <= (1e-10 if prec == 0 else 1e-8) * np.linalg.norm(xs)
    P.release()
