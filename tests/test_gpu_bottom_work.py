"""Device memory of the bottom inverse: a bottom of thousands of unknowns holds
its inverse and not the work arrays it was formed in, after the set-up and
after new coefficients, which still solve as a fresh problem does."""
import ctypes as C

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


def _bytes(P):
    by = C.c_int64()
    P.ctx.check(ebmg._lib.ebmg_query(P.h, None, None, None, C.byref(by)), "ebmg_query")
    return by.value


@pytest.mark.parametrize("n", [32, 33, 61])
def test_work_given_back(ctx, n):
    print("bottom work", n, flush=True)
    p1, p2 = W.eddington(2, n, 2.0, seed=3), W.eddington(2, n, 37.0, seed=4)
    P, Q = ebmg.Problem(ctx, p1, bottom_max_dof=4096), ebmg.Problem(ctx, p2, bottom_max_dof=4096)
    assert P.levels == 1
    dof = n * n
    # the inverse, and (up to 1024 unknowns) its work; beside them some 30 FP64 vectors at most
    most = 8 * dof * dof * (3 if dof <= 1024 else 1) + 300 * dof + (1 << 16)
    assert _bytes(P) <= most
    rho = torch.tensor(p2.rho.ravel(), dtype=torch.float64, device=DEV)
    out = []
    for A in (P, Q, P):
        if A is P:
            P.set_coefficients(p2)
            assert _bytes(P) <= most
        phi = torch.zeros(dof, dtype=torch.float64, device=DEV)
        torch.cuda.synchronize()
        A.solve(rho, phi, rtol=1e-11)
        out.append(phi.cpu().numpy())
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    P.release()
    Q.release()
