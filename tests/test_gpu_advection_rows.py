"""The z-marching advection step at the edges of its tiles (60 cells by 6 or 14
rows by 8 or 32 planes): one more and one less of each, single cells, both
block shapes, velocities of every sign and inflow on every face, with and
without cut cells; against the oracle, every cell. 1e-12 of the density scale,
as for one step in the other advection tests."""
import numpy as np
import pytest

import workloads as W
from oracle.advection import Advection

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


def _check(ctx, pr, rng):
    h = pr.h
    A = Advection(pr)
    P = ebmg.Problem(ctx, pr)
    n0 = np.where(A.gas, rng.uniform(0.5, 1.5, size=pr.shape), 0.0)
    u = []
    for d in range(3):
        shape = [pr.n[2 - a] + (1 if 2 - a == d else 0) for a in range(3)]
        u.append(rng.normal(size=shape))
    dt = 0.4 * h / max(float(np.abs(x).max()) for x in u)
    inflow = tuple(rng.uniform(0.5, 1.5, size=6))
    y = torch.full((pr.ncells,), np.nan, dtype=torch.float64, device=DEV)
    x, ut = _t(n0), [_t(v) for v in u]
    torch.cuda.synchronize()
    P.advect(x, ut, dt, y, inflow=inflow)
    ref = A.step(n0, u, dt, inflow)
    err = np.abs(y.cpu().numpy().reshape(pr.shape) - ref).max() / np.abs(n0).max()
    print("   max difference / scale", err, flush=True)
    assert err <= 1e-12
    P.release()


@pytest.mark.parametrize("n", [(1, 1, 1), (2, 3, 2), (59, 5, 7), (60, 6, 8), (61, 7, 9), (121, 13, 17), (5, 70, 33),
                               (63, 4, 66), (40, 16, 8320)])
def test_plain_box(ctx, n):
    print("advection rows", n, flush=True)
    pr = W.Problem(3, n, 1.0 / max(n), (0.0,) * 3, [], *W._bc(W.BC_DIRICHLET))
    _check(ctx, pr, np.random.default_rng(sum(n)))


@pytest.mark.parametrize("n", [(61, 15, 18), (64, 20, 33)])
def test_cut_cells(ctx, n):
    print("advection rows, sphere", n, flush=True)
    h = 1.0 / max(n)
    Xn = W._nodes(3, n, h, (0.0,) * 3)
    c = tuple(0.5 * m * h for m in n)
    sphere = W.Obj(W.OBJ_ELECTRODE, 1.0, np.ascontiguousarray(W.sdf_sphere(Xn, c, 0.3 * min(n) * h)))
    pr = W.Problem(3, n, h, (0.0,) * 3, [sphere], *W._bc(W.BC_DIRICHLET))
    _check(ctx, pr, np.random.default_rng(sum(n)))
