"""Signed distances next to a mesh of slivers (a unit-length prism and a plate
1e-5 and 1e-6 thick, at an angle to the axes), whose face parameters are
ill-conditioned: the distance is never more than the distance to the nearest
edge of the mesh, which point-segment arithmetic gives to rounding (1e-12 for
coordinates of order one)."""
import numpy as np
import pytest

from oracle.mesh_sdf import node_points

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


def _extruded(outline, z0, z1):
    """Triangles of a convex outline (m, 2) extruded along an oblique axis."""
    ax = np.array([0.3, 0.5, 0.8]) / np.linalg.norm([0.3, 0.5, 0.8])
    u = np.array([ax[1], -ax[0], 0.0]) / np.hypot(ax[0], ax[1])
    frame = np.stack([u, np.cross(ax, u), ax])
    m = len(outline)
    v = np.concatenate([np.column_stack([outline, np.full(m, z)]) for z in (z0, z1)]) @ frame + 0.5
    t = []
    for j in range(m):
        n = (j + 1) % m
        t += [(j, n, m + n), (j, m + n, m + j)]
    for j in range(1, m - 1):
        t += [(0, j + 1, j), (m, m + j, m + j + 1)]
    return v, np.array(t, dtype=np.int32)


def prism(w):
    a = 2 * np.pi * np.arange(6) / 6
    return _extruded(w * np.column_stack([np.cos(a), np.sin(a)]), -0.5, 0.5)


def plate(w):
    return _extruded(np.array([(-0.5, -0.5), (0.5, -0.5), (0.5, 0.5), (-0.5, 0.5)]), -0.5 * w, 0.5 * w)


def _edge_distance(P, v, t):
    d = np.full(len(P), np.inf)
    for a, b in {tuple(sorted((int(q[j]), int(q[(j + 1) % 3])))) for q in t for j in range(3)}:
        e, w = v[b] - v[a], P - v[a]
        q = w - np.clip((w @ e) / (e @ e), 0.0, 1.0)[:, None] * e
        d = np.minimum(d, np.sqrt((q * q).sum(1)))
    return d


@pytest.mark.parametrize("w", [1e-3, 1e-5, 1e-6])
@pytest.mark.parametrize("make", [prism, plate])
def test_never_beyond_the_nearest_edge(ctx, make, w):
    print("sdf slivers", make.__name__, w, flush=True)
    v, t = make(w)
    M = ebmg.Mesh(ctx, v, t)
    n, h = (16, 16, 16), 1e-6
    out = torch.zeros(17 ** 3, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    worst = -np.inf
    for spot in range(24):
        q = v[t[spot % len(t)]]
        s = 0.5 + 0.43 * np.sin(1.0 + spot)
        lo = q[0] + s * (q[1] - q[0]) + 0.5 * (1 - s) * (q[2] - q[0]) - 8e-6
        M.sdf(n, h, lo, out)
        worst = max(worst, float((np.abs(out.cpu().numpy()) - _edge_distance(node_points(n, h, lo), v, t)).max()))
    print("   beyond the nearest edge by", worst, flush=True)
    assert worst <= 1e-12
    M.release()
