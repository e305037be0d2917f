"""Signed distances on lattices at the edges of the search's bricks: fewer
nodes than a brick, extents that leave remainders, and both brick sizes
(2048 * 64 nodes and one less row), against the brute-force oracle at sampled
nodes. 1e-12 as in the other mesh tests (the distance is evaluated in FP64 on
the closest triangle)."""
import numpy as np
import pytest

import workloads as W
from oracle.mesh_sdf import node_points, signed_distance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"

MESHES = {"cube": lambda: W.mesh_cube((0.47, 0.52, 0.5), 0.26),
          "sphere": lambda: W.mesh_icosphere((0.5, 0.46, 0.53), 0.31, subdiv=2),
          "pin": lambda: W.mesh_pin(r=0.05, nseg=16, nring=4, nz=6)}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


@pytest.mark.parametrize("n", [(1, 1, 1), (3, 3, 3), (4, 2, 5), (30, 9, 17), (63, 31, 62), (63, 31, 63), (64, 33, 65)])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_bricks(ctx, name, n):
    print("sdf bricks", name, n, flush=True)
    v, t = MESHES[name]()
    M = ebmg.Mesh(ctx, v, t)
    h, lo = 1.0 / max(n), (0.01, -0.02, 0.03)
    m = [k + 1 for k in n]
    out = torch.full((m[0] * m[1] * m[2] + 64,), np.nan, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    M.sdf(n, h, lo, out)
    got = out.cpu().numpy()
    assert np.isnan(got[-64:]).all() and np.isfinite(got[:-64]).all()
    got = got[:-64]
    P = node_points(n, h, lo)
    idx = np.unique(np.concatenate([np.random.default_rng(1).choice(len(P), size=min(len(P), 600), replace=False),
                                    [0, len(P) - 1, m[0] - 1, len(P) - m[0]]]))
    want = signed_distance(P[idx], v, t)
    assert np.abs(np.abs(got[idx]) - np.abs(want)).max() <= 1e-12
    far = np.abs(want) > 1e-9
    assert np.array_equal(np.sign(got[idx][far]), np.sign(want[far]))
    M.release()
