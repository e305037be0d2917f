"""The composite solve's graphs against direct launches: bitwise the same
iterates, on the first solve and on later ones with other sources and guesses,
with the program's own work and synchronisations between them."""
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


CASES = {
    "2d two boxes": lambda: W.amr_plain(2, 32, [(1, (8, 8), (16, 16)), (1, (40, 32), (20, 24)),
                                               (2, (88, 72), (16, 16))]),
    "3d, odd coarse levels": lambda: W.amr_plain(3, 34, [((20, 20, 28), (34, 30, 20))], alpha=1.0, a_gas=30.0),
    "pin": lambda: W.amr_pin_plane(32, 2, r_pin=0.05),
}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_graphs_equal_launches(ctx, name, prec):
    print("amr graphs", name, prec, flush=True)
    amr = CASES[name]()
    A = [ebmg.Amr(ctx, amr, precision=prec, smoother=4, tail=1, graphs=g) for g in (0, 1)]
    rng = np.random.default_rng(1)
    phi = [[torch.zeros(n, dtype=torch.float64, device=DEV) for n in a.N] for a in A]
    phi2 = [[torch.zeros(n, dtype=torch.float64, device=DEV) if n else None for n in a.N2] for a in A]
    for k in range(4):
        rho = [torch.tensor(rng.normal(size=n), dtype=torch.float64, device=DEV) for n in A[0].N]
        got = []
        for q, a in enumerate(A):
            if k != 2:   # the third solve starts from the second one's solution
                for x in phi[q] + phi2[q]:
                    if x is not None:
                        x.zero_()
            torch.cuda.synchronize()
            _, info = a.solve(rho, phi[q], phi2=phi2[q], max_iters=60)
            torch.cuda.synchronize()
            got.append((info, [x.clone() for x in phi[q] + phi2[q] if x is not None]))
        assert got[0][0]["outer_iters"] == got[1][0]["outer_iters"] and got[0][0]["rel_residual"] == got[1][0]["rel_residual"]
        for x, y in zip(got[0][1], got[1][1]):
            assert torch.equal(x, y)
    for a in A:
        a.release()
