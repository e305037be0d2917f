"""What the coarse-tail tuner times is what solves run: on a problem whose
levels all take the one-launch V-cycle sides, the set-up's V-cycles launch
those (and the one-workgroup engine's candidates), never a level's colour
phases, and neither do the solves. smoother = 4 takes no timing of its own."""
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


def _kernels(fn):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    return sorted({e.name for e in prof.events() if "ebmg" in e.name or "GraphLaunch" in e.name})


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("make", [lambda: W.manufactured_sine(64), lambda: W.two_disks(64, seed=1),
                                  lambda: W.eddington(3, 16, 3.0, seed=1)], ids=["sine", "disks", "eddington3d"])
def test_tuner_times_the_solve_s_cycles(ctx, make, prec):
    print("tail choice", prec, flush=True)
    pr, held = make(), []
    names = _kernels(lambda: held.append(ebmg.Problem(ctx, pr, precision=prec, smoother=4)))
    P = held[0]
    print("   levels", P.levels, "choice", P.tuning(-1), flush=True)
    assert any("k_tile" in n for n in names), names
    assert any("k_tail_vcycle" in n for n in names), names
    assert not [n for n in names if "k_rb" in n], names
    rho = torch.ones(P.N, dtype=torch.float64, device=DEV)
    phi, phi2 = torch.zeros_like(rho), torch.zeros(max(1, P.N2), dtype=torch.float64, device=DEV)
    names = _kernels(lambda: P.solve(rho, phi, phi2=phi2 if P.N2 else None))
    assert any("k_tile" in n or "k_tail_vcycle" in n for n in names), names
    assert not [n for n in names if "k_rb" in n], names
    P.release()


@pytest.mark.parametrize("graphs", [0, 1])
def test_tuner_replays_graphs_where_solves_do(ctx, graphs):
    pr, held = W.eddington(3, 32, 5.0, seed=1), []
    setup = _kernels(lambda: held.append(ebmg.Problem(ctx, pr, precision=1, smoother=4, graphs=graphs)))
    P = held[0]
    rho = torch.ones(P.N, dtype=torch.float64, device=DEV)
    phi = torch.zeros_like(rho)
    solve = _kernels(lambda: P.solve(rho, phi))
    P.release()
    replays = [any("GraphLaunch" in n for n in names) for names in (setup, solve)]
    assert replays == [graphs == 0, graphs == 0], (setup, solve)
