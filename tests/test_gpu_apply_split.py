"""The operator and the field straight from and into a caller's arrays: unaligned
arrays, outputs in front of and behind the inputs, and inputs and outputs that
share memory (staged), against the oracle's matrix and against each other
(bitwise: the same kernels)."""
import numpy as np
import pytest

import workloads as W
from oracle.operator import assemble

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ebmg = pytest.importorskip("paper_1809_03745_amd.ebmg", reason="libebmg.so not built")

DEV = "cuda:0"

CASES = {"two disks 40": lambda: W.two_disks(40, seed=2), "pin 20": lambda: W.pin_plane(20, seed=1),
         "pin 64 (z-marching)": lambda: W.pin_plane(64, seed=1), "plain 2d": lambda: W.manufactured_sine(33),
         "odd 3d 65": lambda: W.eddington(3, 65, 3.0, seed=1)}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ebmg.Context(0)


def _buf(n, shift, rng=None):
    t = torch.zeros(n + 8, dtype=torch.float64, device=DEV)[shift:shift + n]
    if rng is not None:
        t.copy_(torch.tensor(rng.normal(size=n), device=DEV))
    return t


@pytest.mark.parametrize("name", sorted(CASES))
def test_apply(ctx, name):
    print("apply split", name, flush=True)
    pr = CASES[name]()
    P = ebmg.Problem(ctx, pr)
    N, N2 = P.N, P.N2
    ref = x0 = None
    for shift in (0, 1):
        rng = np.random.default_rng(7)
        x, x2 = _buf(N, shift, rng), (_buf(N2, shift, rng) if N2 else None)
        y, y2 = _buf(N, 1 - shift), (_buf(N2, shift) if N2 else None)
        torch.cuda.synchronize()
        P.apply(x, x2, y, y2)
        got = torch.cat([y, y2]) if N2 else y.clone()
        xs = (torch.cat([x, x2]) if N2 else x).cpu().numpy()
        if ref is None:
            S = assemble(pr)
            want = S.A @ xs
            assert np.abs(got.cpu().numpy() - want).max() <= 4e-13 * np.abs(S.A).max() * np.abs(xs).max()
            ref, x0 = got, xs
        assert np.array_equal(xs, x0) and torch.equal(got, ref)
        # in place, and shifted by half an array over itself
        P.apply(x, x2, x, x2)
        assert torch.equal(torch.cat([x, x2]) if N2 else x, ref)
    big = _buf(2 * N, 0, np.random.default_rng(7))
    src = big[N // 2:N // 2 + N]
    src.copy_(torch.tensor(x0[:N], device=DEV))
    x2 = torch.tensor(x0[N:], device=DEV) if N2 else None
    y2 = _buf(N2, 0) if N2 else None
    torch.cuda.synchronize()
    P.apply(src, x2, big[:N], y2)
    assert torch.equal(torch.cat([big[:N], y2]) if N2 else big[:N], ref)
    P.release()


@pytest.mark.parametrize("name", sorted(CASES))
def test_efield(ctx, name):
    pr = CASES[name]()
    P = ebmg.Problem(ctx, pr)
    N, N2, D = P.N, P.N2, pr.dim
    rng = np.random.default_rng(3)
    x, x2 = _buf(N, 1, rng), (_buf(N2, 1, rng) if N2 else None)
    obj = np.linspace(-1.0, 2.0, len(pr.objects)) if pr.objects else None
    E = _buf(D * N, 0)
    torch.cuda.synchronize()
    P.efield(x, x2, E, obj_values=obj)
    # E over the input's memory
    big = _buf(D * N, 1)
    big[:N].copy_(x)
    torch.cuda.synchronize()
    P.efield(big[:N], x2, big, obj_values=obj)
    assert torch.equal(E, big)
    # the solve's own field of the same state (no cycles): bitwise
    phi, phi2, F = x.clone(), (x2.clone() if N2 else None), _buf(D * N, 0)
    tag, _, _ = P.level_arrays(0)
    cov = torch.tensor((tag & 3) == 3, device=DEV)
    phi[cov] = 0.0
    P.efield(phi, phi2, E, obj_values=obj)
    P.solve(torch.ones(N, dtype=torch.float64, device=DEV), phi, phi2=phi2, E=F, max_cycles=0, obj_values=obj,
            check=False)
    assert torch.equal(E, F)
    P.release()
