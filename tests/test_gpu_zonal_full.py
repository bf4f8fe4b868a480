"""Group and register-held zonal kernels with the whole spectrum: N = (I - 1)
/ 2, so that every wavenumber a thread can hold is filled and no bin near I /
2 is left to zero, on rows that span more than one 32-row workspace block
where the oracle's time allows it; and levels of few items, which the group
kernels take too.  All four directions for the shorter rows, oracle on the
first and last field; bounds as for every parity test."""

import functools

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-6}


def _rel(x, ref):
    return np.linalg.norm(x - ref) / np.linalg.norm(ref)


@functools.lru_cache(maxsize=2)
def _case(N, J, I, F, kind, adjoints):
    """FP32-valued inputs of both forms and the oracle's results for fields 0
    and F - 1."""
    gen = torch.Generator().manual_seed(I + N)
    g = torch.randn((F, J, I), generator=gen)
    a = torch.randn((F, (N + 1) * (N + 2) // 2, 2), generator=gen)
    a[:, :N + 1, 1] = 0
    pick = sorted({0, F - 1})
    gh, ah = g[pick].double().numpy(), a[pick].double().numpy()
    ref = [O.forward(gh, N, kind), O.inverse(ah, N, J, I, kind)]
    if adjoints:
        ref += [O.inverse_adjoint(gh, N, kind), O.forward_adjoint(ah, N, J, I, kind)]
    return g, a, pick, ref


def _check(N, J, I, F, form, kind="fejer2", adjoints=True):
    from paper_1711_11296_amd import Plan
    g, a, pick, ref = _case(N, J, I, F, kind, adjoints)
    dt = torch.float64 if form == "fp64" else torch.float32
    g, a = g.to("cuda:0", dt), a.to("cuda:0", dt)
    p = Plan(N, J, I, F, grid=kind, form=form, otf=True)
    out = [p.forward(g), p.inverse(a)]
    if adjoints:
        out += [p.inverse_adjoint(g), p.forward_adjoint(a)]
    torch.cuda.synchronize()
    for x, r in zip(out, ref):
        assert _rel(x[pick].double().cpu().numpy(), r) < TOL[form]
    p.close()


# 11 fields: a partial last group of every group size
@pytest.mark.parametrize("form", ["fp32", "fp64"])
@pytest.mark.parametrize("I,J", [(480, 67), (800, 67), (1024, 67), (1280, 35), (1440, 9), (1920, 9), (2160, 5),
                                 (2880, 5)])
def test_whole_spectrum(form, I, J):
    _check((I - 1) // 2, J, I, 11, form, adjoints=I <= 1024)


# few items and partly or mostly empty groups
@pytest.mark.parametrize("form", ["fp32", "fp64"])
@pytest.mark.parametrize("I,N,J,F", [(288, 100, 40, 1), (400, 133, 64, 8), (480, 160, 65, 1), (960, 320, 71, 3),
                                     (1600, 533, 34, 20), (2400, 799, 9, 2), (3600, 600, 12, 5)])
def test_few_items(form, I, N, J, F):
    _check(N, J, I, F, form, kind="cc_poles", adjoints=I < 960)


# FP64 synthesis at 2880 with items for more than one round (17 row pairs: 510
# items of 2 fields), few and many wavenumbers
@pytest.mark.parametrize("N", [300, 1023])
def test_long_rows(N):
    _check(N, 33, 2880, 60, "fp64", adjoints=N < 1000)
