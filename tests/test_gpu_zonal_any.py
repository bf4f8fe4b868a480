"""Row lengths without a compile-time plan: one to five passes, every radix,
rows that are not whole 16-byte vectors, lengths of few and of many items per
workgroup, and field counts around the group sizes.  Oracle on every field
for the small cases, on the first and last otherwise; bounds as for every
parity test."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from paper_1711_11296_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-6}


def _rel(x, ref):
    return np.linalg.norm(x - ref) / np.linalg.norm(ref)


# (I, N, J, F): radices 2..16, odd lengths (scalar rows), 4 and 5 passes, N at (I - 1) / 2, a zonal mean only
SHAPES = [
    (1, 0, 3, 2), (2, 0, 4, 1), (4, 1, 6, 3), (6, 2, 5, 9), (16, 7, 17, 5), (20, 9, 21, 1), (45, 22, 45, 2),
    (54, 20, 41, 17), (81, 40, 33, 4), (90, 44, 40, 8), (125, 62, 30, 3), (128, 63, 127, 33), (135, 60, 25, 16),
    (240, 79, 160, 12), (243, 121, 21, 5), (256, 85, 171, 7), (512, 170, 40, 19), (625, 300, 9, 3), (720, 30, 61, 41),
    (750, 374, 8, 6), (768, 383, 9, 9), (1024, 511, 12, 5), (1250, 100, 11, 4), (1280, 639, 10, 9),
    (1536, 500, 9, 6), (2000, 40, 21, 3), (2048, 350, 6, 2), (2187, 50, 15, 2), (3072, 20, 33, 7), (3125, 30, 13, 3),
    (3240, 401, 5, 1), (4096, 25, 21, 9),
]


@pytest.mark.parametrize("form", ["fp32", "fp64"])
@pytest.mark.parametrize("I,N,J,F", SHAPES)
def test_lengths(I, N, J, F, form):
    from paper_1711_11296_amd import Plan
    dt = torch.float64 if form == "fp64" else torch.float32
    p = Plan(N, J, I, F, grid="fejer2", form=form)
    pick = sorted({0, F // 2, F - 1})
    g = torch.from_numpy(inputs.random_grid(F, J, I, seed=I)).to("cuda:0", dt)
    a = torch.from_numpy(inputs.random_spectra(N, F, seed=I + 1, profile="white")).to("cuda:0", dt)
    s, x = p.forward(g), p.inverse(a)
    xb, sb = p.forward_adjoint(a), p.inverse_adjoint(g)
    torch.cuda.synchronize()
    gh, ah = g[pick].double().cpu().numpy(), a[pick].double().cpu().numpy()
    host = lambda t: t[pick].double().cpu().numpy()  # noqa: E731
    assert _rel(host(s), O.forward(gh, N, "fejer2")) < TOL[form]
    assert _rel(host(x), O.inverse(ah, N, J, I, "fejer2")) < TOL[form]
    assert _rel(host(xb), O.forward_adjoint(ah, N, J, I, "fejer2")) < TOL[form]
    assert _rel(host(sb), O.inverse_adjoint(gh, N, "fejer2")) < TOL[form]
    p.close()
