"""Column blockings of the Legendre kernels that no power of two gives: odd
numbers of 16-column blocks per tile, whose right-hand operand is filled by
overlapping pieces and read in mixed vector widths.  The blocking is forced
through the autotuner's cache line, or follows from the plan's own rule
(generated P~).  Oracle on the first, a middle and the last field; bounds as
for every parity test (FP64 1e-12, FP32-data forms 1e-6)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from paper_1711_11296_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-6, "bf16x6": 1e-6}


def _rel(x, ref):
    return np.linalg.norm(x - ref) / np.linalg.norm(ref)


def _check(p, N, J, I, F, kind, form):
    dt = torch.float64 if form == "fp64" else torch.float32
    pick = [0, F // 2, F - 1]
    g = torch.from_numpy(inputs.random_grid(F, J, I, seed=F)).to("cuda:0", dt)
    s = p.forward(g)
    a = torch.from_numpy(inputs.random_spectra(N, F, seed=F + 1, profile="white")).to("cuda:0", dt)
    x = p.inverse(a)
    torch.cuda.synchronize()
    assert _rel(s[pick].double().cpu().numpy(), O.forward(g[pick].double().cpu().numpy(), N, kind)) < TOL[form]
    assert _rel(x[pick].double().cpu().numpy(), O.inverse(a[pick].double().cpu().numpy(), N, J, I, kind)) < TOL[form]


@pytest.mark.parametrize("form,k", [("fp32", 3), ("fp32", 5), ("fp32", 6), ("fp32", 7), ("fp32", 9),
                                    ("fp64", 3), ("fp64", 5), ("fp64", 6), ("fp64", 7),
                                    ("bf16x6", 3), ("bf16x6", 5), ("bf16x6", 6), ("bf16x6", 7)])
def test_forced_blocking(form, k, tmp_path, monkeypatch):
    from paper_1711_11296_amd import Plan
    N, J, I = 140, 101, 288  # more than one 128-row tile, four blocks of 16 latitudes or two of 32
    for F in (8 * k - 5, 8 * k, 16 * k - 3, 24 * k - 7):
        cache = tmp_path / ("tune%d.txt" % F)
        monkeypatch.setenv("SHT_TUNE_CACHE", str(cache))
        Plan(N, J, I, F, grid="fejer2", form=form, autotune=True).close()
        key = cache.read_text().splitlines()[0].split("|")[0]
        if int(key.split(",")[-1]) % (16 * k) == 0:  # the row length that this plan chose takes tiles of k blocks
            break
    else:
        pytest.fail("no field count with rows of %d-block tiles" % k)
    # the analysis of FP32 data takes up to 10 blocks, the synthesis 8
    cache.write_text("%s|%d 0 %d 0 1 1\n" % (key, k, k if k <= 8 else 1))
    p = Plan(N, J, I, F, grid="fejer2", form=form, autotune=True)
    assert len(cache.read_text().splitlines()) == 1  # the line was admissible and used
    _check(p, N, J, I, F, "fejer2", form)
    p.close()


@pytest.mark.parametrize("form", ["fp32", "fp64", "bf16x6"])
@pytest.mark.parametrize("F", [24, 51])
def test_generated_odd_blocking(form, F):
    from paper_1711_11296_amd import Plan
    N, J, I = 200, 65, 432
    p = Plan(N, J, I, F, grid="cc_poles", form=form, otf=True)
    _check(p, N, J, I, F, "cc_poles", form)
    p.close()
