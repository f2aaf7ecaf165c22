"""Runs that are no faster on chip stay off it: kernels that are not built, and runs too short for
the cost of the launch (fewer than 8 iterations, or than 16 for many labels and rows per thread)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1512_01383_amd as S  # noqa: E402
from tests.test_gpu_autotune_on_chip import _on_chip  # noqa: E402


def _problem(H, Wd, L, add, groups, storage="fp32"):
    rng = np.random.Generator(np.random.PCG64(91))
    wl = W.Workload("quad", H, Wd, W.equispaced(L), W.QUAD, 0.2, f=rng.uniform(0.0, 1.0, (H, Wd)).astype(np.float32))
    if add:
        wl.tau = wl.gamma.copy()
        wl.samples = rng.normal(0.0, 0.02, (L, H, Wd)).astype(np.float32)
    p = S.Problem.from_workload(wl, storage=storage)
    assert p.get_tiling()[0] == groups   # the automatic tiling
    return p


@pytest.mark.parametrize("storage", ["fp32", "bf16"])
@pytest.mark.parametrize("H,Wd,L,add,groups", [(1501, 192, 7, False, 1), (1001, 320, 7, False, 1),
                                               (701, 256, 10, True, 2), (400, 400, 11, True, 2)])
def test_kernels_that_are_no_faster_are_not_used(H, Wd, L, add, groups, storage):
    p = _problem(H, Wd, L, add, groups, storage)
    assert not _on_chip(p, 60)
    p.close()


@pytest.mark.parametrize("H,Wd,L,storage,least",
                         [(1399, 322, 5, "fp32", 16), (1399, 514, 4, "fp32", 16), (1399, 514, 4, "bf16", 16),
                          (1501, 192, 6, "fp32", 8), (1501, 192, 6, "bf16", 16), (999, 1026, 3, "bf16", 8),
                          (701, 642, 5, "bf16", 8), (64, 64, 2, "fp32", 8)])
def test_short_runs_stay_off_the_chip(H, Wd, L, storage, least):
    p = _problem(H, Wd, L, False, 1, storage)
    assert not _on_chip(p, least - 1)
    assert _on_chip(p, least)
    p.close()
