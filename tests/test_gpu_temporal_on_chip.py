"""Two-iteration passes switched on for an image that fits the chip: runs of 24 iterations and more
go on chip (they write rim words, the passes do not), with the iterates of the passes bit for bit,
also where the automatic tiling has several label groups."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1512_01383_amd as S  # noqa: E402
from tests.test_gpu_autotune_on_chip import _on_chip  # noqa: E402


def _aniso(wl):
    wl.tv = S.TV_ANISO
    return wl


CASES = [("rof", W.rof(H=61, W=150)), ("rof_aniso", _aniso(W.rof(H=64, W=64, seed=45))),
         ("tq_k1", W.truncated_quadratic(L=2, H=521, W=513, seed=41)),
         ("tq_k2", W.truncated_quadratic(L=3, H=40, W=200, seed=42)),
         ("tq_k3", W.truncated_quadratic(L=4, H=40, W=70, seed=43)),
         ("periodic_k3", W.phase_unwrapping(seed=46, H=130, W=90, L=4))]


@pytest.mark.parametrize("n", [24, 31])
@pytest.mark.parametrize("name,wl", CASES, ids=[c[0] for c in CASES])
def test_long_runs_go_on_chip_with_the_same_iterates(name, wl, n):
    a, b = (S.Problem.from_workload(wl) for _ in range(2))
    st = S.pack_state(W.random_state(3, wl.k, wl.H, wl.W))
    for p in (a, b):
        p.set_temporal(True)
        p.load_state(st)
    assert _on_chip(a, n)
    for _ in range(n // 4):
        assert not _on_chip(b, 4)
    b.run(n % 4)
    assert torch.equal(a.save_state(), b.save_state())
    assert not _on_chip(a, 23)
    for p in (a, b):
        p.close()


def test_images_off_the_chip_keep_the_passes():
    wl = W.rof(H=2048, W=2048, seed=5)
    a, b = (S.Problem.from_workload(wl) for _ in range(2))
    a.set_temporal(True)
    assert not _on_chip(a, 48)
    b.run(48)
    assert torch.equal(a.save_state(), b.save_state())
    a.close()
    b.close()
