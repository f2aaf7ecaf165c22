"""The tuner times what a run uses: a problem that runs on chip with its automatic tiling still
does so with the tuned one, and with one from a cache file, whose entries were made off the chip
or name label groups that have no plan there."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1512_01383_amd as S  # noqa: E402
from tests.gpu_tilings import TILINGS  # noqa: E402


def _on_chip(prob, n):
    """Did a run of n iterations write rim words? (They lie behind the 11 k + 1 planes of the state
    and what iterations only read.)"""
    N = prob.H * prob.W
    plane = -(-N // 64) * 64 + (320 if -(-N // 64) * 64 % (1 << 18) == 0 else 0)
    before = prob.workspace.clone()
    prob.run(n)
    torch.cuda.synchronize()
    return int(torch.nonzero(prob.workspace != before).max()) >= (11 * prob.k + 1) * plane * 4


@pytest.mark.parametrize("H,Wd,L", [(256, 256, 20), (330, 360, 13), (200, 250, 5), (64, 64, 2)])
def test_tuned_runs_stay_on_chip(H, Wd, L):
    p = S.Problem.from_workload(W.truncated_quadratic(L=L, H=H, W=Wd, seed=81))
    assert _on_chip(p, 8) and not _on_chip(p, 7)
    assert p.autotune(iters=10) in TILINGS
    assert _on_chip(p, 8) and not _on_chip(p, 7)
    p.close()


def test_cached_tilings_keep_it_on_chip(tmp_path):
    """256x256, L = 20 has a plan with four label groups only."""
    wl = W.truncated_quadratic(L=20, H=256, W=256, seed=82)
    p = S.Problem.from_workload(wl)
    cache = tmp_path / "tiling.cache"
    p.autotune(iters=10, cache=str(cache))
    key, best = cache.read_text().strip().rsplit("|", 1)
    one_group = TILINGS.index((1, 4, 64))
    for line in (f"{key}|{one_group}", f"{key.replace(' chip=1', '')}|{one_group}"):
        cache.write_text(line + "\n")
        q = S.Problem.from_workload(wl)
        assert q.autotune(iters=10, cache=str(cache))[0] == 4
        assert _on_chip(q, 8)
        q.close()
    cache.write_text(f"{key}|{best}\n")
    assert p.autotune(iters=10, cache=str(cache)) == TILINGS[int(best)]   # read, not timed again
    assert cache.read_text() == f"{key}|{best}\n"
    p.close()


def test_a_problem_off_the_chip_keeps_its_cache_entries(tmp_path):
    wl = W.truncated_quadratic(L=16, H=600, W=600, seed=83)
    p = S.Problem.from_workload(wl)
    assert not _on_chip(p, 8)
    cache = tmp_path / "tiling.cache"
    t = p.autotune(iters=4, cache=str(cache))
    line = cache.read_text()
    assert "chip" not in line
    q = S.Problem.from_workload(wl)
    assert q.autotune(iters=4, cache=str(cache)) == t and cache.read_text() == line
    p.close()
    q.close()
