"""An on-chip run whose tiles give up waiting for each other: whoever reads its result is told.
The limit of the wait is set to nothing from the host, so that a wave which does not find its
neighbour's word at the first look gives up at once; in a launch of some hundred blocks, which
do not start at the same moment, some do. Every wave still ends normally."""
import ctypes as C

import pytest

import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1512_01383_amd as S  # noqa: E402

DEVICE_ERROR = 3


def _limit(prob, looks):
    f = S.lib().slx_set_wait_limit
    f.argtypes, f.restype = [C.c_void_p, C.c_uint], None
    f(prob.h, looks)


def _refused(call, *args):
    with pytest.raises(S.SublabelError) as e:
        call(*args)
    assert e.value.status == DEVICE_ERROR, e.value


@pytest.mark.parametrize("tv", [0, 1])
@pytest.mark.parametrize("storage", ["fp32", "bf16"])
def test_a_lost_state_is_reported_until_another_is_loaded(storage, tv):
    wl = W.truncated_quadratic(L=5, H=256, W=256, seed=61)
    wl.tv = tv
    good = S.Problem.from_workload(wl, storage=storage)
    good.run(40)
    start = good.save_state()
    good.run(24)
    want = good.save_state()
    p = S.Problem.from_workload(wl, storage=storage)
    p.run(40)
    _limit(p, 0)
    p.run(200)
    p.run(5)        # single launches do not bring the state back, nor does another on-chip run
    p.run(50)
    lifted, u = p.read_u()
    assert torch.isnan(lifted).all() and torch.isnan(u).all()
    assert torch.isnan(p.save_state()).all()
    _refused(p.energy)
    _refused(p.residuals)
    _refused(p.run_to_gap, 1e-3, 100)
    p.load_state(start)
    p.run(24)       # off the chip from here on
    assert torch.equal(p.save_state(), want)
    assert p.energy()["primal_ub"] == good.energy()["primal_ub"]
    p.close()
    good.close()


@pytest.mark.parametrize("adaptive", [True, False])
def test_a_solve_that_gives_up_returns_an_error(adaptive):
    p = S.Problem.from_workload(W.rof(H=700, W=700), adaptive=adaptive)
    _limit(p, 0)
    _refused(p.run_to_gap, 1e-3, 400)
    p.close()


def test_a_replay_that_gives_up_returns_no_gradients():
    wl = W.truncated_quadratic(L=5, H=256, W=256, seed=62)
    p = S.Problem.from_workload(wl)
    p.unrolled_forward(60, 30)
    u = p.read_u()[1]
    assert torch.isfinite(u).all()
    _limit(p, 0)
    _refused(p.unrolled_backward, u)
    p.close()
