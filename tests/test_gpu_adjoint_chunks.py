"""The adjoint's dual kernel with every number of label chunks per pixel (1, 2, 4, 8, chosen by the
image's size), for straddling intervals done after the label walk. GPU only.

Three iterations reach three rows and their adjoint three more, so the gradients of the first rows
of a tall image equal those of the same rows of its top strip, which the FP64 oracle can do. The
tolerances are those of the oracle comparison of gradients at other sizes: 1e-3 in relative L2,
every entry within 1e-2 of the largest (FP32 may pick the neighbouring part of a graph).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1512_01383_amd as S  # noqa: E402

K, STRIP, ROWS, WIDTH = 3, 16, 6, 513


def _workload(H, L, add):
    wl = W.truncated_quadratic(L=L, H=H, W=WIDTH, seed=21)
    if add:
        wl.tau = wl.gamma.copy()
        wl.samples = np.random.default_rng(22).normal(0, 0.02, (L, H, WIDTH)).astype(np.float32)
    return wl


def _top(wl, L, add):
    top = _workload(STRIP, L, add)
    top.f = np.ascontiguousarray(wl.f[:STRIP])
    if add:
        top.samples = np.ascontiguousarray(wl.samples[:, :STRIP])
    return top


@pytest.mark.parametrize("add", [True, False])
@pytest.mark.parametrize("H,L", [(16, 10), (17, 4), (140, 3), (140, 7), (260, 6), (512, 5)])
def test_first_rows_match_the_oracle(orc, H, L, add):
    wl = _workload(H, L, add)
    top = _top(wl, L, add)
    g = np.random.default_rng(23).uniform(0, 1, (H, WIDTH)).astype(np.float32)
    p = S.Problem.from_workload(wl)
    p.unrolled_forward(K, 2)
    _, u = p.read_u()
    gu = 2.0 * (u - torch.as_tensor(g, device=u.device))
    gf, _, gw = p.unrolled_backward(gu)
    o = orc.Problem(top)
    o.unrolled_forward(K)
    gfo, _, gwo = o.unrolled_backward(gu[:STRIP].double().cpu().numpy())
    for got, ref in [(gf, gfo)] + ([(gw, gwo)] if add else []):
        a, b = got.double().cpu().numpy()[..., :ROWS, :], ref[..., :ROWS, :]
        assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b)
        assert np.abs(a - b).max() <= 1e-2 * np.abs(b).max()


@pytest.mark.parametrize("add", [True, False])
@pytest.mark.parametrize("data,H,Wd,L", [("trunc", 37, 130, 5), ("trunc", 64, 65, 8), ("trunc", 41, 70, 12),
                                         ("trunc", 33, 64, 16), ("phase", 49, 100, 9), ("trunc", 40, 90, 24)])
def test_replay_on_chip_equals_replay_by_single_launches(data, H, Wd, L, add):
    """Segments of 12 iterations are replayed on chip (chunks of one to four labels; six: by single
    launches), segments of four by single launches: the gradients have the same bits."""
    wl = W.phase_unwrapping(H=H, W=Wd, L=L, seed=31) if data == "phase" else W.truncated_quadratic(L=L, H=H, W=Wd, seed=31)
    if add and data == "trunc":
        wl.tau = wl.gamma.copy()
        wl.samples = np.random.default_rng(32).normal(0, 0.02, (L, H, Wd)).astype(np.float32)
    out = []
    for every in (12, 4):
        p = S.Problem.from_workload(wl)
        p.unrolled_forward(27, every)
        _, u = p.read_u()
        gf, gl, gw = p.unrolled_backward(2.0 * u)
        out.append((gf, gl, gw))
        torch.cuda.synchronize()
        p.close()
    assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
    assert (out[0][2] is None and out[1][2] is None) or torch.equal(out[0][2], out[1][2])
