"""Every kernel that an on-chip run can pick (labels, label groups and rows per thread, one group
of threads or several, each data term) against the same iterations one launch at a time: the
states must be equal bit for bit. The sizes are the smallest images that lead to the kernel, with
tiles, rows per thread and label chunks that do not come out even; a run that stayed off the chip
fails (an on-chip launch writes rim words).

Reverse passes: a replay on chip writes rim words into the problem's workspace, which the reverse
pass leaves alone otherwise."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1512_01383_amd as S  # noqa: E402

# (labels, label groups, rows) per thread and most groups of threads: H, W, L, label groups
SHAPES = {
    (1, 1, 1, 4): (33, 129, 2, 1),
    (2, 1, 1, 4): (33, 129, 6, 4),
    (3, 1, 1, 4): (33, 129, 11, 4),
    (4, 1, 1, 4): (33, 129, 14, 4),
    (5, 1, 1, 4): (33, 129, 18, 4),
    (6, 1, 1, 4): (33, 129, 22, 4),
    (7, 1, 1, 1): (999, 193, 8, 1),
    (7, 1, 1, 4): (33, 129, 26, 4),
    (8, 1, 1, 1): (999, 193, 9, 1),
    (8, 1, 1, 4): (63, 1538, 16, 2),
    (9, 1, 1, 1): (999, 193, 10, 1),
    (2, 2, 1, 2): (513, 70, 4, 4),
    (4, 2, 1, 2): (513, 70, 6, 4),
    (6, 2, 1, 2): (513, 70, 11, 4),
    (8, 2, 1, 1): (1399, 70, 8, 2),
    (8, 2, 1, 2): (513, 70, 14, 4),
    (10, 2, 1, 1): (1399, 70, 10, 2),
    (4, 4, 1, 1): (1101, 70, 4, 4),
    (8, 4, 1, 1): (1101, 70, 6, 4),
}
ROWS = {   # several rows per thread; those of truncated quadratics first
    (1, 1, 2, 1): (1399, 129, 2, 1),
    (1, 1, 3, 1): (1399, 322, 2, 1),
    (1, 1, 4, 1): (1399, 514, 2, 1),
    (1, 1, 6, 1): (999, 1026, 2, 1),
    (2, 1, 2, 1): (1501, 129, 3, 1),
    (2, 1, 3, 1): (1399, 322, 3, 1),
    (3, 1, 2, 1): (1501, 129, 4, 1),
    (1, 1, 8, 1): (999, 1538, 2, 1),
    (1, 1, 12, 1): (1399, 1538, 2, 1),
    (2, 1, 4, 1): (1399, 514, 3, 1),
    (2, 1, 6, 1): (999, 1026, 3, 1),
    (3, 1, 3, 1): (1399, 322, 4, 1),
    (3, 1, 4, 1): (1399, 514, 4, 1),
    (4, 1, 2, 1): (1501, 129, 5, 1),
    (4, 1, 3, 1): (1399, 322, 5, 1),
    (5, 1, 2, 1): (1501, 129, 6, 1),
}
OFF = ("quad+w", (10, 2, 1, 1))   # as fast off the chip
CASES = ([(data, shape) for shape in SHAPES for data in ("trunc", "trunc+w", "quad", "quad+w", "sampled")
          if (data, shape) != OFF] +
         [(data, shape) for i, shape in enumerate(ROWS) for data in (("trunc", "quad") if i < 7 else ("quad",))])


def _workload(data, H, Wd, L, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    gamma = W.equispaced(L)
    if data == "sampled":
        tau = W.equispaced(3 * (L - 1) + 1)
        gamma = tau[::3].copy()
        return W.Workload(data, H, Wd, gamma, W.SAMPLED, 0.3, tau=tau,
                          samples=rng.uniform(0.0, 0.2, (len(tau), H, Wd)).astype(np.float32))
    f = rng.uniform(-0.1, 1.1, (H, Wd)).astype(np.float32)
    if data.startswith("quad") and L % 3 == 0:
        wl = W.Workload(data, H, Wd, gamma, W.PERIODIC_QUAD, 0.2, f=f, a=2.0, nu=0.5)
    elif data.startswith("quad"):
        wl = W.Workload(data, H, Wd, gamma, W.QUAD, 0.2, f=f)
    else:
        wl = W.Workload(data, H, Wd, gamma, W.TRUNC_QUAD, 0.25, f=f, a=2.0, nu=0.025)
    if data.endswith("+w") and wl.rho == W.PERIODIC_QUAD:
        wl.rho = W.QUAD
    if data.endswith("+w"):
        wl.tau = gamma.copy()
        wl.samples = rng.normal(0.0, 0.02, (L, H, Wd)).astype(np.float32)
    return wl


def _on_chip(prob, n):
    """Did a run of n iterations write rim words? (They lie behind the 11 k + 1 planes of the state
    and what iterations only read.)"""
    N = prob.H * prob.W
    plane = -(-N // 64) * 64 + (320 if -(-N // 64) * 64 % (1 << 18) == 0 else 0)
    before = prob.workspace.clone()
    prob.run(n)
    torch.cuda.synchronize()
    return int(torch.nonzero(prob.workspace != before).max()) >= (11 * prob.k + 1) * plane * 4


@pytest.mark.parametrize("data,shape", CASES, ids=["%s-%d.%d.%d.%d" % ((c[0],) + c[1]) for c in CASES])
def test_every_on_chip_kernel_equals_single_launches(data, shape):
    H, Wd, L, groups = SHAPES.get(shape) or ROWS[shape]
    wl = _workload(data, H, Wd, L, seed=sum(shape))
    wl.tv = L % 2
    storage = "bf16" if (L + groups) % 2 else "fp32"
    a, b = (S.Problem.from_workload(wl, storage=storage) for _ in range(2))
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    st = 0.5 * torch.randn(a.state_size() // 4, generator=gen, device="cuda:0")
    for p in (a, b):
        p.set_tiling(groups, 4)
        p.load_state(st)
    least = 16 if shape[0] >= 3 and shape[0] * shape[2] >= (10 if storage == "bf16" else 12) else 8
    assert _on_chip(a, least) and not _on_chip(b, 1)
    a.run(least + 1)
    for _ in range(2 * least):
        b.run(1)
    sa, sb = a.save_state(), b.save_state()
    assert torch.isfinite(sa).all()
    assert torch.equal(sa, sb)
    a.close()
    b.close()


@pytest.mark.parametrize("data", ["trunc", "trunc+w", "quad", "quad+w"])
@pytest.mark.parametrize("L,on_chip", [(2, True), (6, True), (11, True), (14, True), (18, False)])
def test_replay_on_chip_runs_and_equals_single_launches(data, L, on_chip):
    """Label chunks of one to four have a kernel that keeps every state; five do not."""
    wl = _workload(data, 33, 129, L, seed=L)
    out = []
    for every in (12, 4):
        p = S.Problem.from_workload(wl)
        p.unrolled_forward(27, every)
        u = p.read_u()[1]
        before = p.workspace.clone()
        out.append(p.unrolled_backward(2.0 * u))
        assert torch.equal(p.workspace, before) == (not (on_chip and every == 12))
        p.close()
    (fa, la, wa), (fb, lb, wb) = out
    assert torch.equal(fa, fb) and la == lb
    assert (wa is None and wb is None) or torch.equal(wa, wb)
