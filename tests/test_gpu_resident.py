"""Runs of several iterations in one on-chip launch (state in registers and LDS, the rims of
the tiles exchanged between blocks) against the same iterations one launch at a time, which
the parity tests pin to the oracle. Both walk, sum and round alike, so the states must be
equal bit for bit. Sizes sit at the edges of the layout: one tile, one column of tiles, tiles
of one valid row or column, label chunks that do not fill their threads, more than one label
group per thread, every data term, both TV kinds and both dual storages."""
import dataclasses

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)


def _workload(data, H, Wd, L, tv):
    if data == "trunc":
        wl = W.truncated_quadratic(L=L, H=H, W=Wd, seed=11)
    elif data == "quad":
        rng = np.random.Generator(np.random.PCG64(12))
        wl = W.Workload("quad", H, Wd, W.equispaced(L), W.QUAD, 0.2, f=rng.uniform(-0.2, 1.2, (H, Wd)).astype(np.float32))
    elif data == "phase":
        wl = W.phase_unwrapping(H=H, W=Wd, L=L, seed=13)
    elif data == "add":
        wl = W.differentiation(H=H, W=Wd, L=L, seed=14)
        wl.samples = (0.05 * np.random.Generator(np.random.PCG64(15)).normal(size=wl.samples.shape)).astype(np.float32)
    else:
        wl = W.stereo(H=H, W=Wd, L=L, n_disp=7 * (L - 1) + 1, seed=16)
    return dataclasses.replace(wl, tv=tv)


CASES = [
    ("quad", 64, 64, 2, 0, "fp32", None),       # one interval, one column of tiles
    ("quad", 2, 5, 2, 1, "fp32", None),         # less than a tile
    ("quad", 33, 65, 3, 0, "bf16", None),       # a tile of one column, a tile of one row
    ("trunc", 37, 150, 6, 0, "fp32", None),     # k = 5 in chunks of 2: an empty group
    ("trunc", 63, 129, 16, 1, "bf16", None),    # k = 15 in chunks of 4: a short group
    ("trunc", 50, 64, 20, 0, "fp32", None),
    ("trunc", 41, 70, 2, 0, "fp32", None),      # both edges of the band in one interval
    ("trunc", 200, 250, 5, 0, "fp32", (1, 4, 64)),    # one group, four labels per thread
    ("trunc", 500, 512, 7, 0, "fp32", (2, 4, 64)),    # two groups per thread
    ("phase", 49, 100, 9, 0, "fp32", None),
    ("phase", 570, 400, 5, 0, "bf16", (4, 4, 64)),    # four groups per thread
    ("add", 45, 130, 8, 0, "fp32", None),
    ("sampled", 40, 90, 4, 0, "fp32", None),
    ("sampled", 31, 64, 9, 1, "bf16", (1, 4, 64)),
    # several rows per thread: two (a last tile of one row), three, twelve; two of several labels
    ("quad", 521, 513, 2, 0, "fp32", None),
    ("trunc", 700, 705, 2, 0, "bf16", None),
    ("quad", 1531, 2039, 2, 0, "fp32", None),
    ("phase", 500, 700, 6, 1, "fp32", None),
    ("trunc", 530, 513, 4, 0, "fp32", None),
    # long label chunks, whose rim words are waited for in turns
    ("trunc", 353, 517, 10, 1, "fp32", None),
    ("trunc", 490, 510, 9, 0, "bf16", None),
    ("sampled", 260, 333, 9, 0, "fp32", (1, 4, 64)),
]


def _changed(prob, n):
    before = prob.workspace.clone()
    prob.run(n)
    torch.cuda.synchronize()
    return int(torch.nonzero(prob.workspace != before).max())


@pytest.mark.parametrize("data,H,Wd,L,tv,storage,tiling", CASES,
                         ids=[f"{c[0]}-{c[1]}x{c[2]}-L{c[3]}-tv{c[4]}-{c[5]}" for c in CASES])
def test_on_chip_iterations_equal_single_launches(data, H, Wd, L, tv, storage, tiling):
    import paper_1512_01383_amd as S

    wl = _workload(data, H, Wd, L, tv)
    a, b = (S.Problem.from_workload(wl, storage=storage) for _ in range(2))
    if tiling:
        a.set_tiling(*tiling)
        b.set_tiling(*tiling)
    st = torch.as_tensor(np.concatenate([x.reshape(-1) for x in (W.random_state(9, wl.k, H, Wd)[n] for n in W.STATE_ORDER)]))
    a.load_state(st)
    b.load_state(st)
    # odd and even counts (every rotation of the buffers), one after another on the same
    # handle; a single launch writes the state only, an on-chip one also the rim words, which
    # lie behind everything else
    one = _changed(a, 1)
    b.run(1)
    assert _changed(a, 8) > one or (H <= 2 and Wd <= 64)
    for n in (9, 13):
        a.run(n)
    for _ in range(8 + 9 + 13):
        b.run(1)
    sa, sb = a.save_state(), b.save_state()
    assert torch.isfinite(sa).all()
    assert torch.equal(sa, sb)
    ua, ub = a.read_u()[1], b.read_u()[1]
    assert torch.equal(ua, ub)
    a.close()
    b.close()


def test_a_captured_run_replays_single_launches():
    """Twelve iterations captured into a graph (two periods of the buffers' rotation) and
    replayed, with eager work in between, against the same iterations run eagerly."""
    import paper_1512_01383_amd as S

    wl = _workload("trunc", 48, 96, 6, 0)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        a, b = (S.Problem.from_workload(wl) for _ in range(2))
        a.run(12)
        b.run(12)
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            a.run(12)
        for _ in range(3):
            g.replay()
            b.run(12)
            side.synchronize()
            assert torch.equal(a.save_state(), b.save_state())
    torch.cuda.synchronize()


def test_two_streams_run_on_chip_side_by_side():
    """Problems on two streams, each large enough to want most of the chip: their launches
    are queued against each other and each must finish with its own result."""
    import paper_1512_01383_amd as S

    wl = _workload("trunc", 256, 256, 9, 0)
    ref = S.Problem.from_workload(wl)
    ref.run(60)
    want = ref.save_state()
    streams = [torch.cuda.Stream() for _ in range(2)]
    probs = []
    for s in streams:
        with torch.cuda.stream(s):
            probs.append(S.Problem.from_workload(wl))
    torch.cuda.synchronize()
    for _ in range(3):
        for p in probs:
            p.run(20)
    torch.cuda.synchronize()
    for s, p in zip(streams, probs):
        with torch.cuda.stream(s):
            got = p.save_state()
        s.synchronize()
        assert torch.equal(got, want)
