"""A batch needs its members' planes and the work tables, and no rim words of the on-chip
iteration, which no member runs: a workspace without them is accepted (and left alone behind
its end). The bytes needed are those that the refusal of an empty workspace names."""
import ctypes as C
import re

import numpy as np
import pytest

import paper_1512_01383_amd as S
import workloads as W

WORKSPACE_ERROR = 4


def _needed(descs):
    h = C.c_void_p()
    assert S.lib().sl_batch_create(descs, len(descs), C.c_void_p(256), 0, None, C.byref(h)) == WORKSPACE_ERROR
    return int(re.search(r"than the (\d+) needed", S.lib().sl_last_error().decode()).group(1))


def _desc(H, W_, L):
    d = S.Desc()
    d._gamma = np.linspace(0.0, 1.0, L)
    d.gamma = d._gamma.ctypes.data_as(C.POINTER(C.c_double))
    d.H, d.W, d.L = H, W_, L
    d.rho = S.RHO_TRUNC_QUAD
    d.f = 16           # not read by these calls
    d.a, d.nu, d.lam = 2.0, 0.025, 0.25
    d.check_every, d.normalize_labels = 48, 1
    return d


@pytest.mark.parametrize("H,Wd,L", [(64, 64, 2), (64, 64, 20), (256, 256, 20), (353, 517, 10)])
def test_members_need_no_rim_words(H, Wd, L):
    d = _desc(H, Wd, L)
    lone = C.c_size_t()
    assert S.lib().sl_workspace_size(C.byref(d), C.byref(lone)) == 0
    member = _needed((S.Desc * 2)(d, d)) - _needed((S.Desc * 1)(d))   # a member and its place in the tables
    # a lone problem on the chip: two slots of at least 128 words of 8 bytes per tile and label,
    # the tiles at most 16 rows of 64 pixels per label group and 4 groups
    tiles = -(-Wd // 64) * -(-H // 16)
    table = 8192 + 16 * -(-Wd // 64) * H
    assert member <= lone.value - 2 * tiles * (L - 1) * 128 * 8 + table


@pytest.mark.gpu
def test_a_workspace_without_rim_words_serves():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():  # pragma: no cover
        pytest.skip("needs a GPU")
    wls = [W.truncated_quadratic(L=20, H=64, W=64, seed=71), W.truncated_quadratic(L=10, H=97, W=130, seed=72)]
    b = S.BatchProblem(wls)
    b.run_to_gap(0.0, 96)
    insts, descs = [], (S.Desc * 2)()
    for j, wl in enumerate(wls):
        it = S._Inst()
        descs[j] = S._make_desc(it, wl.H, wl.W, wl.gamma, wl.rho, wl.lam, wl.f, wl.a, wl.nu, None, None, "fp32", True, 48,
                                b.device, True)
        insts.append(it)
    need = _needed(descs)
    ws = torch.full((need + 4096,), 0xAB, dtype=torch.uint8, device=b.device)
    h, done = C.c_void_p(), C.c_int32()
    S._check(S.lib().sl_batch_create(descs, 2, C.c_void_p(ws.data_ptr()), need,
                                     C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(h)))
    S._check(S.lib().sl_run_to_gap(h, 0.0, 96, C.byref(done)))
    for i, it in enumerate(insts):
        u = torch.empty((it.H, it.W), dtype=torch.float32, device=b.device)
        S._check(S.lib().sl_batch_read_u(h, i, None, C.c_void_p(u.data_ptr())))
        assert torch.equal(u, b.read_u_of(i)[1])
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xAB).all())
    S.lib().sl_destroy(h)
    b.close()
