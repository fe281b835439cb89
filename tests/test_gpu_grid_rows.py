"""GPU parity of blink_grid's row strips at the edges of their layout: every grid size, natural and
uniform weighting, with and without counts, one baseline, more records in a strip than its threads
load at once, pairs that are no multiple of eight, arrays that start at an odd element, and a
workspace that holds one pair at a time. Counts, cell indices, weight sums and out-of-grid counts
are bit-exact; grids are within 1e-6 of the oracle's in relative L2: FP32 sums of at most 1000 terms
of one cell in any order, with an error below 1000 * 2^-24 = 6e-5 of it in the worst case and about
sqrt(1000) * 2^-25 = 9e-7 at random, and a few terms in nearly all cells.
"""
import numpy as np
import pytest

import oracle
from image_checks import rel_l2

pytestmark = pytest.mark.gpu

FREQ = 150.0e6
C_LIGHT = 299792458.0
DL = 1.0e-3


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.fixture(scope="module")
def ctx(torch):
    import paper_2505_15204_amd as blink
    c = blink.Context(0)
    yield c
    c.close()


def check(torch, ctx, N, B, weighting, counts, T=1, C=3, P=2, odd=False, one_pair=False, rows=None):
    import ctypes
    import paper_2505_15204_amd as blink

    print(f"[gpu-case] grid rows N={N} B={B} w={weighting} counts={counts} T={T} C={C} P={P} odd={odd}", flush=True)
    g = np.random.default_rng(5 + N + B)
    uvw = np.zeros((T, B, 3))
    uvw[..., :2] = g.uniform(-0.55 * N, 0.55 * N, (T, B, 2))
    if rows is not None:
        uvw[..., 1] = g.integers(-rows, rows + 1, (T, B))
    uvw /= FREQ / C_LIGHT * (N * DL)
    freq = np.full(C, FREQ)
    vis = (g.normal(size=(T, C, P, B)) + 1j * g.normal(size=(T, C, P, B))).astype(np.complex64)
    flags = (g.random((T, C, B)) < 0.1).astype(np.uint8)
    d = "cuda:0"
    tv, tf, tu, tq = (torch.from_numpy(x).to(d) for x in (vis, flags, uvw, freq))
    n_img, cells, off = T * C * P, N * N, 1 if odd else 0
    grids = torch.full((n_img * cells + off,), float("nan"), dtype=torch.complex64, device=d)[off:]
    cnt = torch.full((T * C * cells + off,), -5, dtype=torch.int32, device=d)[off:]
    wsum = torch.zeros(n_img, dtype=torch.float64, device=d)
    idx = torch.zeros((T, C, B), dtype=torch.int32, device=d)
    nout = torch.zeros((T, C), dtype=torch.int32, device=d)
    t, c = (1, 1) if one_pair else (T, C)
    size = ctypes.c_size_t()
    lib = blink.lib()
    assert lib.blink_grid_workspace_size(t, c, B, N, ctypes.byref(size)) == 0
    ws = torch.full((size.value,), 255, dtype=torch.uint8, device=d)
    ptr = lambda x: ctypes.c_void_p(x.data_ptr())
    st = lib.blink_grid(ctx.handle, ptr(tv), ptr(tf), ptr(tu), ptr(tq), T, C, P, B, N, ctypes.c_double(DL), weighting,
                        ptr(grids), ptr(cnt) if counts else None, ptr(wsum), ptr(idx), ptr(nout), ptr(ws),
                        ctypes.c_size_t(size.value), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    torch.cuda.synchronize()
    got, cn = grids.cpu().numpy().reshape(T, C, P, N, N), cnt.cpu().numpy()
    for i in range(T):
        for j in range(C):
            ref = oracle.grid(vis[i, j], flags[i, j], uvw[i], FREQ, N, DL, weighting)
            assert int(nout[i, j]) == ref["n_out"]
            for p in range(P):
                assert float(wsum[(i * C + j) * P + p]) == ref["weight_sum"]
                assert rel_l2(got[i, j, p], ref["grid"][p]) <= 1e-6, (i, j, p)
            if counts:
                assert np.array_equal(cn.reshape(T, C, N, N)[i, j], ref["counts"])
    if not counts:
        assert (cn == -5).all()


@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096])
def test_every_size(torch, ctx, N, weighting, counts):
    check(torch, ctx, N, 300, weighting, counts, C=3 if N <= 1024 else 1, P=2 if N <= 1024 else 1)


@pytest.mark.parametrize("B,T,C,P", [(1, 1, 1, 1), (257, 3, 3, 4), (1000, 2, 8, 1)])
def test_shapes(torch, ctx, B, T, C, P):
    check(torch, ctx, 128, B, 0, True, T=T, C=C, P=P)
    check(torch, ctx, 128, B, 1, True, T=T, C=C, P=P, one_pair=True)


@pytest.mark.parametrize("weighting", [0, 1])
def test_crowded_strip(torch, ctx, weighting):
    check(torch, ctx, 512, 6000, weighting, True, rows=2)


@pytest.mark.parametrize("N", [8, 256])
def test_odd_addresses(torch, ctx, N):
    check(torch, ctx, N, 200, 1, True, odd=True)
