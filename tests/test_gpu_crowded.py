"""Crowded coverages in the folded path: segments of placements that run on far beyond the diagonals (a pile on
one cell, a compact array, a column of cells), with the lists behind the diagonals on both sides of one
workgroup's threads and of their vectors, in every precision form and both weightings, against the
FP64 oracle: weight sums and out-of-grid counts bit-exact, images within a relative L2 of 1e-5 (FP32) or
1e-3 (split forms). And their cost: a call on a pile may take at most twice the time of the same call on a
coverage spread over the grid.
"""
import numpy as np
import pytest

import oracle
from image_checks import rel_l2

pytestmark = pytest.mark.gpu

IMAGE_TOL = {0: 1e-5, 1: 1e-3, 2: 1e-3}
FREQ = 150.0e6
DL = 1.0e-3
WAVES_PER_CELL = FREQ / 299792458.0 * DL      # times N


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


def uvw_of(cells, N):
    uvw = np.zeros((1, len(cells), 3))
    uvw[0, :, :2] = np.asarray(cells, dtype=float) / (WAVES_PER_CELL * N)
    return uvw


def check(torch, ctx, what, cells, N, weighting, prec=0, P=1):
    import paper_2505_15204_amd as blink

    B = len(cells)
    print(f"[gpu-case] crowded {what} B={B} N={N} w={weighting} prec={prec}", flush=True)
    g = np.random.default_rng(B + N)
    uvw, freq = uvw_of(cells, N), np.array([FREQ])
    vis = (g.normal(size=(1, 1, P, B)) + 1j * g.normal(size=(1, 1, P, B))).astype(np.complex64)
    d = "cuda:0"
    ws = torch.full((blink.image_batch_workspace_size(1, 1, P, B, N, weighting, prec),), 255, dtype=torch.uint8, device=d)
    res = ctx.blink_image_batch(torch.from_numpy(vis).to(d), None, torch.from_numpy(uvw).to(d),
                                torch.from_numpy(freq).to(d), N, DL, weighting, precision=prec, workspace=ws)
    torch.cuda.synchronize()
    ref = oracle.image_batch(vis, None, uvw, freq, N, DL, weighting)
    assert np.array_equal(res["weight_sum"].cpu().numpy(), ref["weight_sum"])
    assert np.array_equal(res["n_out"].cpu().numpy(), ref["n_out"])
    for p in range(P):
        assert rel_l2(res["images"][0, 0, p].cpu().numpy(), ref["images"][0, 0, p]) <= IMAGE_TOL[prec], p


def piles(lengths, N, seed):
    """Piles of the given lengths, each on a cell of its own with neighbours in the same folded cell."""
    g = np.random.default_rng(seed)
    rows = N * N // 16384 if N > 128 else 1            # classes of rows: cells this far apart fold onto one
    step = N // rows
    out = []
    for i, n in enumerate(lengths):
        u, v = 1 + 3 * i, int(g.integers(-N // 4, N // 4))
        kv = v + step * g.integers(0, min(rows, 3), n) if i % 2 else np.full(n, v)
        kv = (kv + N // 2) % N - N // 2
        kv[kv == -N // 2] = v
        out += [(u, int(k)) for k in kv]
    g.shuffle(out)
    return out


# placements beyond the diagonals (16 of a segment): one, up to the threads of the workgroup, past them, whole
# vectors of a lane and one less or more, a second round of the workgroup
@pytest.mark.parametrize("beyond", [1, 63, 64, 511, 512, 513, 519, 520, 4096, 4097, 8000])
def test_one_pile(torch, ctx, beyond):
    check(torch, ctx, "one pile", [(5, 7)] * (16 + beyond), 512, 0)


@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("lengths", [[17] * 40, [24, 40, 64, 65, 100, 16, 15, 3] * 4, [257, 256, 255, 300, 700], [1000, 5000],
                                     [20] * 200])
def test_piles(torch, ctx, lengths, weighting):
    check(torch, ctx, "piles", piles(lengths, 512, 1), 512, weighting)
    check(torch, ctx, "piles", piles(lengths, 2048, 2), 2048, weighting, P=2)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("N", [256, 1024, 4096])
def test_compact_array(torch, ctx, N, weighting, prec):
    g = np.random.default_rng(3)
    check(torch, ctx, "compact", np.rint(g.normal(0, 4, (6000, 2))), N, weighting, prec)


@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("B", [8192, 16384])
def test_all_on_the_centre(torch, ctx, B, weighting):
    check(torch, ctx, "centre", [(0, 0)] * B, 512, weighting)        # each with its mirror in the same cell
    check(torch, ctx, "column", [(0, i % 101 - 50) for i in range(B)], 2048, weighting)


def call_us(torch, ctx, cells, N, C, weighting):
    import paper_2505_15204_amd as blink

    d, B = "cuda:0", len(cells)
    vis = torch.randn((1, C, 1, B), device=d, dtype=torch.complex64)
    uvw, freq = torch.from_numpy(uvw_of(cells, N)).to(d), torch.full((C,), FREQ, dtype=torch.float64, device=d)
    out = torch.empty((1, C, 1, N, N), device=d)
    ws = torch.empty(blink.image_batch_workspace_size(1, C, 1, B, N, weighting, 0), dtype=torch.uint8, device=d)
    best = 1.0e9
    for _ in range(6):                                               # the first one warms up
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            ctx.blink_image_batch(vis, None, uvw, freq, N, DL, weighting, out=out, workspace=ws)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 3 * 1e3)
    return best


@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("N,C", [(1024, 64), (2048, 16)])
def test_a_pile_costs_no_more_than_twice_a_spread_coverage(torch, ctx, N, C, weighting):
    print(f"[gpu-case] crowded timing N={N} w={weighting}", flush=True)
    r = N // 2 - 1
    spread = call_us(torch, ctx, np.random.default_rng(4).uniform(-r, r, (8128, 2)), N, C, weighting)
    pile = call_us(torch, ctx, [(2, 2)] * 8128, N, C, weighting)
    assert pile <= 2.0 * spread, (pile, spread)
