"""blink_grid on coverages along one axis and on one cell, at sizes with one tile, one row and column of tiles, and many,
against the oracle (counts and weight sums bit-exact, grids within 1e-6 in relative L2: whole-number visibilities
are summed exactly), and what an east-west array (v = 0) costs: at most twice the same call on a coverage over
the whole grid.
"""
import numpy as np
import pytest

import oracle
from image_checks import rel_l2

pytestmark = pytest.mark.gpu

FREQ = 150.0e6
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


def coverage(kind, N, B):
    g = np.random.default_rng(N + B)
    x = np.zeros((1, B, 3))
    x[0, :, :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (B, 2))
    if kind == "row":
        x[0, :, 1] = 0
    if kind == "column":
        x[0, :, 0] = 0
    if kind == "diagonal":
        x[0, :, 1] = x[0, :, 0]
    if kind == "pile":
        x[0, :, :2] = 1
    return x / (FREQ / 299792458.0 * (N * DL))


@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("kind", ["row", "column", "diagonal", "pile"])
@pytest.mark.parametrize("N", [8, 64, 128, 256, 1024, 4096])
def test_axes(torch, ctx, N, kind, weighting):
    B, C, P = 1500, 3 if N < 4096 else 1, 2
    print(f"[gpu-case] grid tiles N={N} {kind} w={weighting}", flush=True)
    g = np.random.default_rng(N)
    uvw, freq = coverage(kind, N, B), np.full(C, FREQ)
    vis = (g.integers(-9, 10, (1, C, P, B)) + 1j * g.integers(-9, 10, (1, C, P, B))).astype(np.complex64)
    flags = (g.random((1, C, B)) < 0.1).astype(np.uint8)
    res = ctx.blink_grid(*(torch.from_numpy(x).to("cuda:0") for x in (vis, flags, uvw, freq)), N, DL, weighting)
    torch.cuda.synchronize()
    for c in range(C):
        ref = oracle.grid(vis[0, c], np.ascontiguousarray(flags[0, c]), uvw[0], FREQ, N, DL, weighting)
        assert np.array_equal(res["counts"][0, c].cpu().numpy(), ref["counts"])
        for p in range(P):
            assert float(res["weight_sum"][0, c, p]) == ref["weight_sum"]
            assert rel_l2(res["grids"][0, c, p].cpu().numpy(), ref["grid"][p]) <= 1e-6, (c, p)


def test_an_east_west_array_costs_no_more_than_twice(torch, ctx):
    import paper_2505_15204_amd as blink
    N, C, B, d = 256, 64, 8128, "cuda:0"
    print("[gpu-case] grid tiles timing", flush=True)
    vis = torch.randn((1, C, 2, B), device=d, dtype=torch.complex64)
    freq = torch.full((C,), FREQ, dtype=torch.float64, device=d)
    ws = torch.empty(blink.grid_workspace_size(1, C, B, N), dtype=torch.uint8, device=d)

    def call_us(kind):
        uvw = torch.from_numpy(coverage(kind, N, B)).to(d)
        best = 1.0e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                ctx.blink_grid(vis, None, uvw, freq, N, DL, 0, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 4 * 1e3)
        return best
    line, whole = call_us("row"), call_us("whole")
    assert line <= 2.0 * whole, (line, whole)
