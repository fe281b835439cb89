"""The tiled de-dispersion kernel where its dispatch takes it, against the oracle, bit for bit: every compiled tile length,
channel counts on both sides of a stage of four, a last tile and a last trial pair that are not full, several workgroups per
pixel block, and both sides of each line of the rule. The rule is restated here, so every case says which kernel it is for.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


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


def tiling(delays, t_out, N):
    """(tiled, steps of a tile, most steps of a channel in a workgroup, workgroups per 64 pixels): a unit is two trials x a
    tile of at most 13 steps, a workgroup 16 units; tiled with at most 4096 channels, at most 60 steps of a channel,
    at least 96 workgroups, 8 units and 2.5 reads of each copied step."""
    n_dm, C = delays.shape
    tiles = -(-t_out // 13)
    tb = -(-t_out // tiles)
    units = -(-n_dm // 2) * tiles
    groups = -(-units // 16)
    rows = copied = 0
    for q in range(groups):
        lo, hi = np.full(C, 1 << 30), np.zeros(C, int)
        for u in range(16 * q, min(16 * q + 16, units)):
            t0, t1 = u % tiles * tb, min(u % tiles * tb + tb, t_out)
            for k in range(u // tiles * 2, min(u // tiles * 2 + 2, n_dm)):
                lo, hi = np.minimum(lo, t0 + delays[k]), np.maximum(hi, t1 + delays[k])
        rows = max(rows, int((hi - lo).max()))
        copied += int((hi - lo).sum())
    fits = C <= 4096 and rows <= 60 and N * N // 64 * groups >= 96 and units >= 8 and 2 * n_dm * t_out * C >= 5 * copied
    return fits, tb, rows, groups


def check(torch, ctx, T, C, N, n_dm, t_out, tiled, tb=None, rows=None, groups=None):
    g = np.random.default_rng(T * 100 + C)
    delays = g.integers(0, T - t_out + 1, (n_dm, C)).astype(np.int32)
    delays[0], delays[1] = 0, T - t_out                   # the first pair spans every step
    fits, b, r, q = tiling(delays, t_out, N)
    assert fits == tiled and b == (tb or b) and r == (rows or r) and q == (groups or q), (fits, b, r, q)
    imgs = g.normal(size=(T, C, N, N)).astype(np.float32)
    print(f"[gpu-case] de-dispersion T={T} C={C} N={N} n_dm={n_dm} t_out={t_out} tiled={tiled}", flush=True)
    out = ctx.blink_dedisperse(torch.from_numpy(imgs).to("cuda:0"), delays, t_out).cpu().numpy()
    assert np.array_equal(out, oracle.dedisperse(imgs, delays, t_out).astype(np.float32))


@pytest.mark.parametrize("t_out", range(1, 14))
def test_every_tile_length(torch, ctx, t_out):
    check(torch, ctx, t_out + 4, 1 + t_out % 9, 128, 16, t_out, True, tb=t_out, groups=1)


@pytest.mark.parametrize("T,C,N,n_dm,t_out,tiled,what", [
    (60, 6, 128, 8, 40, True, dict(rows=60, tb=10)),
    (61, 6, 128, 8, 40, False, dict(rows=61)),
    (60, 5, 128, 12, 38, True, dict(rows=60, tb=13, groups=2)),     # the last tile one step short, reads past the stage
    (30, 7, 128, 33, 27, True, dict(tb=9, groups=4)),               # a trial alone, a workgroup of three units
    (19, 4, 128, 17, 15, True, dict(tb=8, groups=2)),
    (9, 3, 128, 14, 6, False, dict()),                              # seven units
    (9, 3, 128, 15, 6, True, dict()),                               # eight
    (7, 2, 128, 16, 1, False, dict(rows=7)),                        # 16 reads of 7 copied steps
    (6, 2, 128, 16, 1, True, dict(rows=6)),                         # of 6
    (5, 3, 64, 16, 2, False, dict(groups=1)),                       # 64 workgroups
    (5, 3, 64, 33, 2, True, dict(groups=2)),                        # 128
    (3, 4096, 32, 192, 1, True, dict(groups=6)),
    (3, 4097, 32, 192, 1, False, dict(groups=6)),
])
def test_both_sides_of_the_rule(torch, ctx, T, C, N, n_dm, t_out, tiled, what):
    check(torch, ctx, T, C, N, n_dm, t_out, tiled, **what)
