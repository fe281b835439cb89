"""Folded imaging of many polarisations of few pairs, whose values a launch of its own writes (from four polarisations on, below
256 pairs), against the FP64 oracle: weight sums and out-of-grid counts bit-exact, images within a relative L2 of
1e-5 (FP32) or 1e-3 (split forms); positions in one window and in several, corrected visibilities, chunks. And the
cost: 64 images of one pair may take at most twice what 64 pairs of one image take.
"""
import numpy as np
import pytest

import oracle
from image_checks import rel_l2
from test_gpu_fold import check

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


@pytest.mark.parametrize("P,C", [(3, 2), (4, 1), (5, 3), (17, 2)])
@pytest.mark.parametrize("weighting", [0, 1])
def test_polarisations(torch, ctx, weighting, P, C):
    check(torch, ctx, "uniform", 700, 512, weighting, 0, C=C, P=P)
    check(torch, ctx, "pile", 3000, 1024, weighting, 0, C=C, P=P, shift=False)


@pytest.mark.parametrize("prec,weighting", [(0, 0), (0, 1), (1, 0), (2, 1)])
@pytest.mark.parametrize("kind,B", [("uniform", 1), ("uniform", 4095), ("uniform", 8192), ("column0", 8192), ("uniform", 8193),
                                    ("column0", 16384)])
def test_windows(torch, ctx, kind, B, prec, weighting):
    check(torch, ctx, kind, B, 512, weighting, prec, P=4)


@pytest.mark.parametrize("corrected", [False, True])
def test_chunks(torch, ctx, corrected):
    import paper_2505_15204_amd as blink
    N, C, P, B, d = 512, 5, 6, 4950, "cuda:0"
    g = np.random.default_rng(2)
    uvw = np.zeros((1, B, 3))
    uvw[0, :, :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (B, 2)) / (FREQ / 299792458.0 * (N * DL))
    vis = (g.normal(size=(1, C, P, B)) + 1j * g.normal(size=(1, C, P, B))).astype(np.complex64)
    flags, freq = (g.random((1, C, B)) < 0.1).astype(np.uint8), np.full(C, FREQ)
    ref = oracle.image_batch(vis, flags, uvw, freq, N, DL, 0)
    call = ctx.blink_image_batch_corrected if corrected else ctx.blink_image_batch
    pair = 8448 + (2 * B + 1024) * (4 + 8 * P) + 12 * B + (8 * B * P if corrected else 0) + 2048
    for nbytes in (6 * pair, int(2.5 * pair)):
        print(f"[gpu-case] pols chunks corrected={corrected} bytes={nbytes}", flush=True)
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=d)
        res = call(*(torch.from_numpy(x).to(d) for x in (vis, flags, uvw, freq)), N, DL, 0, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(res["weight_sum"].cpu().numpy(), ref["weight_sum"])
        for c in range(C):
            for p in range(P):
                assert rel_l2(res["images"][0, c, p].cpu().numpy(), ref["images"][0, c, p]) <= 1e-5, (nbytes, c, p)


def test_images_of_one_pair_cost_no_more_than_twice(torch, ctx):
    import paper_2505_15204_amd as blink
    N, B, d = 512, 8128, "cuda:0"
    g = np.random.default_rng(3)
    uvw = np.zeros((1, B, 3))
    uvw[0, :, :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (B, 2)) / (FREQ / 299792458.0 * (N * DL))
    uvw = torch.from_numpy(uvw).to(d)
    print("[gpu-case] pols timing", flush=True)

    def call_us(C, P):
        vis = torch.randn((1, C, P, B), device=d, dtype=torch.complex64)
        freq = torch.full((C,), FREQ, dtype=torch.float64, device=d)
        out = torch.empty((1, C, P, N, N), device=d)
        ws = torch.empty(blink.image_batch_workspace_size(1, C, P, B, N, 0, 0), dtype=torch.uint8, device=d)
        best = 1.0e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                ctx.blink_image_batch(vis, None, uvw, freq, N, DL, 0, out=out, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 4 * 1e3)
        return best
    one, many = call_us(1, 64), call_us(64, 1)
    assert one <= 2.0 * many, (one, many)
