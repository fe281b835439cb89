"""The batch autotuner times the two-pass form, which its plan steers, also on problems that blink_image_batch images in
the folded form. Visibilities are small whole numbers, so grids are exact in any order of summation and each
form's images are the same bits on every run: the tuner's images have to be those of the two-pass form (the same problem
with flagged baselines added up to 16385, which only that form takes), not those of the folded one.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FREQ = 150.0e6
DL = 1.0e-3


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("prec,weighting", [(0, 0), (0, 1), (1, 0), (2, 0)])
def test_tunes_the_two_pass_form(torch, prec, weighting):
    import paper_2505_15204_amd as blink

    N, C, B, more = 512, 3, 700, 16385
    print(f"[gpu-case] autotune N={N} prec={prec} w={weighting}", flush=True)
    g = np.random.default_rng(9)
    uvw = np.zeros((1, more, 3))
    uvw[..., :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (1, more, 2)) / (FREQ / 299792458.0 * (N * DL))
    vis = (g.integers(-8, 9, (1, C, 1, more)) + 1j * g.integers(-8, 9, (1, C, 1, more))).astype(np.complex64)
    flags = np.ones((1, C, more), np.uint8)
    flags[..., :B] = 0
    d = "cuda:0"
    freq = torch.full((C,), FREQ, dtype=torch.float64, device=d)
    part = [torch.from_numpy(np.ascontiguousarray(x)).to(d) for x in (vis[..., :B], flags[..., :B], uvw[:, :B])]
    whole = [torch.from_numpy(x).to(d) for x in (vis, flags, uvw)]
    with blink.Context(0) as ctx:
        out = torch.empty((1, C, 1, N, N), device=d)
        plan, ms = ctx.autotune_image_batch(*part, freq, N, DL, weighting, precision=prec, out=out)
        torch.cuda.synchronize()
        assert ms > 0 and ctx.get_plan(N, weighting, prec) == plan
        two_pass = ctx.blink_image_batch(*whole, freq, N, DL, weighting, precision=prec)["images"]
        folded = ctx.blink_image_batch(*part, freq, N, DL, weighting, precision=prec)["images"]
        torch.cuda.synchronize()
        assert torch.equal(out, two_pass)
        assert not torch.equal(out, folded)
