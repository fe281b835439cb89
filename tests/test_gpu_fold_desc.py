"""GPU parity of the staged uneven-batch form's folded kernels (up to 16384 baselines an image): every
grid size in one batch, images without and with one baseline, image counts beside the groups of
eight, a batch larger than the workspace holds at a time, images that share pixels (more work items
than the first launch takes), and the baseline counts on both sides of the path's limits. Bars as
for the other parity tests: weight sums and out-of-grid counts bit-exact, images within a relative
L2 of 1e-5 (FP32) or 1e-3 (split forms) of the FP64 oracle.
"""
import numpy as np
import pytest

import oracle
from image_checks import rel_l2

pytestmark = pytest.mark.gpu

IMAGE_TOL = {0: 1e-5, 1: 1e-3, 2: 1e-3}
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
    c.set_desc_plan(512, 0, form=1)
    yield c
    c.close()


def check(torch, ctx, what, images, weighting=0, prec=0, max_b=None, max_n=None, share=False, flagged=0.1):
    """images: [(N, B)]; share: all of them in the same pixels, with the same inputs."""
    import paper_2505_15204_amd as blink

    print(f"[gpu-case] fold desc {what} n_img={len(images)} w={weighting} prec={prec}", flush=True)
    n_img = len(images)
    g = np.random.default_rng(77 + n_img)
    desc = np.zeros(n_img, blink.DESC_DTYPE)
    uvw, vis, flags, pix, at = [], [], [], 0, 0
    for i, (N, B) in enumerate(images):
        desc["grid_n"][i], desc["n_baselines"][i] = N, B
        desc["freq_hz"][i], desc["pixel_scale"][i] = FREQ, DL
        if share and i:
            for f in ("vis_offset", "uvw_offset", "flag_offset", "image_offset"):
                desc[f][i] = 0
            continue
        for f in ("vis_offset", "uvw_offset", "flag_offset"):
            desc[f][i] = at
        desc["image_offset"][i] = pix
        r = N // 2 - 1
        x = np.zeros((B, 3))
        x[:, :2] = g.uniform(-1.1 * r, 1.1 * r, (B, 2)) / (FREQ / C_LIGHT * (N * DL))
        uvw.append(x)
        vis.append((g.normal(size=B) + 1j * g.normal(size=B)).astype(np.complex64))
        flags.append((g.random(B) < flagged).astype(np.uint8))
        at += B
        pix += N * N
    uvw, vis, flags = np.concatenate(uvw), np.concatenate(vis), np.concatenate(flags)
    d = "cuda:0"
    out = torch.full((pix,), float("nan"), device=d)
    wsum = torch.zeros(n_img, dtype=torch.float64, device=d)
    nout = torch.zeros(n_img, dtype=torch.int32, device=d)
    status = torch.full((1,), -1, dtype=torch.int32, device=d)
    ctx.blink_image_batch_desc(torch.from_numpy(desc.view(np.uint8).copy()).to(d), torch.from_numpy(vis).to(d),
                               torch.from_numpy(uvw).to(d), torch.from_numpy(flags).to(d), out,
                               max_b or max(b for _, b in images), max_n or max(n for n, _ in images),
                               weighting=weighting, weight_sum=wsum, n_out=nout, status=status, precision=prec)
    torch.cuda.synchronize()
    assert int(status[0]) == 0
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    ref = None
    for i, (N, B) in enumerate(images):
        o, p = int(desc["vis_offset"][i]), int(desc["image_offset"][i])
        if ref is None or not share:
            if B == 0:
                ref = (np.zeros((N, N)), 0.0, 0)
            else:
                gr = oracle.grid(vis[o:o + B], flags[o:o + B], uvw[o:o + B], FREQ, N, DL, weighting)
                ref = (oracle.ifft2d(gr["grid"][0], gr["weight_sum"], shift=True)[0], gr["weight_sum"], gr["n_out"])
        img = got[p:p + N * N].reshape(N, N)
        assert float(wsum[i]) == ref[1] and int(nout[i]) == ref[2], i
        if ref[0].any():
            assert rel_l2(img, ref[0]) <= IMAGE_TOL[prec], (i, N, B)
        else:
            assert not img.any(), (i, N, B)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("weighting", [0, 1])
def test_every_size(torch, ctx, weighting, prec):
    sizes = [8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096]
    check(torch, ctx, "every size", [(n, b) for n in sizes for b in ((1, 65) if n > 2048 else (0, 1, 300, 64))],
          weighting, prec, max_b=301)


@pytest.mark.parametrize("n_img", [1, 7, 8, 9, 17])
def test_image_counts(torch, ctx, n_img):
    check(torch, ctx, "counts", [(128, 50 + i) for i in range(n_img)] + [(32, 9)] * n_img)


def test_more_images_than_the_workspace_holds(torch, ctx):
    check(torch, ctx, "several launches", [(64 >> i % 3, 30 + i % 7) for i in range(200)], max_b=4000)


@pytest.mark.parametrize("weighting", [0, 1])
def test_shared_pixels(torch, ctx, weighting):
    check(torch, ctx, "shared pixels", [(512, 400)] * 200, weighting, share=True)


@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("max_b", [8192, 8193, 16384, 16385])
def test_baseline_limits(torch, ctx, max_b, weighting):
    check(torch, ctx, "limits", [(256, max_b), (64, 100), (128, max_b - 1)], weighting)


def test_everything_flagged(torch, ctx):
    check(torch, ctx, "flagged", [(256, 100), (64, 3)], flagged=1.1)
