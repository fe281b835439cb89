"""Which form a call takes, by the launches that the context's kernel timing counts: the two-pass form
launches row kernels, the folded form none.
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


@pytest.fixture(scope="module")
def ctx(torch):
    import paper_2505_15204_amd as blink
    c = blink.Context(0)
    yield c
    c.close()


def row_launches(torch, ctx, call):
    ctx.profile_enable(True)
    call()
    torch.cuda.synchronize()
    launches = ctx.profile_read()["row_fft"][1]
    ctx.profile_enable(False)
    return launches


def image_call(torch, ctx, B, N, C, weighting, prec, P=1):
    g = np.random.default_rng(B + N)
    d = "cuda:0"
    uvw = np.zeros((1, B, 3))
    uvw[0, :, :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (B, 2)) / (FREQ / 299792458.0 * (N * DL))
    vis = torch.randn((1, C, P, B), device=d, dtype=torch.complex64)
    uvw, freq = torch.from_numpy(uvw).to(d), torch.full((C,), FREQ, dtype=torch.float64, device=d)
    return lambda: ctx.blink_image_batch(vis, None, uvw, freq, N, DL, weighting, precision=prec)


# both sides of the lines at 256^2, and the sizes beside it
@pytest.mark.parametrize("B,N,C,weighting,prec,folded", [
    (4095, 256, 191, 0, 0, False), (300, 256, 192, 0, 0, True), (4096, 256, 1, 0, 0, True), (4096, 256, 1, 0, 2, True),
    (4096, 256, 63, 0, 1, False), (4096, 256, 64, 0, 1, True), (4096, 256, 1, 1, 0, False), (8128, 256, 127, 1, 0, False),
    (8128, 256, 128, 1, 0, True), (8128, 256, 127, 1, 1, False), (300, 256, 192, 1, 2, True), (45, 512, 1, 1, 1, True),
    (8128, 128, 300, 0, 0, False), (16384, 512, 1, 0, 0, True), (16385, 512, 1, 0, 0, False)])
def test_image_batch(torch, ctx, B, N, C, weighting, prec, folded):
    print(f"[gpu-case] route B={B} N={N} C={C} w={weighting} prec={prec}", flush=True)
    assert (row_launches(torch, ctx, image_call(torch, ctx, B, N, C, weighting, prec)) == 0) == folded


# several images of a pair, and lists that outgrow the workspace query at 256^2
@pytest.mark.parametrize("B,C,P,folded", [(8128, 1, 3, True), (8128, 1, 4, False), (8128, 4, 16, True), (16384, 4, 16, False)])
def test_polarisations(torch, ctx, B, C, P, folded):
    print(f"[gpu-case] route B={B} C={C} P={P}", flush=True)
    assert (row_launches(torch, ctx, image_call(torch, ctx, B, 256, C, 0, 0, P)) == 0) == folded


def desc_call(torch, ctx, N, B, n_img):
    import paper_2505_15204_amd as blink

    g = np.random.default_rng(B + N)
    d = "cuda:0"
    desc = np.zeros(n_img, blink.DESC_DTYPE)
    desc["grid_n"], desc["n_baselines"], desc["freq_hz"], desc["pixel_scale"] = N, B, FREQ, DL
    desc["image_offset"] = np.arange(n_img) * N * N
    uvw = np.zeros((B, 3))                           # every image reads the same visibilities
    uvw[:, :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (B, 2)) / (FREQ / 299792458.0 * (N * DL))
    vis = torch.randn((B,), device=d, dtype=torch.complex64)
    out = torch.empty(n_img * N * N, device=d)
    ws = torch.empty(blink.desc_workspace_size(n_img, B, N) + (1 << 26), dtype=torch.uint8, device=d)
    desc, uvw = torch.from_numpy(desc.view(np.uint8).copy()).to(d), torch.from_numpy(uvw).to(d)
    return lambda: ctx.blink_image_batch_desc(desc, vis, uvw, None, out, B, N, workspace=ws)


@pytest.mark.parametrize("N,B,n_img,folded", [(128, 45, 20, True), (64, 8000, 400, False), (64, 4096, 1024, True),
                                              (64, 45, 1024, False), (32, 4095, 400, False), (32, 4096, 100, True),
                                              (16, 45, 400, False), (16, 2048, 100, True), (8, 45, 2000, False)])
def test_uneven_batch(torch, ctx, N, B, n_img, folded):
    print(f"[gpu-case] route uneven N={N} B={B} n_img={n_img}", flush=True)
    ctx.set_desc_plan(512, 0, form=1)
    assert (row_launches(torch, ctx, desc_call(torch, ctx, N, B, n_img)) == 0) == folded
