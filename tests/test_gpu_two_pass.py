"""The two-pass form at 512^2 and above, which serves more than 16384 baselines (and the descriptor form's chunks there): every
compiled strip width, row block and loop of blink_image_batch, and the chunked uneven batch, in every precision form
and weighting, against the FP64 oracle: weight sums and out-of-grid counts bit-exact, images within a relative
L2 of 1e-5 (FP32) or 1e-3 (split forms). The workspace is filled with 0xFF bytes (NaN), the coverage leaves columns
empty, and every case makes sure from the kernel timing that row kernels ran.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

IMAGE_TOL = {0: 1e-5, 1: 1e-3, 2: 1e-3}
FREQ = 150.0e6
DL = 1.0e-3
B = 16385


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


def coverage(g, N, n, extent):
    x = np.zeros((n, 3))
    x[:, 0] = g.uniform(-extent * N / 2, extent * N / 2, n)
    x[:, 1] = g.uniform(-0.52 * N, 0.52 * N, n)               # some outside the grid
    x[:, :2] /= FREQ / 299792458.0 * (N * DL)
    return x


def rel_l2(torch, got, ref):
    got = got.double()
    return float(torch.linalg.vector_norm(got - ref) / torch.linalg.vector_norm(ref))


def with_rows(ctx, torch, call):
    """call(), which has to launch row kernels."""
    ctx.profile_enable(True)
    res = call()
    torch.cuda.synchronize()
    assert ctx.profile_read()["row_fft"][1] > 0, "folded, not two-pass"
    ctx.profile_enable(False)
    return res


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("N", [512, 1024, 2048, 4096])
def test_every_plan(torch, ctx, N, weighting, prec):
    import paper_2505_15204_amd as blink

    g = np.random.default_rng(N)
    C, d = 2, "cuda:0"
    uvw = coverage(g, N, B, 0.8)[None]
    vis = (g.normal(size=(1, C, 1, B)) + 1j * g.normal(size=(1, C, 1, B))).astype(np.complex64)
    flags = (g.random((1, C, B)) < 0.7).astype(np.uint8)
    freq = np.array([FREQ, FREQ * 0.999])
    ref = oracle.image_batch(vis, flags, uvw, freq, N, DL, weighting)
    images = torch.from_numpy(np.ascontiguousarray(ref["images"])).to(d).double()
    dev = [torch.from_numpy(x).to(d) for x in (vis, flags, uvw, freq)]
    ws = torch.empty(blink.image_batch_workspace_size(1, C, 1, B, N, weighting, prec), dtype=torch.uint8, device=d)
    cols, rows = blink.plan_options(N, weighting)
    default = ctx.get_plan(N, weighting, prec)
    plans = [(c, r, 1 if i % 2 else 0, 1) for i, c in enumerate(cols) for r in rows] + [(c, rows[0], 0, n) for c in cols for n in (3, 4)]
    try:
        for col, row, group, loop in plans:
            print(f"[gpu-case] two-pass N={N} w={weighting} prec={prec} {col, row, group, loop}", flush=True)
            ctx.set_plan(N, weighting, col, row, group, precision=prec, col_loop=loop)
            ws.fill_(255)
            res = with_rows(ctx, torch, lambda: ctx.blink_image_batch(*dev, N, DL, weighting, precision=prec, workspace=ws))
            assert np.array_equal(res["weight_sum"].cpu().numpy(), ref["weight_sum"])
            assert np.array_equal(res["n_out"].cpu().numpy(), ref["n_out"])
            for c in range(C):
                assert rel_l2(torch, res["images"][0, c, 0], images[0, c, 0]) <= IMAGE_TOL[prec], (col, row, group, loop, c)
    finally:
        ctx.set_plan(N, weighting, default["col_strip"], default["row_block"], default["group"], precision=prec,
                     col_loop=default["col_loop"])


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("weighting", [0, 1])
def test_chunks_of_an_uneven_batch(torch, ctx, weighting, prec):
    import paper_2505_15204_amd as blink

    g = np.random.default_rng(31)
    d = "cuda:0"
    sizes = [(4096, 300), (512, B), (2048, 900), (1024, 4000), (512, 64), (1024, 0), (2048, 1), (512, 5000)]
    desc = np.zeros(len(sizes), blink.DESC_DTYPE)
    uvw, at, pix = [], 0, 0
    for i, (N, n) in enumerate(sizes):
        desc["grid_n"][i], desc["n_baselines"][i], desc["freq_hz"][i], desc["pixel_scale"][i] = N, n, FREQ, DL
        for f in ("vis_offset", "uvw_offset", "flag_offset"):
            desc[f][i] = at
        desc["image_offset"][i] = pix
        uvw.append(coverage(g, N, n, 0.7))
        at += n
        pix += N * N
    uvw = np.concatenate(uvw)
    vis = (g.normal(size=at) + 1j * g.normal(size=at)).astype(np.complex64)
    flags = (g.random(at) < 0.1).astype(np.uint8)
    flags[int(desc["flag_offset"][6])] = 0
    uvw[int(desc["uvw_offset"][6]), :2] = 0.3 / (FREQ / 299792458.0 * (2048 * DL))
    out = torch.full((pix,), float("nan"), device=d)
    wsum = torch.zeros(len(sizes), dtype=torch.float64, device=d)
    nout = torch.zeros(len(sizes), dtype=torch.int32, device=d)
    status = torch.full((1,), -1, dtype=torch.int32, device=d)
    ws = torch.full((blink.desc_workspace_size(len(sizes), B, 4096),), 255, dtype=torch.uint8, device=d)
    print(f"[gpu-case] chunked uneven batch w={weighting} prec={prec}", flush=True)
    args = [torch.from_numpy(x).to(d) for x in (desc.view(np.uint8).copy(), vis, uvw, flags)]
    with_rows(ctx, torch, lambda: ctx.blink_image_batch_desc(*args, out, B, 4096, weighting=weighting, precision=prec,
                                                             weight_sum=wsum, n_out=nout, status=status, workspace=ws))
    assert int(status[0]) == 0
    for i, (N, n) in enumerate(sizes):
        o, p = int(desc["vis_offset"][i]), int(desc["image_offset"][i])
        img = out[p:p + N * N].view(N, N)
        if n == 0:
            assert not img.any() and float(wsum[i]) == 0.0
            continue
        gr = oracle.grid(vis[o:o + n], flags[o:o + n], uvw[o:o + n], FREQ, N, DL, weighting)
        want = torch.from_numpy(np.ascontiguousarray(oracle.ifft2d(gr["grid"][0], gr["weight_sum"], shift=True)[0])).to(d).double()
        assert float(wsum[i]) == gr["weight_sum"] and int(nout[i]) == gr["n_out"], i
        assert rel_l2(torch, img, want) <= IMAGE_TOL[prec], (i, N, n)
