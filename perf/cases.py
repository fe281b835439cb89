"""The measured work of this framework: dirty imaging of MWA-shaped visibilities and the steps
before and after it (correlation, averaging, de-dispersion), each through the binding's public
entry points with the tuned execution plans loaded.

A case is a dict with an "op" and the sizes that op takes:

  image      blink_image_batch: T x C x P images of N^2, natural or uniform weighting, any precision form
  corrected  blink_image_batch_corrected: the same on visibilities corrected by antenna factors and moved
             to another phase centre
  conv       blink_image_batch_conv: convolutional gridding
  uneven     blink_image_batch_desc: images of different grid sizes and visibility counts in one call
  dense      blink_grid, then blink_ifft2d of its grids
  correlate  blink_correlate: int8 voltages to visibilities
  average    blink_image_average: Stokes I and band averages of image cubes
  dedisperse blink_dedisperse: trial-DM sums of an image cube

Inputs follow synth.py: a dense core plus a disc of tiles, 50 point sources, Gaussian noise of 0.1 Jy,
10% flags; tiles, sky, noise and flags are drawn from the seed.
"""
import math

import numpy as np
import torch

import paper_2505_15204_amd as blink
from paper_2505_15204_amd import synth

DEV = "cuda:0"
C_LIGHT = synth.C_LIGHT


def listed():
    return [
        # the smallest call: one channel, one polarisation, 256^2 (the "tiny" workload): latency
        dict(name="tiny-256", op="image", tiles=128, T=1, C=1, P=1, N=256, pixel=1.0, f0=150.0e6, df=40.0e3,
             weighting=0, precision=0, flagged=0.0),
        # one coarse channel (32 x 40 kHz) of one time step, both polarisations: an ordinary call
        dict(name="coarse-1024", op="image", tiles=128, T=1, C=32, P=2, N=1024, pixel=1.0, f0=150.52e6, df=40.0e3,
             weighting=0, precision=0, flagged=0.1),
        # the headline workload: one time step of the whole VCS band
        dict(name="vcs-1024", op="image", tiles=128, T=1, C=768, P=2, N=1024, pixel=1.0, f0=139.0e6, df=40.0e3,
             weighting=0, precision=0, flagged=0.1),
        # Phase II shape: 144 tiles, 2048^2, uniform weighting, a slice of 32 fine channels
        dict(name="phase2-2048-uniform", op="image", tiles=144, T=1, C=32, P=2, N=2048, pixel=0.75, f0=185.0e6,
             df=10.0e3, weighting=1, precision=0, flagged=0.1),
        # the largest grids, one polarisation, in the split FP16 form
        dict(name="precision-4096-f16", op="image", tiles=128, T=1, C=16, P=1, N=4096, pixel=1.0, f0=139.0e6,
             df=120.0e3, weighting=0, precision=1, flagged=0.1),
        # calibrated imaging of a smaller array over several time steps: odd counts, ragged sizes
        dict(name="corrected-512", op="corrected", tiles=100, T=5, C=13, P=2, N=512, pixel=2.0, f0=170.0e6, df=160.0e3,
             weighting=0, precision=0, flagged=0.1),
        # convolutional gridding at its documented width
        dict(name="conv-1024-w8", op="conv", tiles=128, T=1, C=96, P=2, N=1024, pixel=1.0, f0=139.0e6, df=320.0e3,
             width=8, precision=0, flagged=0.1),
        # uneven batch: 70-300 MHz, 512^2 .. 2048^2, 70-100% of the baselines per image
        dict(name="uneven-2048", op="uneven", tiles=128, images=400, n_lo=512, precision=0),
        # grids kept by the caller, transformed by a second call
        dict(name="dense-512", op="dense", tiles=128, T=2, C=24, P=2, N=512, pixel=2.0, f0=150.0e6, df=40.0e3,
             weighting=1, precision=0, flagged=0.1),
        # correlator: 10 kHz fine channels averaged by 4, 100 us samples integrated to 20 ms
        dict(name="correlate-128", op="correlate", tiles=128, T=2, C=384, n_int=200, n_favg=4, pol_mode=4),
        # Stokes I and band average of one time step's images
        dict(name="average-1024", op="average", T=1, C=768, P=2, N=1024, axes=6),
        # FRB search cube: 50 ms steps, the whole band, 16 trial DMs up to 10 pc cm^-3
        dict(name="dedisperse-512", op="dedisperse", T=40, C=768, N=512, n_dm=16, dm_max=10.0, dt=0.05),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["image", "image", "image", "corrected", "conv", "uneven", "dense", "correlate", "average",
                     "dedisperse"])
    tiles = rng.randint(24, 144)
    if op == "uneven":
        return dict(op=op, tiles=tiles, images=_log_int(rng, 20, 400), n_lo=rng.choice([128, 256, 512]),
                    precision=rng.choice([0, 0, 1, 2]))
    if op == "correlate":
        return dict(op=op, tiles=4 * rng.randint(4, 36), T=rng.randint(1, 5), C=_log_int(rng, 8, 300),
                    n_int=rng.randint(20, 200), n_favg=rng.choice([1, 2, 4]), pol_mode=rng.choice([2, 4]))
    if op == "average":
        N = rng.choice([256, 512, 1024, 2048])
        T, P = rng.randint(1, 6), rng.randint(1, 2)
        return dict(op=op, T=T, C=_log_int(rng, 3, max(4, (700 << 20) // (N * N * T * P))), P=P, N=N,
                    axes=rng.choice([1, 2, 3, 6, 7] if P == 2 else [1, 2, 3]))
    if op == "dedisperse":
        T = rng.randint(20, 60)
        return dict(op=op, T=T, C=_log_int(rng, 24, 400), N=rng.choice([128, 256, 512]), n_dm=rng.randint(2, 24),
                    dm_max=rng.uniform(2.0, 12.0), dt=rng.choice([0.05, 0.1]))
    N = rng.choice([128, 256, 512, 1024, 1024, 2048] + ([4096] if op == "image" else []))
    P = rng.choice([1, 2])
    # all drawn batches stay well below the headline workload's pixels
    pairs = _log_int(rng, 1, max(2, ((128 if op == "dense" else 400) << 20) // (N * N * P * (4 if op == "conv" else 1))))
    T = rng.randint(1, max(1, min(8, pairs)))
    c = dict(op=op, tiles=tiles, T=T, C=max(1, min(768, pairs // T)), P=P, N=N,
             pixel=round(max(0.75, 1024.0 / N) * rng.uniform(0.8, 1.1), 4), f0=rng.uniform(120e6, 190e6),
             df=rng.choice([10.0e3, 40.0e3]), flagged=rng.choice([0.0, 0.05, 0.1]))
    if op == "conv":
        return dict(c, width=rng.randint(4, 10), precision=0)
    return dict(c, weighting=rng.choice([0, 0, 1]), precision=0 if op == "dense" else rng.choice([0, 0, 0, 1, 2]))


# ---------------------------------------------------------------------------- inputs
_ctx = None


def _context():
    """One library context with the tuned plans, as a program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = blink.Context(0)
        _ctx.load_plans(blink.PLANS_PATH)
    return _ctx


def _rngs(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1))
    return np.random.default_rng(seed), g


def _observation(case, seed):
    """uvw_m [T][B][3], freq_hz [C], flags [T][C][B] and vis [T][C][P][B] on the GPU."""
    host, g = _rngs(seed)
    T, C, P = case["T"], case["C"], case["P"]
    pos = synth.tile_positions(case["tiles"], host)
    uvw = synth.baseline_uvw(pos)
    height = host.normal(0.0, 3.0, case["tiles"])
    i, j = np.tril_indices(case["tiles"], -1)
    uvw[:, 2] = height[i] - height[j]
    s, l, m = (torch.from_numpy(x).to(DEV) for x in synth.sky_model(50, host))
    B = uvw.shape[0]
    uvw_t = np.empty((T, B, 3))
    for t in range(T):                                  # the sky turns between the time steps
        a = 1.0e-3 * t
        uvw_t[t, :, 0] = math.cos(a) * uvw[:, 0] - math.sin(a) * uvw[:, 1]
        uvw_t[t, :, 1] = math.sin(a) * uvw[:, 0] + math.cos(a) * uvw[:, 1]
        uvw_t[t, :, 2] = uvw[:, 2]
    uvw_d = torch.from_numpy(uvw_t).to(DEV)
    freq = torch.from_numpy(case["f0"] + case["df"] * (np.arange(C) + 0.5)).to(DEV)
    vis = torch.randn((T, C, P, B, 2), generator=g, device=DEV) * 0.1
    for t in range(T):
        ul = uvw_d[t, :, 0:1] * l[None] + uvw_d[t, :, 1:2] * m[None]
        for c0 in range(0, C, 64):
            ph = (-2.0 * math.pi / C_LIGHT) * freq[c0:c0 + 64, None, None] * ul[None]
            vis[t, c0:c0 + 64, :, :, 0] += (torch.cos(ph) @ s).float()[:, None]
            vis[t, c0:c0 + 64, :, :, 1] += (torch.sin(ph) @ s).float()[:, None]
    flags = (torch.rand((T, C, B), generator=g, device=DEV) < case["flagged"]).to(torch.uint8)
    return dict(uvw_m=uvw_d, freq_hz=freq, flags=flags, vis=torch.view_as_complex(vis), pixel=case["pixel"] * synth.ARCMIN)


def _gains(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(7919 * (seed + 1))
    shape = (case["C"], case["P"], case["tiles"])
    amp = 0.5 + torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
    pha = 2 * math.pi * torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
    return torch.polar(amp, pha).to(torch.complex64)


PHASE_CENTRE = (0.02, -0.015)


def _uneven(case, seed):
    n = case["n_lo"]
    return synth.uneven_layout(n_img=case["images"], config=100 + seed % (1 << 31), n_tiles=case["tiles"],
                               sizes=(n, 2 * n, 4 * n))


def _delays(case):
    freq = 139.0e6 + 30.72e6 / case["C"] * (np.arange(case["C"]) + 0.5)
    return blink.dispersion_delays(freq, case["dt"], np.linspace(0.0, case["dm_max"], case["n_dm"]))


def _steps(case):
    """Output time steps of a de-dispersion: those for which every delay stays inside the cube."""
    return max(1, case["T"] - int(_delays(case).max()))


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    op, ctx = case["op"], _context()
    st = dict(op=op, case=case, ctx=ctx)
    if op in ("image", "corrected", "conv", "dense"):
        T, C, P, N = case["T"], case["C"], case["P"], case["N"]
        st.update(_observation(case, seed))
        B = st["vis"].shape[-1]
        w, p = case.get("weighting", 0), case["precision"]
        if op == "image":
            n = blink.image_batch_workspace_size(T, C, P, B, N, w, p)
        elif op == "corrected":
            n = blink.image_batch_corrected_workspace_size(T, C, P, B, N, w, p)
            st["gains"] = _gains(case, seed)
        elif op == "conv":
            n = blink.image_batch_conv_workspace_size(T, C, P, B, N, case["width"], p)
        else:
            n = blink.grid_workspace_size(T, C, B, N)
            st["ws2"] = _bytes(blink.ifft2d_workspace_size(T * C * P, N, p))
        st["ws"] = _bytes(n)
        st["images"] = torch.empty((T, C, P, N, N), dtype=torch.float32, device=DEV)
        st["weight_sum"] = torch.empty((T, C, P), dtype=torch.float64, device=DEV)
        st["n_out"] = torch.empty((T, C), dtype=torch.int32, device=DEV)
    elif op == "uneven":
        lay = _uneven(case, seed)
        st["vis"] = synth.uneven_vis_device(lay, DEV, seed=seed)
        st["uvw_m"] = torch.from_numpy(lay["uvw_ext"]).to(DEV)
        st["desc"] = torch.from_numpy(synth.uneven_descriptors(lay, blink.DESC_DTYPE).view(np.uint8).copy()).to(DEV)
        st["max_b"], st["max_n"] = lay["max_b"], lay["max_n"]
        st["images"] = torch.empty(lay["images_len"], dtype=torch.float32, device=DEV)
        st["weight_sum"] = torch.empty(lay["n_img"], dtype=torch.float64, device=DEV)
        st["n_out"] = torch.empty(lay["n_img"], dtype=torch.int32, device=DEV)
        st["status"] = torch.empty(1, dtype=torch.int32, device=DEV)
        st["ws"] = _bytes(blink.desc_workspace_size(lay["n_img"], lay["max_b"], lay["max_n"]))
    elif op == "correlate":
        _, g = _rngs(seed)
        A, B = case["tiles"], case["tiles"] * (case["tiles"] - 1) // 2
        S, F = case["T"] * case["n_int"], case["C"] * case["n_favg"]
        st["volt"] = torch.randint(-128, 128, (S, F, A, 2, 2), generator=g, device=DEV, dtype=torch.int8)
        st["vis"] = torch.empty((case["T"], case["C"], case["pol_mode"], B), dtype=torch.complex64, device=DEV)
    else:
        _, g = _rngs(seed)
        T, C, P, N = case["T"], case["C"], case.get("P", 1), case["N"]
        cube = torch.randn((T, C, P, N, N), generator=g, device=DEV)
        if op == "average":
            a = case["axes"]
            st["images"] = cube
            st["out"] = torch.empty((1 if a & 1 else T, 1 if a & 2 else C, 1 if a & 4 else P, N, N), device=DEV)
        else:
            st["images"] = cube.view(T, C, N, N)
            st["delays"] = np.minimum(_delays(case), T - 1)
            st["out"] = torch.empty((case["n_dm"], _steps(case), N, N), device=DEV)
            st["ws"] = _bytes(blink.dedisperse_workspace_size(C, case["n_dm"]))
    return st


def run(st):
    op, case, ctx = st["op"], st["case"], st["ctx"]
    if op == "image":
        return ctx.blink_image_batch(st["vis"], st["flags"], st["uvw_m"], st["freq_hz"], case["N"], st["pixel"],
                                     case["weighting"], precision=case["precision"], out=st["images"],
                                     weight_sum=st["weight_sum"], n_out=st["n_out"], workspace=st["ws"])
    if op == "corrected":
        return ctx.blink_image_batch_corrected(st["vis"], st["flags"], st["uvw_m"], st["freq_hz"], case["N"],
                                               st["pixel"], case["weighting"], gains=st["gains"], l0=PHASE_CENTRE[0],
                                               m0=PHASE_CENTRE[1], precision=case["precision"], out=st["images"],
                                               weight_sum=st["weight_sum"], n_out=st["n_out"], workspace=st["ws"])
    if op == "conv":
        return ctx.blink_image_batch_conv(st["vis"], st["flags"], st["uvw_m"], st["freq_hz"], case["N"], st["pixel"],
                                          kernel_width=case["width"], kernel_beta=2.3 * case["width"],
                                          precision=case["precision"], out=st["images"], weight_sum=st["weight_sum"],
                                          n_out=st["n_out"], workspace=st["ws"])
    if op == "uneven":
        images = ctx.blink_image_batch_desc(st["desc"], st["vis"], st["uvw_m"], None, st["images"], st["max_b"],
                                            st["max_n"], precision=case["precision"], weight_sum=st["weight_sum"],
                                            n_out=st["n_out"], status=st["status"], workspace=st["ws"])
        return dict(images=images, weight_sum=st["weight_sum"], n_out=st["n_out"], status=st["status"])
    if op == "dense":
        res = ctx.blink_grid(st["vis"], st["flags"], st["uvw_m"], st["freq_hz"], case["N"], st["pixel"],
                             case["weighting"], workspace=st["ws"])
        res["images"] = ctx.blink_ifft2d(res["grids"], res["weight_sum"], precision=case["precision"],
                                         out=st["images"], workspace=st["ws2"])
        return res
    if op == "correlate":
        return ctx.blink_correlate(st["volt"], case["n_int"], case["n_favg"], case["pol_mode"], out=st["vis"])["vis"]
    if op == "average":
        return ctx.blink_image_average(st["images"], case["axes"], out=st["out"])
    return ctx.blink_dedisperse(st["images"], st["delays"], st["out"].shape[1], out=st["out"], workspace=st["ws"])


# ---------------------------------------------------------------------------- what a pass cannot do without
def _fft_flops(N):
    """Real-output 2D transform of one N^2 image: half of 5 n log2 n, n = N^2."""
    return 2.5 * N * N * 2 * math.log2(N)


def work(case):
    op = case["op"]
    if op in ("image", "corrected", "conv", "dense"):
        T, C, P, N = case["T"], case["C"], case["P"], case["N"]
        B = case["tiles"] * (case["tiles"] - 1) // 2
        n_img = T * C * P
        nbytes = T * C * B * (8 * P + 1) + 24 * T * B + 8 * C + n_img * (4 * N * N + 8) + 4 * T * C
        flops = n_img * (_fft_flops(N) + 4 * B)
        if op == "corrected":
            nbytes += 8 * C * P * case["tiles"]
            flops += n_img * B * 24
        if op == "conv":
            flops += n_img * 2 * B * 4 * case["width"] ** 2
        if op == "dense":                               # grids written, then read; counts and cells written
            nbytes += n_img * 16 * N * N + T * C * (4 * N * N + 4 * B)
        return dict(bytes=nbytes, flops=flops)
    if op == "uneven":
        lay = _uneven(case, 0)
        n = lay["grid_n"].astype(np.float64)
        return dict(bytes=float((4 * n * n).sum() + 8 * lay["vis_len"] + 24 * lay["B"] + 76 * lay["n_img"]),
                    flops=float((2.5 * n * n * 2 * np.log2(n)).sum() + 4 * lay["vis_len"]))
    if op == "correlate":
        A, T, C, K = case["tiles"], case["T"], case["C"], case["n_int"] * case["n_favg"]
        B = A * (A - 1) // 2
        return dict(bytes=T * C * (K * A * 4 + case["pol_mode"] * B * 8), flops=T * C * B * case["pol_mode"] * K * 8)
    N2 = case["N"] ** 2
    if op == "average":
        T, C, P, a = case["T"], case["C"], case["P"], case["axes"]
        n_out = (1 if a & 1 else T) * (1 if a & 2 else C) * (1 if a & 4 else P)
        return dict(bytes=4 * N2 * (T * C * P + n_out), flops=N2 * T * C * P)
    t_out = _steps(case)
    d = np.minimum(_delays(case), case["T"] - 1)
    used = sum(len({int(x) + t for x in np.unique(d[:, c]) for t in range(t_out)}) for c in range(case["C"]))
    return dict(bytes=4 * N2 * (used + case["n_dm"] * t_out), flops=N2 * case["n_dm"] * t_out * case["C"])


# ---------------------------------------------------------------------------- the same in 64 bits, in plain torch
def _cells(x, N):
    """Nearest cells of coordinates x = u k (ties to even) and whether they lie on the grid."""
    r = torch.round(x)
    return r, torch.abs(r) < N // 2


def _to_image(G, W, N):
    """Re(IDFT2(G)) / W, unnormalised transform, phase centre at (N/2, N/2)."""
    img = torch.fft.fftshift(torch.fft.ifft2(G).real * float(N * N), dim=(-2, -1))
    return img / W[:, None, None] if float(W.min()) > 0 else torch.zeros_like(img)


def _grid_pair(V, uvw, ok, k, N, uniform):
    """Nearest-cell grids [P][N][N] and weight sums of one (time, channel) pair; V complex128 [P][B]."""
    iu, on_u = _cells(uvw[:, 0] * k, N)
    iv, on_v = _cells(uvw[:, 1] * k, N)
    keep = ok & on_u & on_v
    iu, iv, V = iu[keep].long(), iv[keep].long(), V[:, keep]
    cell = torch.cat([(iv % N) * N + iu % N, ((-iv) % N) * N + (-iu) % N])
    G = torch.zeros((V.shape[0], N * N), dtype=torch.complex128, device=DEV)
    G.index_add_(1, cell, torch.cat([V, V.conj()], dim=1))
    W = float(cell.numel())
    if uniform:
        n = torch.bincount(cell, minlength=N * N)
        G /= torch.clamp(n, min=1)
        W = float((n > 0).sum())
    return G.view(-1, N, N), torch.full((V.shape[0],), W, dtype=torch.float64, device=DEV)


def _corrected(V, uvw, f, gains, tiles):
    i, j = (torch.from_numpy(x).to(DEV) for x in np.tril_indices(tiles, -1))
    l0, m0 = PHASE_CENTRE
    n0 = math.sqrt(1.0 - l0 * l0 - m0 * m0)
    turns = (f / C_LIGHT) * (uvw[:, 0] * l0 + uvw[:, 1] * m0 + uvw[:, 2] * (n0 - 1.0))
    J = gains.to(torch.complex128)
    return J[:, i] * V * J[:, j].conj() * torch.polar(torch.ones_like(turns), 2 * math.pi * turns)


def _conv_pair(V, uvw, ok, k, N, width, beta):
    """Spread grids [P][N][N] and weight sums of one pair (exponential-of-semicircle kernel)."""
    x, y = uvw[:, 0] * k, uvw[:, 1] * k
    keep = ok & _cells(x, N)[1] & _cells(y, N)[1]
    x, y, V = x[keep], y[keep], V[:, keep]
    x, y, V = torch.cat([x, -x]), torch.cat([y, -y]), torch.cat([V, V.conj()], dim=1)
    h = 0.5 * width

    def taps(p):
        j = torch.floor(p - h)[:, None] + torch.arange(width + 2, device=DEV, dtype=torch.float64)
        z = (j - p[:, None]) / h
        w = torch.where(z.abs() < 1, torch.exp(beta * (torch.sqrt(torch.clamp(1 - z * z, min=0.0)) - 1.0)), 0.0)
        return j.long() % N, w

    ju, wu = taps(x)
    jv, wv = taps(y)
    cell = (jv[:, :, None] * N + ju[:, None, :]).reshape(-1)
    w = (wv[:, :, None] * wu[:, None, :])
    G = torch.zeros((V.shape[0], N * N), dtype=torch.complex128, device=DEV)
    for p in range(V.shape[0]):
        G[p].index_add_(0, cell, (V[p][:, None, None] * w).reshape(-1))
    return G.view(-1, N, N), torch.full((V.shape[0],), float(x.numel()), dtype=torch.float64, device=DEV)


def _conv_correction(N, width, beta):
    """The kernel's Fourier transform at pixel offsets X/N, X = -N/2 .. N/2 - 1 (d = (W/2) sin t, Gauss-Legendre)."""
    t, w = np.polynomial.legendre.leggauss(200)
    t, w = (t + 1.0) * math.pi / 4.0, w * math.pi / 4.0
    nu = (np.arange(N) - N // 2) / N
    f = np.exp(beta * (np.cos(t) - 1.0)) * np.cos(t) * w
    return torch.from_numpy(width * (np.cos(math.pi * width * nu[:, None] * np.sin(t)[None]) @ f)).to(DEV)


def _exact_imaging(case, seed):
    op, N, P = case["op"], case["N"], case["P"]
    d = _observation(case, seed)
    T, C, B = case["T"], case["C"], d["vis"].shape[-1]
    gains = _gains(case, seed) if op == "corrected" else None
    images = torch.empty((T, C, P, N, N), dtype=torch.float64, device=DEV)
    weight_sum = torch.empty((T, C, P), dtype=torch.float64, device=DEV)
    grids = torch.empty((T, C, P, N, N), dtype=torch.complex128, device=DEV) if op == "dense" else None
    corr = _conv_correction(N, case["width"], 2.3 * case["width"]) if op == "conv" else None
    freq = d["freq_hz"].cpu().numpy()
    for t in range(T):
        for c in range(C):
            k = (float(freq[c]) / C_LIGHT) * (float(N) * d["pixel"])
            V, uvw, ok = d["vis"][t, c].to(torch.complex128), d["uvw_m"][t], d["flags"][t, c] == 0
            if op == "conv":
                G, W = _conv_pair(V, uvw, ok, k, N, case["width"], 2.3 * case["width"])
            else:
                if op == "corrected":
                    V = _corrected(V, uvw, float(freq[c]), gains[c], case["tiles"])
                G, W = _grid_pair(V, uvw, ok, k, N, case["weighting"] == 1)
            img = _to_image(G, W, N)
            images[t, c] = img / (corr[:, None] * corr[None]) if op == "conv" else img
            weight_sum[t, c] = W
            if grids is not None:
                grids[t, c] = G
    out = dict(images=images, weight_sum=weight_sum, n_out=None)
    return dict(out, grids=grids, counts=None, cell_idx=None) if op == "dense" else out


def _exact_uneven(case, seed):
    lay = _uneven(case, seed)
    vis = synth.uneven_vis_device(lay, DEV, seed=seed).to(torch.complex128)
    ext = torch.from_numpy(lay["uvw_ext"]).to(DEV)
    images = torch.empty(lay["images_len"], dtype=torch.float64, device=DEV)
    weight_sum = torch.empty(lay["n_img"], dtype=torch.float64, device=DEV)
    for i in range(lay["n_img"]):
        n, N = int(lay["n_baselines"][i]), int(lay["grid_n"][i])
        u, v, o = int(lay["uvw_offset"][i]), int(lay["vis_offset"][i]), int(lay["image_offset"][i])
        k = (float(lay["freq_hz"][i]) / C_LIGHT) * (float(N) * float(lay["pixel_scale"][i]))
        ok = torch.ones(n, dtype=torch.bool, device=DEV)
        G, W = _grid_pair(vis[None, v:v + n], ext[u:u + n], ok, k, N, False)
        images[o:o + N * N] = _to_image(G, W, N).reshape(-1)
        weight_sum[i] = W[0]
    return dict(images=images, weight_sum=weight_sum, n_out=None, status=None)


def _exact_correlate(case, seed):
    volt = prepare(case, seed)["volt"]
    T, C, A, n_int, n_favg = case["T"], case["C"], case["tiles"], case["n_int"], case["n_favg"]
    i, j = (torch.from_numpy(x).to(DEV) for x in np.tril_indices(A, -1))
    out = torch.empty((T, C, case["pol_mode"], i.numel()), dtype=torch.complex128, device=DEV)
    products = [(0, 0), (0, 1), (1, 0), (1, 1)] if case["pol_mode"] == 4 else [(0, 0), (1, 1)]
    for t in range(T):
        for c in range(C):
            x = volt[t * n_int:(t + 1) * n_int, c * n_favg:(c + 1) * n_favg].reshape(-1, 2 * A, 2).double()
            re, im = x[..., 0], x[..., 1]
            ret, imt = re.t().contiguous(), im.t().contiguous()
            Rr, Ri = ret @ re + imt @ im, imt @ re - ret @ im
            for q, (a, b) in enumerate(products):
                out[t, c, q] = torch.complex(Rr[2 * i + a, 2 * j + b], Ri[2 * i + a, 2 * j + b]) / x.shape[0]
    return out


def exact(case, seed):
    op = case["op"]
    if op in ("image", "corrected", "conv", "dense"):
        return _exact_imaging(case, seed)
    if op == "uneven":
        return _exact_uneven(case, seed)
    if op == "correlate":
        return _exact_correlate(case, seed)
    st = prepare(case, seed)
    x = st["images"]
    if op == "average":
        axes = [k for k, bit in enumerate((1, 2, 4)) if case["axes"] & bit]
        acc = torch.zeros(st["out"].shape, dtype=torch.float64, device=DEV)
        for c in range(x.shape[1]):                     # channel by channel: the cube in 64 bits would be large
            s = x[:, c:c + 1].double()
            for k in (0, 2):
                s = s.sum(dim=k, keepdim=True) if k in axes else s
            if 1 in axes:
                acc += s
            else:
                acc[:, c:c + 1] = s
        return acc / math.prod(x.shape[k] for k in axes)
    out = torch.zeros(st["out"].shape, dtype=torch.float64, device=DEV)
    for c in range(x.shape[1]):
        s = x[:, c].double()
        for k in range(out.shape[0]):
            d = int(st["delays"][k, c])
            out[k] += s[d:d + out.shape[1]]
    return out / x.shape[1]
