"""Workspaces of the folded path: one pair of the two-pass form is the least that blink_image_batch and
blink_image_batch_corrected take, whichever form a call takes; every workspace from there on gives the same images
(several chunks of pairs, the last one short), plain and corrected, as the FP64 oracle within the usual bars.
"""
import numpy as np
import pytest

import oracle
from image_checks import rel_l2

pytestmark = pytest.mark.gpu

FREQ = 150.0e6
DL = 1.0e-3
IMAGE_TOL = {0: 1e-5, 1: 1e-3, 2: 1e-3}


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


def problem(tiles, N, T, C, P):
    B = tiles * (tiles - 1) // 2
    g = np.random.default_rng(N + B)
    uvw = np.zeros((T, B, 3))
    uvw[..., :2] = g.uniform(-N / 2 + 1, N / 2 - 1, (T, B, 2)) / (FREQ * 1.02 / 299792458.0 * (N * DL))
    freq = FREQ * (1.0 + 0.001 * np.arange(C))
    vis = (g.normal(size=(T, C, P, B)) + 1j * g.normal(size=(T, C, P, B))).astype(np.complex64)
    flags = (g.random((T, C, B)) < 0.1).astype(np.uint8)
    return uvw, freq, vis, flags


def run(torch, ctx, prob, N, weighting, prec, nbytes, corrected):
    uvw, freq, vis, flags = (torch.from_numpy(x).to("cuda:0") for x in prob)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda:0")
    call = ctx.blink_image_batch_corrected if corrected else ctx.blink_image_batch
    res = call(vis, flags, uvw, freq, N, DL, weighting, precision=prec, workspace=ws)
    torch.cuda.synchronize()
    return res


@pytest.mark.parametrize("corrected", [False, True])
@pytest.mark.parametrize("weighting", [0, 1])
@pytest.mark.parametrize("N", [512, 2048])
def test_less_than_one_pair_is_refused(torch, ctx, N, weighting, corrected):
    import paper_2505_15204_amd as blink
    prob = problem(25, N, 1, 2, 1)
    size = blink.image_batch_corrected_workspace_size if corrected else blink.image_batch_workspace_size
    one = size(1, 1, 1, 300, N, weighting, 0)
    run(torch, ctx, prob, N, weighting, 0, one, corrected)
    with pytest.raises(blink.BlinkError) as e:
        run(torch, ctx, prob, N, weighting, 0, one - 256, corrected)
    assert e.value.status == 2


def check_against_oracle(res, ref, prec, what):
    assert np.array_equal(res["weight_sum"].cpu().numpy(), ref["weight_sum"]), what
    assert np.array_equal(res["n_out"].cpu().numpy(), ref["n_out"]), what
    got = res["images"].cpu().numpy()
    for i in np.ndindex(ref["images"].shape[:3]):
        assert rel_l2(got[i], ref["images"][i]) <= IMAGE_TOL[prec], (what, i)


def lists(B, P, corrected):
    """Bytes of one pair in the folded form: the tables, 4 + 8 P for each of 2 B + 1024 entries, corrected values."""
    up = lambda x: (x + 255) // 256 * 256
    return 256 + 8192 + up(4 * (2 * B + 1024)) + up(8 * P * (2 * B + 1024)) + (up(8 * P * B) if corrected else 0)


# all pairs at once, three and a half (chunks of three, the last one short), the least: one at a time
@pytest.mark.parametrize("corrected", [False, True])
@pytest.mark.parametrize("prec,weighting", [(0, 0), (0, 1), (1, 0), (2, 1)])
def test_chunks(torch, ctx, prec, weighting, corrected):
    import paper_2505_15204_amd as blink
    T, C, P, N = 2, 5, 2, 512
    prob = problem(181, N, T, C, P)
    B = prob[2].shape[-1]
    ref = oracle.image_batch(prob[2], prob[3], prob[0], prob[1], N, DL, weighting)
    size = blink.image_batch_corrected_workspace_size if corrected else blink.image_batch_workspace_size
    one = size(1, 1, 1, B, N, weighting, prec) + (8 * B + 512 if corrected else 256)      # P = 2, one intermediate
    for nbytes in (size(T, C, P, B, N, weighting, prec), max(one, int(3.5 * lists(B, P, corrected))), one):
        print(f"[gpu-case] chunks prec={prec} w={weighting} corrected={corrected} bytes={nbytes}", flush=True)
        check_against_oracle(run(torch, ctx, prob, N, weighting, prec, nbytes, corrected), ref, prec, nbytes)


# 16290 baselines on a 256^2 grid: the least workspace holds a pair of the two-pass form, not of the lists
@pytest.mark.parametrize("corrected", [False, True])
def test_lists_that_do_not_fit(torch, ctx, corrected):
    import paper_2505_15204_amd as blink
    N, P = 256, 2
    prob = problem(181, N, 1, 1, P)
    B = prob[2].shape[-1]
    ref = oracle.image_batch(prob[2], prob[3], prob[0], prob[1], N, DL, 0)
    fits = lists(B, P, corrected)
    for nbytes, folded in ((fits - 256, False), (fits, True)):
        print(f"[gpu-case] lists corrected={corrected} bytes={nbytes}", flush=True)
        ctx.profile_enable(True)
        res = run(torch, ctx, prob, N, 0, 0, nbytes, corrected)
        rows = ctx.profile_read()["row_fft"][1]
        ctx.profile_enable(False)
        assert (rows == 0) == folded, (nbytes, rows)
        check_against_oracle(res, ref, 0, nbytes)
