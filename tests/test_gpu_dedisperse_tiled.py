"""The tiled de-dispersion kernel (images of 128^2 and above, at most 60 time steps of a channel per
workgroup) against the oracle, bit for bit: trial counts and output steps that do not fill its
units, several workgroups per pixel block, channel counts around the stages of four, delays without
any order over the trials, and step ranges on both sides of the stage's 60.
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


@pytest.mark.parametrize("T,C,N,n_dm,t_out", [
    (9, 1, 128, 1, 9),        # one trial, no delay, one channel
    (14, 3, 128, 3, 1),       # one output step
    (20, 4, 128, 5, 13),      # a full tile
    (20, 5, 128, 2, 14),      # two tiles of seven
    (40, 7, 128, 16, 27),     # three tiles, two workgroups per pixel block
    (60, 6, 128, 4, 31),      # step range 60
    (61, 6, 128, 4, 31),      # 61: the untiled kernel
    (30, 9, 256, 33, 5),      # 17 trial pairs
])
def test_tiled_matches_oracle(torch, ctx, T, C, N, n_dm, t_out):
    g = np.random.default_rng(T * 100 + C)
    delays = g.integers(0, T - t_out + 1, (n_dm, C)).astype(np.int32)
    delays[0, 0], delays[-1, 0] = 0, T - t_out
    imgs = g.normal(size=(T, C, N, N)).astype(np.float32)
    print(f"[gpu-case] tiled de-dispersion T={T} C={C} N={N} n_dm={n_dm} t_out={t_out}", flush=True)
    out = ctx.blink_dedisperse(torch.from_numpy(imgs).to("cuda:0"), delays, t_out).cpu().numpy()
    assert np.array_equal(out, oracle.dedisperse(imgs, delays, t_out).astype(np.float32))
