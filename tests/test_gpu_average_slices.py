"""The sliced image averages against numpy: input counts around the 16 that select the slices and the
8 loads in flight, axes that merge into one run and axes that do not, and images on both sides of
the size where the wider form is taken. FP64 sums rounded once: half a unit in the last place of the
float result, plus the few FP64 roundings that the order of the sum can move (relative 1e-14)."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("T,C,P,N,axes", [
    (1, 15, 1, 8, 2), (1, 16, 1, 8, 2), (1, 17, 1, 16, 2), (3, 23, 2, 64, 2), (3, 23, 2, 64, 5), (3, 23, 2, 64, 7),
    (2, 131, 2, 32, 6), (17, 3, 2, 128, 1), (2, 9, 2, 1024, 3), (1, 20, 2, 1024, 6),
])
def test_average_matches_numpy(torch, ctx, T, C, P, N, axes):
    g = np.random.default_rng(T * 1000 + C)
    x = (g.normal(size=(T, C, P, N, N)) + 3.0).astype(np.float32)
    want = x.astype(np.float64).mean(axis=tuple(k for k in range(3) if axes >> k & 1), keepdims=True)
    print(f"[gpu-case] average T={T} C={C} P={P} N={N} axes={axes}", flush=True)
    got = ctx.blink_image_average(torch.from_numpy(x).to("cuda:0"), axes).cpu().numpy().astype(np.float64)
    scale = np.abs(x).astype(np.float64).max()
    assert (np.abs(got - want) <= 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-14 * scale).all()
