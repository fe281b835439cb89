"""blink_image_average over images smaller than a wave's pixels and over batches that the last-level cache holds, on
both sides of the lines between its kernels: against FP64 sums, bit-exact for whole numbers, and the cost of many
small outputs beside that of the same bytes in larger ones (at most twice).
"""
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


# (T, C, P, N, axes): outputs of 2 to 40 inputs, small and large images, few and many of them; 64^2 x 100 outputs
# are 1600 blocks of a wave, 32 x 512^2 x 40 inputs more than 300 MB
@pytest.mark.parametrize("shape", [(1, 3, 2, 8, 4), (3, 50, 2, 8, 4), (15, 70, 1, 8, 1), (20, 70, 1, 8, 1), (20, 100, 1, 64, 1),
                                   (33, 100, 1, 64, 1), (16, 9, 2, 16, 3), (8, 33, 2, 32, 1), (1, 40, 2, 256, 4),
                                   (15, 20, 1, 512, 1), (3, 100, 1, 512, 1), (40, 8, 1, 512, 1)])
def test_sums(torch, ctx, shape):
    T, C, P, N, axes = shape
    print(f"[gpu-case] average {shape}", flush=True)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(N + T)
    x = torch.randint(-1000, 1000, (T, C, P, N, N), generator=g, device="cuda:0").float()
    dims = [d for d in range(3) if axes >> d & 1]
    n = 1
    for d in dims:
        n *= x.shape[d]
    want = (x.double().sum(dim=dims, keepdim=True) * (1.0 / n)).float()
    got = ctx.blink_image_average(x, axes)
    assert torch.equal(got.view(want.shape), want)


def average_us(torch, ctx, T, C, P, N, axes):
    x = torch.zeros((T, C, P, N, N), device="cuda:0")
    out = torch.empty((1 if axes & 1 else T, 1 if axes & 2 else C, 1 if axes & 4 else P, N, N), device="cuda:0")
    best = 1.0e9
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            ctx.blink_image_average(x, axes, out=out)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 5 * 1e3)
    return best


def test_many_small_outputs_cost_their_bytes(torch, ctx):
    print("[gpu-case] average timing", flush=True)
    small, large = average_us(torch, ctx, 1, 80000, 2, 8, 4), average_us(torch, ctx, 1, 313, 2, 128, 4)
    assert small <= 2.0 * large, (small, large)
