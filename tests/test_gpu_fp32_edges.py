"""fp32 tiles where cutting their values into bf16 parts does not do: values whose parts overflow, and sums of few products.
Oracle: fp64.  Tolerance: T multiply-adds rounded one after the other, each within 2^-24 of the sum so far, which is at
most S, the sum of the magnitudes of an entry's products (and half as much again for the order of four in an MFMA)."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(64, 64), (130, 65), (3, 257)]          # whole tiles, edges, a layer narrower than a lane's columns


@pytest.fixture(scope="module")
def ctx():
    import paper_2508_18182_amd as A
    c = A.Context(0)
    yield c
    c.close()


def _rows(B, T, d_in, d_out, scale_a, scale_d, seed=0):
    import torch
    g = torch.Generator().manual_seed(B * 1000 + T + d_in + seed)
    a, d = (torch.randn(B, T, w, generator=g) * s for w, s in ((d_in, scale_a), (d_out, scale_d)))
    # rows of an odd number of floats, one float past the start of the allocation
    return [torch.cat([x.new_full((B, T, 1), float("nan")), x, x.new_full((B, T, 1 + x.shape[2] % 2), float("nan"))], 2)
            .cuda()[:, :, 1:1 + x.shape[2]] for x in (a, d)]


def _check(ctx, a, d, B, T):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc
    d_in, d_out = a.shape[2], d.shape[2]
    g = torch.stack([d[i].double().t().contiguous() @ a[i].double() for i in range(B)])
    S = torch.stack([d[i].double().abs().t().contiguous() @ a[i].double().abs() for i in range(B)])
    bound = 1.5 * T * 2.0 ** -24 * S if T > 1 else 2.0 ** -24 * S
    G, G_bound = g.sum(0), bound.sum(0) + (B - 1) * 2.0 ** -24 * S.sum(0)
    sq, sq_bound = g.pow(2).sum((1, 2)), (2 * g.abs() * bound + bound.pow(2)).sum((1, 2))
    G32 = G.float()
    ip, ip_bound = (g * G32.double()).sum((1, 2)), (bound * G32.double().abs()).sum((1, 2))

    def same(got, want, tol):
        assert bool(((got.double() - want).abs() <= tol + (2.0 ** -24 * want.abs() if got.dim() == 1 else 0.0)).all())

    for form in (1, 2, 5, 6):
        ctx.set_tuning("plain_tiles", form)
        ctx.set_tuning("profile", 1)
        try:
            grad, ps = torch.full((d_out, d_in), float("nan"), device=DEV), torch.zeros(B, device=DEV)
            A.adloco_grad_stats(ctx, [dict(a=a, delta=d, grad_sum=grad)], B, T, A.ADLOCO_F32, ps, None, new_acc())
            assert ctx.profile_read("tile_stats")[1] == 1
            same(grad, G, G_bound)
            same(ps, sq, sq_bound)
            dots, ps = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
            A.adloco_inner_products(ctx, [dict(a=a, delta=d, grad_sum=G32)], B, T, A.ADLOCO_F32, dots, ps,
                                    torch.zeros(4, dtype=torch.float64, device=DEV))
            same(ps, sq, sq_bound)
            same(dots, ip, ip_bound)
        finally:
            ctx.set_tuning("plain_tiles", 0)
            ctx.set_tuning("profile", 0)


@pytest.mark.parametrize("T", [6, 32, 75])
@pytest.mark.parametrize("d_in,d_out", SHAPES)
def test_large_values_throughout(ctx, T, d_in, d_out):
    # parts of a overflow (from 2^103), the products and the norms do not
    a, d = _rows(3, T, d_in, d_out, 2.0 ** 108, 2.0 ** -60)
    _check(ctx, a, d, 3, T)


@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("d_in,d_out", SHAPES)
def test_few_rows(ctx, T, d_in, d_out):
    # a single product is rounded to nearest; at full size and where the products left out are the largest
    a, d = _rows(2, T, d_in, d_out, 1.0, 1.0)
    _check(ctx, a, d, 2, T)
    a[:, :, ::3] = d[:, :, ::2] = 1 + 2.0 ** -8 - 2.0 ** -17
    _check(ctx, a, d, 2, T)


def test_large_values_take_no_more_than_a_few_times_as_long(ctx):
    # (2.7 times here; 58 when each entry was summed by one thread)
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc
    B, T, d_in, d_out = 8, 256, 768, 3072
    took = []
    for scale in (1.0, 2.0 ** 108):
        a, d = (torch.randn(B, T, w, device=DEV) * s for w, s in ((d_in, scale), (d_out, 2.0 ** -60)))
        layers = [dict(a=a, delta=d, grad_sum=torch.zeros(d_out, d_in, device=DEV))]
        ps, acc = torch.zeros(B, device=DEV), new_acc()
        A.adloco_grad_stats(ctx, layers, B, T, A.ADLOCO_F32, ps, None, acc)
        ctx.set_tuning("profile", 1)
        for _ in range(5):
            A.adloco_grad_stats(ctx, layers, B, T, A.ADLOCO_F32, ps, None, acc)
        ms, n = ctx.profile_read("tile_stats")
        ctx.set_tuning("profile", 0)
        assert n == 5 and bool(torch.isfinite(ps).all())
        took.append(ms)
    assert took[1] < 12 * took[0]
