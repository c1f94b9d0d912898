"""fp32 tiles formed from three bf16 parts of every value, against fp64: tile edges, chunk ends, rows that are aligned to
nothing but their elements, columns from 2^-70 to 2^40, denormals, values whose parts overflow, infinities and NaN.
Tolerance, S the sum of the magnitudes of an entry's products: six sums of 32 products a chunk are rounded (or T
multiply-adds, where a part overflows), each within 2^-23 S with the sum so far; the products left out are below 2^-24 S."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2508_18182_amd as A
    c = A.Context(0)
    yield c
    c.close()


def _inputs(kind, B, T, d_in, d_out):
    import torch
    g = torch.Generator().manual_seed(B * 1000 + T + d_in)
    a, d = torch.randn(B, T, d_in, generator=g), torch.randn(B, T, d_out, generator=g)
    if kind == "wide":
        a *= torch.pow(2.0, torch.randint(-70, 40, (d_in,), generator=g).float())
        d *= torch.pow(2.0, torch.randint(-30, 20, (d_out,), generator=g).float())
    if kind == "denormal":
        d *= 2.0 ** -140
        a *= 2.0 ** 20
    if kind == "overflow":
        a[B // 2, T // 2, d_in // 2] = 2.0 ** 105
        d[0, T // 3, d_out // 2] = -2.0 ** 120
        d *= 2.0 ** -4
    if kind == "infinite":
        a[B // 2, T // 2, d_in // 2] = float("inf")
        d[0, T - 1, d_out - 1] = float("-inf")
        a[B - 1, 0, 0] = float("nan")
    # rows of an odd number of floats, one float past the start of the allocation
    return [torch.cat([x.new_full((B, T, 1), float("nan")), x, x.new_full((B, T, 1 + x.shape[2] % 2), float("nan"))], 2)
            .cuda()[:, :, 1:1 + x.shape[2]] for x in (a, d)]


@pytest.mark.parametrize("kind", ["plain", "wide", "denormal", "overflow", "infinite"])
@pytest.mark.parametrize("B,T,d_in,d_out", [(1, 1, 3, 1), (3, 31, 63, 130), (2, 33, 129, 65), (9, 96, 257, 68), (2, 130, 64, 256)])
def test_parts(ctx, kind, B, T, d_in, d_out):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc
    a, d = _inputs(kind, B, T, d_in, d_out)
    g = torch.stack([d[i].double().t().contiguous() @ a[i].double() for i in range(B)])
    S = torch.stack([d[i].double().abs().t().contiguous() @ a[i].double().abs() for i in range(B)])
    bound = (6 * ((T + 31) // 32) + T * (kind == "overflow") + 2) * 2.0 ** -23 * S + 2.0 ** -148
    G, G_bound = g.sum(0), bound.sum(0) + B * 2.0 ** -23 * S.sum(0)
    sq, sq_bound = g.pow(2).sum((1, 2)), (2 * g.abs() * bound + bound.pow(2)).sum((1, 2))
    G32 = G.float()
    ip, ip_bound = (g * G32.double()).sum((1, 2)), (bound * G32.double().abs()).sum((1, 2))

    def same(got, want, tol):
        got = got.double()
        want32 = want.float()
        odd = ~torch.isfinite(want32)
        assert torch.equal(torch.isnan(got), torch.isnan(want32))
        assert torch.equal(got[odd & ~torch.isnan(got)], want32[odd & ~torch.isnan(want32)].double())
        assert bool(((got - want).abs()[~odd] <= (tol + 2.0 ** -23 * want.abs() + 2.0 ** -148)[~odd]).all())

    for form in (1, 2, 5, 6):
        ctx.set_tuning("plain_tiles", form)
        try:
            for _ in range(2):
                grad, ps = torch.full((d_out, d_in), float("nan"), device=DEV), torch.zeros(B, device=DEV)
                A.adloco_grad_stats(ctx, [dict(a=a, delta=d, grad_sum=grad)], B, T, A.ADLOCO_F32, ps, None, new_acc())
                same(grad, G, G_bound)
                same(ps, sq, sq_bound)
            dots, ps = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
            A.adloco_inner_products(ctx, [dict(a=a, delta=d, grad_sum=G32)], B, T, A.ADLOCO_F32, dots, ps,
                                    torch.zeros(4, dtype=torch.float64, device=DEV))
            same(ps, sq, sq_bound)
            if kind != "infinite":                # (0 * inf of a zero gradient entry: NaN here and there)
                same(dots, ip, ip_bound)
        finally:
            ctx.set_tuning("plain_tiles", 0)
