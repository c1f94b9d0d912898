"""Infinite inputs (an overflow in fp16) on the kernels that form per-sample gradients tile by tile, at widths where tiles
reach past the layer: the sample's norm is +Inf and not NaN, and every other sample's is what it is without it.  A NaN
would make the norm test refuse the batch, where an infinite norm asks for the largest one."""
import math

import numpy as np
import pytest

import adloco_synth as synth

pytestmark = pytest.mark.gpu

EDGES, WHOLE, ODD = (200, 328), (128, 256), (77, 101)     # past the edge on both sides; nowhere; also unaligned rows


@pytest.fixture(scope="module")
def ctx():
    import paper_2508_18182_amd as A
    c = A.Context(0)
    yield c
    c.close()


def _layers(dtype, shape, B, T, provided=False):
    import torch
    from gpu_util import DEV, to_dev
    host = synth.custom_grad_stats_inputs(8100 + B + T, [shape, WHOLE], B, T, dtype, std_delta=0.2, rho=0.4)
    return [dict(a=to_dev(l["a"]), delta=to_dev(l["delta"]), provided=provided,
                 grad_sum=torch.full((l["d_out"], l["d_in"]), 0.5, device=DEV)) for l in host]


def _stats(ctx, layers, dtype, B, T):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of, new_acc, read_acc
    ps, acc = torch.zeros(B, device=DEV), new_acc()
    ctx.set_tuning("profile", 1)
    A.adloco_grad_stats(ctx, layers, B, T, code_of(dtype), ps, None, acc)
    torch.cuda.synchronize()
    tiles = ctx.profile_read("tile_stats")[1]
    ctx.set_tuning("profile", 0)
    assert tiles == 1                   # the route that this file is about
    return ps.cpu().numpy(), acc, read_acc(acc)[0]


STATS = [("f16", EDGES, 3, 64, False), ("bf16", EDGES, 3, 200, False), ("f32", EDGES, 3, 50, False),
         ("f16", WHOLE, 3, 96, False), ("f16", EDGES, 2, 288, False), ("f16", EDGES, 64, 1024, True), ("f32", ODD, 40, 512, True)]


@pytest.mark.parametrize("where", ["delta", "a"])
@pytest.mark.parametrize("dtype,shape,B,T,provided", STATS)
def test_norms(ctx, dtype, shape, B, T, provided, where):
    import paper_2508_18182_amd as A
    layers = _layers(dtype, shape, B, T, provided)
    want, _, _ = _stats(ctx, layers, dtype, B, T)
    assert np.isfinite(want).all()
    layers[0][where][1, T - 1, 5] = float("inf")
    got, acc, S1 = _stats(ctx, layers, dtype, B, T)
    assert got[1] == np.inf and S1 == np.inf
    rest = np.arange(B) != 1
    assert np.array_equal(got[rest], want[rest])
    for l in layers:
        l["grad_sum"].fill_(0.5)
    t = A.adloco_norm_test(ctx, layers, acc, 0.3, B, 32, 2, 256)
    assert t["S1"] == math.inf and t["b_req"] == 256


@pytest.mark.parametrize("T", [50, 64, 544])       # ragged, short and long sequences
@pytest.mark.parametrize("shape", [EDGES, WHOLE, ODD])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_inner_products(ctx, dtype, shape, T):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of
    B = 3
    layers = _layers(dtype, shape, B, T)

    def run():
        c, sq = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
        A.adloco_inner_products(ctx, layers, B, T, code_of(dtype), c, sq, torch.zeros(4, dtype=torch.float64, device=DEV))
        return c.cpu().numpy(), sq.cpu().numpy()

    c0, sq0 = run()
    G = layers[0]["grad_sum"]
    G[-1, -1] = float("inf")            # c_i takes the sign of g_i there, the norms do not see it
    g = torch.einsum("bt,bt->b", layers[0]["delta"][..., -1].double(), layers[0]["a"][..., -1].double()).cpu().numpy()
    c, sq = run()
    assert np.array_equal(c, np.sign(g) * np.inf) and np.array_equal(sq, sq0)
    G[-1, -1] = 0.5
    for where in ("delta", "a"):
        old = layers[0][where][1, 0, 5].clone()
        layers[0][where][1, 0, 5] = float("inf")
        c, sq = run()
        layers[0][where][1, 0, 5] = old
        assert sq[1] == np.inf and not np.isfinite(c[1])
        assert np.array_equal(sq[[0, 2]], sq0[[0, 2]]) and np.array_equal(c[[0, 2]], c0[[0, 2]])
