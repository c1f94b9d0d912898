"""GPU parity of the route of adloco_grad_stats that takes the per-sample norms from the 256 x 128
tiles of the per-sample gradients on their way into the gradient sum (aligned bf16 and fp16 blocks,
gradient sum formed by the library), against the CPU oracle and against the Gram route: short and
long sequences (a kernel each), ragged ones, tiles on the edge of a layer, entries split along the
samples (few tiles) and whole entries (more than 32 tiles on an XCD), accumulation over
micro-batches, bitwise repeatability."""
import numpy as np
import pytest

import adloco_synth as synth
from oracle import adloco_oracle as orc

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-3


@pytest.fixture(scope="module")
def ctx():
    import paper_2508_18182_amd as A
    c = A.Context(0)
    yield c
    c.close()


def _check(ctx, layers, flags=0, acc=None, grad_sums=None):
    from gpu_util import run_grad_stats, rel_err
    got = run_grad_stats(ctx, layers, flags=flags, acc=acc, grad_sums=grad_sums)
    return got


def _compare(got, want):
    from gpu_util import rel_err
    assert rel_err(got["per_layer"], want["n_layer_sample"]) < TOL_BF16
    assert rel_err(got["per_sample"], want["n_sample"]) < TOL_BF16
    assert rel_err(got["S1"], want["S1"]) < TOL_BF16
    for l, (g, w) in enumerate(zip(got["G"], want["G"])):
        scale = float(np.sqrt(np.mean(w * w))) + 1e-300
        assert float(np.max(np.abs(g.astype(np.float64) - w))) / scale < 1e-4, l


@pytest.mark.parametrize("B,T,shapes", [
    (5, 32, [(72, 264)]),                  # one chunk per sample, both edges ragged
    (1, 64, [(256, 128)]),                 # exactly one tile, one sample
    (7, 96, [(320, 520), (8, 8)]),         # three chunks per sample, a tiny block
    (40, 32, [(128, 256)]),                # more samples than pieces: uneven sample runs
    (3, 160, [(136, 72), (264, 8), (16, 392)]),
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_tile_route_small(ctx, dtype, B, T, shapes):
    layers = synth.custom_grad_stats_inputs(6000 + B + T, shapes, B, T, dtype, std_delta=0.2, rho=0.4)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in layers], two_pass=False)
    ctx.set_tuning("stats_variant", 1)
    got = _check(ctx, layers)
    assert got["n_samples"] == B
    _compare(got, want)
    # the Gram route agrees to rounding, and the route itself repeats bit for bit
    again = _check(ctx, layers)
    assert np.array_equal(again["per_layer"], got["per_layer"])
    for g0, g1 in zip(got["G"], again["G"]):
        assert np.array_equal(g0, g1)
    ctx.set_tuning("stats_variant", 0)
    gram = _check(ctx, layers)
    ctx.set_tuning("stats_variant", 1)
    assert np.max(np.abs(gram["per_layer"] - got["per_layer"]) / got["per_layer"]) < 1e-4


def test_tile_route_whole_and_split_entries(ctx):
    # 288 tiles: every XCD holds 36, one full round of whole entries and four entries split along
    # the three samples; the second layer straddles two XCDs
    B, T = 3, 32
    shapes = [(2048, 2048), (2048, 2048), (2048, 264)]
    layers = synth.custom_grad_stats_inputs(6100, shapes, B, T, "bf16", std_delta=0.05, rho=0.3)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in layers], two_pass=False)
    ctx.set_tuning("stats_variant", 1)
    got = _check(ctx, layers)
    _compare(got, want)


def test_tile_route_extreme_aspect_ratios(ctx):
    # one tile row of 32 tile columns, one tile column of 16 tile rows, and a 5 x 9 grid: the blocks in
    # which the tiles of a layer are ordered are cut off by the layer's edge in every way
    B, T = 2, 32
    shapes = [(4096, 8), (8, 4096), (1160, 1288)]
    layers = synth.custom_grad_stats_inputs(6300, shapes, B, T, "bf16", std_delta=0.05, rho=0.3)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in layers], two_pass=False)
    ctx.set_tuning("stats_variant", 1)
    got = _check(ctx, layers)
    _compare(got, want)
    ctx.set_tuning("stats_variant", 0)       # the gradient-sum GEMM orders its 256 x 256 tiles the same way
    _compare(_check(ctx, layers), want)
    ctx.set_tuning("stats_variant", 1)


def test_tile_route_accumulates_over_micro_batches(ctx):
    # switch mode: S1, n and the gradient sums continue over three micro-batches; whole and split
    # entries both add to what is there
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc
    B, T = 2, 64
    shapes = [(1024, 2048), (520, 136)]
    mbs = [synth.custom_grad_stats_inputs(6200 + 10 * k, shapes, B, T, "bf16", std_delta=0.1, rho=0.3)
           for k in range(3)]
    want = orc.grad_stats(orc.concat_micro_batches([[(l["a"], l["delta"]) for l in mb] for mb in mbs]),
                          two_pass=False)
    ctx.set_tuning("stats_variant", 1)
    gs = [torch.full((do, di), float("nan"), device=DEV) for di, do in shapes]
    acc = new_acc()
    per_layer = []
    for k, mb in enumerate(mbs):
        got = _check(ctx, mb, flags=A.ADLOCO_ACCUMULATE if k else 0, acc=acc, grad_sums=gs)
        per_layer.append(got["per_layer"])
    from gpu_util import rel_err
    assert got["n_samples"] == 3 * B
    assert rel_err(np.concatenate(per_layer, axis=1), want["n_layer_sample"]) < TOL_BF16
    assert rel_err(got["S1"], want["S1"]) < TOL_BF16
    for l, w in enumerate(want["G"]):
        g = gs[l].cpu().numpy().astype(np.float64)
        assert float(np.max(np.abs(g - w))) / (float(np.sqrt(np.mean(w * w))) + 1e-300) < 1e-4


@pytest.mark.parametrize("B,T,shapes", [
    (3, 1, [(8, 8)]),                      # one row per sample, the rest of its chunk zeros
    (9, 33, [(136, 264)]),                 # two chunks (even), the second of one row; more chunks than stages
    (2, 95, [(72, 520), (256, 256)]),      # three chunks (odd), the last one row short
    (1, 250, [(264, 8)]),                  # one sample of eight chunks: the load pipeline never wraps
    (300, 7, [(128, 256)]),                # long runs of one-chunk samples
    (2, 45, [(1024, 2048)]),               # short for the widths: Gram contraction and gradient sum of ragged rows
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_tile_route_ragged_sequences(ctx, dtype, B, T, shapes):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of
    layers = synth.custom_grad_stats_inputs(6400 + B + T, shapes, B, T, dtype, std_delta=0.2, rho=0.4)
    entries = [(l["a"], l["delta"]) for l in layers]
    want = orc.grad_stats(entries, two_pass=False)
    ctx.set_tuning("stats_variant", 1)
    got = _check(ctx, layers)
    _compare(got, want)
    again = _check(ctx, layers)
    assert np.array_equal(again["per_layer"], got["per_layer"])
    # the inner products go through the same tiles, against the gradient sums just formed
    c, sq = torch.full((B,), float("nan"), device=DEV), torch.full((B,), float("nan"), device=DEV)
    A.adloco_inner_products(ctx, got["layers"], B, T, code_of(dtype), c, sq,
                            torch.zeros(4, dtype=torch.float64, device=DEV))
    c_want = orc.inner_products(entries, G=want["G"])
    assert np.max(np.abs(c.cpu().numpy() - c_want) / np.sqrt(want["n_sample"] * want["S2"])) < TOL_BF16
    assert np.max(np.abs(sq.cpu().numpy() - want["n_sample"]) / want["n_sample"]) < TOL_BF16
    # and without the explicit norms
    c2 = torch.full((B,), float("nan"), device=DEV)
    A.adloco_inner_products(ctx, got["layers"], B, T, code_of(dtype), c2, None,
                            torch.zeros(4, dtype=torch.float64, device=DEV))
    assert torch.equal(c, c2)


@pytest.mark.parametrize("B,T", [(3, 32), (2, 96), (5, 256),        # the tile kernel for short sequences: one chunk, odd, even
                                 (2, 288), (3, 320),                # statistics by the other one, odd and even
                                 (2, 544), (2, 576),                # inner products too
                                 (1, 64), (1, 288)])                # one piece: tiles stored where they belong
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_short_and_long_sequences(ctx, dtype, B, T):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of
    layers = synth.custom_grad_stats_inputs(6450 + B + T, [(136, 264), (256, 128), (8, 520)], B, T, dtype, std_delta=0.2, rho=0.4)
    entries = [(l["a"], l["delta"]) for l in layers]
    want = orc.grad_stats(entries, two_pass=False)
    ctx.set_tuning("stats_variant", 1)
    got = _check(ctx, layers)
    _compare(got, want)
    for sq in (torch.full((B,), float("nan"), device=DEV), None):
        c = torch.full((B,), float("nan"), device=DEV)
        A.adloco_inner_products(ctx, got["layers"], B, T, code_of(dtype), c, sq, torch.zeros(4, dtype=torch.float64, device=DEV))
        c_want = orc.inner_products(entries, G=want["G"])
        assert np.max(np.abs(c.cpu().numpy() - c_want) / np.sqrt(want["n_sample"] * want["S2"])) < TOL_BF16
        if sq is not None:
            assert np.max(np.abs(sq.cpu().numpy() - want["n_sample"]) / want["n_sample"]) < TOL_BF16
    # added to what is there: twice the sums
    gs = [l["grad_sum"] for l in got["layers"]]
    _check(ctx, layers, flags=A.ADLOCO_ACCUMULATE, acc=got["acc"], grad_sums=gs)
    for g, w in zip(gs, want["G"]):
        assert np.max(np.abs(g.cpu().numpy() - 2 * w)) < 2e-4 * float(np.sqrt(np.mean(w * w)))


@pytest.mark.parametrize("B,T,shapes", [
    (1, 1, [(8, 8)]),                      # one token row
    (5, 77, [(136, 264)]),                 # 385 rows: one over twelve chunks
    (3, 21, [(128, 256), (520, 72)]),      # 63 rows: a short second chunk, fewer chunks than pieces
    (2, 512, [(256, 768), (1032, 264)]),   # whole chunks, tiles on the edge
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_gradient_sum_alone(ctx, dtype, B, T, shapes):
    # the gradient-only call: short last chunk, pieces of split tiles (more than chunks), added to a sum
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of, to_dev
    host = synth.custom_grad_stats_inputs(6500 + B + T, shapes, B, T, dtype, std_delta=0.2, rho=0.4)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in host], two_pass=False)["G"]
    layers = [dict(a=to_dev(l["a"]), delta=to_dev(l["delta"]),
                   grad_sum=torch.full((l["d_out"], l["d_in"]), float("nan"), device=DEV)) for l in host]
    for k, flags in enumerate((0, A.ADLOCO_ACCUMULATE)):
        A.adloco_grad_stats(ctx, layers, B, T, code_of(dtype), None, None, None, A.ADLOCO_SUM_ONLY | flags)
        for l, w in zip(layers, want):
            err = np.max(np.abs(l["grad_sum"].cpu().numpy().astype(np.float64) - (k + 1) * w))
            assert err < (k + 1) * 1e-4 * float(np.sqrt(np.mean(w * w)))


@pytest.mark.parametrize("B,T,shapes", [
    (3, 513, [(64, 128), (128, 64)]),      # long for the widths: tiles of the per-sample gradients, ragged
    (2, 1024, [(136, 72), (8, 264)]),      # whole chunks, widths that are no multiple of 64
    (40, 160, [(64, 64)]),                 # several samples per entry
    (2, 96, [(512, 1024)]),                # short: the Gram contraction
])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_norms_of_supplied_gradients(ctx, dtype, B, T, shapes):
    # both routes against the oracle; the supplied gradient sums are read by nobody and stay as they are
    import torch
    from gpu_util import DEV, rel_err, run_grad_stats
    layers = synth.custom_grad_stats_inputs(6600 + B + T, shapes, B, T, dtype, std_delta=0.2, rho=0.4)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in layers], two_pass=False)
    gs = [torch.full((l["d_out"], l["d_in"]), 7.0, device=DEV) for l in layers]
    for variant in (1, 0):
        ctx.set_tuning("stats_variant", variant)
        got = run_grad_stats(ctx, layers, grad_sums=gs, provided=True)
        assert rel_err(got["per_layer"], want["n_layer_sample"]) < (1e-4 if dtype == "f32" else TOL_BF16)
        assert rel_err(got["S1"], want["S1"]) < (1e-4 if dtype == "f32" else TOL_BF16)
        assert all(bool((g == 7.0).all()) for g in gs)
    ctx.set_tuning("stats_variant", 1)
