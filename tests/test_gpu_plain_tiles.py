"""GPU parity of the plain tile kernel, which forms the per-sample gradients of fp32 blocks (statistics, gradient sum,
inner products) and of unaligned 16-bit blocks (inner products), at the edges of its tiles, chunks and entries, against
the CPU oracle.  Tolerances: fp32 sums of exact products, so the bars of the fp32 norms (1e-4) hold for every input
type; gradient-sum entries within 1e-4 of the layer's rms."""
import numpy as np
import pytest

import adloco_synth as synth
from oracle import adloco_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2508_18182_amd as A
    c = A.Context(0)
    yield c
    c.close()


CASES = [
    (1, 1, [(1, 1)]),                              # one product
    (3, 17, [(63, 65), (64, 64)]),                 # 64-wide tiles: one short, exact, one over; a ragged chunk
    (5, 31, [(129, 7)]),                           # scalar staging, several tile columns
    (70, 3, [(64, 128)]),                          # more samples than pieces of a split tile
    (2, 33, [(1032, 2056), (1030, 2049)]),         # 128-wide tiles, aligned and unaligned rows, whole entries
]


@pytest.mark.parametrize("B,T,shapes", CASES)
def test_statistics_fp32(ctx, B, T, shapes):
    import paper_2508_18182_amd as A
    from gpu_util import rel_err, run_grad_stats
    layers = synth.custom_grad_stats_inputs(7000 + B + T, shapes, B, T, "f32", std_delta=0.2, rho=0.4)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in layers], two_pass=False)
    got = run_grad_stats(ctx, layers)
    assert rel_err(got["per_layer"], want["n_layer_sample"]) < 1e-4
    assert rel_err(got["S1"], want["S1"]) < 1e-4
    # added to what is there, and without the statistics
    gs = [l["grad_sum"] for l in got["layers"]]
    again = run_grad_stats(ctx, layers, flags=A.ADLOCO_ACCUMULATE, acc=got["acc"], grad_sums=gs)
    assert np.array_equal(again["per_layer"], got["per_layer"])
    A.adloco_grad_stats(ctx, got["layers"], B, T, A.ADLOCO_F32, None, None, None, A.ADLOCO_ACCUMULATE | A.ADLOCO_SUM_ONLY)
    for g1, g2, g3, w in zip(got["G"], again["G"], gs, want["G"]):
        scale = float(np.sqrt(np.mean(w * w)))
        assert np.max(np.abs(g1 - w)) < 1e-4 * scale
        assert np.max(np.abs(g2 - 2 * w)) < 2e-4 * scale
        assert np.max(np.abs(g3.cpu().numpy() - 3 * w)) < 3e-4 * scale


@pytest.mark.parametrize("B,T,shapes", CASES)
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_inner_products(ctx, dtype, B, T, shapes):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of, to_dev
    host = synth.custom_grad_stats_inputs(7100 + B + T, shapes, B, T, dtype, std_delta=0.2, rho=0.4)
    entries = [(l["a"], l["delta"]) for l in host]
    want = orc.grad_stats(entries, two_pass=False)
    layers = [dict(a=to_dev(l["a"]), delta=to_dev(l["delta"]), grad_sum=torch.from_numpy(g.astype(np.float32)).to(DEV))
              for l, g in zip(host, want["G"])]
    c, sq = torch.full((B,), float("nan"), device=DEV), torch.full((B,), float("nan"), device=DEV)
    A.adloco_inner_products(ctx, layers, B, T, code_of(dtype), c, sq, torch.zeros(4, dtype=torch.float64, device=DEV))
    c_want = orc.inner_products(entries, G=want["G"])
    scale = np.sqrt(want["n_sample"] * want["S2"])
    assert np.max(np.abs(c.cpu().numpy() - c_want) / scale) < 1e-4
    assert np.max(np.abs(sq.cpu().numpy() - want["n_sample"]) / want["n_sample"]) < 1e-4


def test_provided_blocks_are_left_alone(ctx):
    # one block's gradient sum supplied: the gradient-only call forms the other one and does not touch it
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, to_dev
    B, T = 3, 20
    host = synth.custom_grad_stats_inputs(7200, [(40, 72), (72, 40)], B, T, "f32", std_delta=0.2, rho=0.4)
    want = orc.grad_stats([(l["a"], l["delta"]) for l in host], two_pass=False)
    layers = [dict(a=to_dev(l["a"]), delta=to_dev(l["delta"]), provided=i == 0,
                   grad_sum=torch.full((l["d_out"], l["d_in"]), 7.0, device=DEV)) for i, l in enumerate(host)]
    A.adloco_grad_stats(ctx, layers, B, T, A.ADLOCO_F32, None, None, None, A.ADLOCO_SUM_ONLY)
    assert bool((layers[0]["grad_sum"] == 7.0).all())
    assert np.max(np.abs(layers[1]["grad_sum"].cpu().numpy() - want["G"][1])) < 1e-4 * np.sqrt(np.mean(want["G"][1] ** 2))


@pytest.mark.parametrize("form", [1, 2, 5, 6])     # 64- or 128-wide tiles, split along the samples or whole
def test_forms_of_the_statistics(ctx, form):
    # the same sums from every form that the time model chooses from, at a batch with fewer and with more samples than pieces
    from gpu_util import rel_err, run_grad_stats
    for B, T, shapes in ((5, 40, [(200, 136), (130, 70)]), (150, 3, [(64, 128)])):
        layers = synth.custom_grad_stats_inputs(7300 + B, shapes, B, T, "f32", std_delta=0.2, rho=0.4)
        want = orc.grad_stats([(l["a"], l["delta"]) for l in layers], two_pass=False)
        ctx.set_tuning("plain_tiles", form)
        got = run_grad_stats(ctx, layers)
        ctx.set_tuning("plain_tiles", 0)
        assert rel_err(got["per_layer"], want["n_layer_sample"]) < 1e-4
        for g, w in zip(got["G"], want["G"]):
            assert np.max(np.abs(g - w)) < 1e-4 * float(np.sqrt(np.mean(w * w)))


@pytest.mark.parametrize("B,T,shapes", [
    (1, 3, [(5, 7)]), (7, 33, [(63, 65), (130, 70)]),        # 64-wide tiles; odd row counts, unaligned widths
    (3, 111, [(1032, 2056), (1030, 2049)]),                  # 128-wide tiles
])
def test_gradient_sum_is_the_vector_kernels_bit_for_bit(ctx, B, T, shapes):
    # the matrix instruction adds the token rows in order, as fused multiply-adds, as the vector unit's kernel does: a
    # training step divides by sqrt(v) right after, where a last bit matters.  Denormal inputs and products included
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, to_dev
    host = synth.custom_grad_stats_inputs(7400 + B, shapes, B, T, "f32", std_delta=0.2, rho=0.4)
    rng = np.random.default_rng(7)
    out = []
    layers = []
    for l in host:
        a, delta = l["a"].copy(), l["delta"].copy()
        for x in (a, delta):
            x[rng.random(x.shape) < 0.05] *= 1e-38            # denormal, and products that are
            x[rng.random(x.shape) < 0.05] *= 1e-20
        layers.append(dict(a=to_dev(a), delta=to_dev(delta)))
    for variant in (1, 0):
        ctx.set_tuning("stats_variant", variant)
        G = [torch.full((l["d_out"], l["d_in"]), 0.25, device=DEV) for l in host]
        for flags in (0, A.ADLOCO_ACCUMULATE):
            A.adloco_grad_stats(ctx, [dict(l, grad_sum=g) for l, g in zip(layers, G)], B, T, A.ADLOCO_F32, None, None, None,
                                A.ADLOCO_SUM_ONLY | flags)
            out.append([g.clone() for g in G])
    ctx.set_tuning("stats_variant", 1)
    for k in (0, 1):
        for x, y in zip(out[k], out[k + 2]):
            assert torch.equal(x, y)
