"""GPU parity of the region kernel of the Gram contraction (256 x 256 regions of A A^T and delta delta^T) against the CPU
oracle: sequence ends around the 256-row blocks, their halves and the 32-row blocks of the diagonal, either operand the
wider one, the fewest chunks of both, layers that share their activations (up to four to a group), strided rows.
Tolerance: exact products, fp32 sums, the bar of the 16-bit norms (2e-3; the same sums in another order differ by 1e-6)."""
import numpy as np
import pytest

import adloco_synth as synth
from oracle import adloco_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2508_18182_amd as A
    c = A.Context(0)
    c.set_tuning("stats_variant", 0)
    c.set_tuning("gram_variant", 3)
    yield c
    c.close()


def _check(ctx, host, share, B, T, dtype, pad=0):
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, code_of, new_acc, rel_err, to_dev
    for l, first in share.items():
        host[l]["a"] = host[first]["a"]
    want = orc.grad_stats([(l["a"], l["delta"]) for l in host], two_pass=False)

    def rows(x):
        x = to_dev(x)
        if not pad:
            return x
        wide = torch.full((B, T, x.shape[2] + pad), float("nan"), dtype=x.dtype, device=DEV)
        wide[:, :, :x.shape[2]] = x
        return wide[:, :, :x.shape[2]]

    a = {id(l["a"]): rows(l["a"]) for l in host}
    layers = [dict(a=a[id(l["a"])], delta=rows(l["delta"]), provided=True,
                   grad_sum=torch.zeros(l["d_out"], l["d_in"], device=DEV)) for l in host]
    for _ in range(2):
        ps, pl, acc = torch.zeros(B, device=DEV), torch.zeros(len(layers), B, device=DEV), new_acc()
        A.adloco_grad_stats(ctx, layers, B, T, code_of(dtype), ps, pl, acc)
        assert ctx.gram_kernel() == 3
        assert rel_err(pl.cpu().numpy(), want["n_layer_sample"]) < 1e-5
        assert rel_err(ps.cpu().numpy(), want["n_sample"]) < 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("T", [1, 32, 129, 255, 256, 257, 384, 511, 520, 769])
def test_sequence_ends(ctx, dtype, T):
    host = synth.custom_grad_stats_inputs(8100 + T, [(128, 192), (320, 128), (128, 128)], 2, T, dtype, std_delta=0.05, rho=0.5)
    _check(ctx, host, {}, 2, T, dtype)


@pytest.mark.parametrize("T", [200, 512, 600])
def test_shared_activations_and_strides(ctx, T):
    shapes = [(128, 256)] * 5 + [(256, 128), (192, 128)]
    host = synth.custom_grad_stats_inputs(8200 + T, shapes, 3, T, "bf16", std_delta=0.05, rho=0.5)
    _check(ctx, host, {1: 0, 2: 0, 3: 0, 4: 0}, 3, T, "bf16", pad=40)      # five readers: a group of four and one


def test_an_infinite_row_stays_with_its_sample(ctx):
    # the last token, which rows past the end of the sequence repeat
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc, to_dev
    B, T = 3, 300
    host = synth.custom_grad_stats_inputs(8300, [(128, 256)], B, T, "bf16", std_delta=0.05, rho=0.5)
    a, d = to_dev(host[0]["a"]), to_dev(host[0]["delta"])
    G = torch.zeros(256, 128, device=DEV)
    got = []
    for x in (0.0, float("inf")):
        a[1, T - 1, 5] = x
        ps, acc = torch.zeros(B, device=DEV), new_acc()
        A.adloco_grad_stats(ctx, [dict(a=a, delta=d, provided=True, grad_sum=G)], B, T, A.ADLOCO_BF16, ps, None, acc)
        assert ctx.gram_kernel() == 3
        got.append(ps.cpu().numpy())
    assert np.all(np.isfinite(got[0])) and not np.isfinite(got[1][1])
    assert got[0][0] == got[1][0] and got[0][2] == got[1][2]


@pytest.mark.parametrize("T", [700, 1024])
def test_another_batch_may_take_the_other_kernel_and_be_captured(T):
    # one sequence length: large batches take the region kernel, a single sample the dual-tile kernel and its job table
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc, to_dev
    shapes = [(512, 1536), (512, 512), (512, 2048), (2048, 512)]

    def call(B):
        host = synth.custom_grad_stats_inputs(8400 + B, shapes, B, T, "bf16", std_delta=0.05, rho=0.5)
        layers = [dict(a=to_dev(l["a"]), delta=to_dev(l["delta"]), provided=True,
                       grad_sum=torch.zeros(l["d_out"], l["d_in"], device=DEV)) for l in host]
        ps, pl, acc = torch.zeros(B, device=DEV), torch.zeros(len(layers), B, device=DEV), new_acc()
        return lambda c: A.adloco_grad_stats(c, layers, B, T, A.ADLOCO_BF16, ps, pl, acc), [ps, pl, acc]

    def context():
        c = A.Context(0)
        c.set_tuning("stats_variant", 0)
        return c

    (many, many_out), (one, one_out) = call(16), call(1)
    want = []
    for run, out, kernel in ((many, many_out, 3), (one, one_out, 2)):      # each on a context of its own
        with context() as own:
            run(own)
            torch.cuda.synchronize()
            assert own.gram_kernel() == kernel
            want.append([t.clone() for t in out])
    with context() as ctx:
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            many(ctx)
        torch.cuda.synchronize()
        builds = ctx.table_builds()
        with torch.cuda.stream(s):
            one(ctx)
        torch.cuda.synchronize()
        assert ctx.table_builds() == builds
    with context() as ctx:
        with torch.cuda.stream(s):
            many(ctx)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            one(ctx)
        for _ in range(3):
            for t in one_out + many_out:
                t.fill_(-1)
            g.replay()
            many(ctx)
            torch.cuda.synchronize()
            for got, w in zip(one_out + many_out, want[1] + want[0]):
                assert torch.equal(got, w)


def _gpt(d, blocks):
    return [(d, 3 * d, 0), (d, d, 1), (d, 4 * d, 2), (4 * d, d, 3)] * blocks


def _llama(d, ff, blocks):
    return [(d, d, 0), (d, d, 0), (d, d, 0), (d, d, 1), (d, ff, 2), (d, ff, 2), (ff, d, 3)] * blocks


@pytest.mark.parametrize("name,shapes,B,T,kernel", [
    # the dual-tile kernel contracts shared activations once only where no tile is ragged
    ("llama ragged", _llama(832, 2048, 2), 37, 500, 3),
    ("llama, whole tiles", _llama(1664, 3328, 1), 8, 512, 2),
    # two row blocks of 256: full, and nearly empty
    ("gpt2", _gpt(768, 2), 32, 512, 3),
    ("gpt2 ragged", _gpt(768, 2), 32, 300, 2),
    # few units: the XCD with the most of them counts
    ("two blocks of gpt2, few samples", _gpt(768, 2), 4, 512, 2),
    # tiles of the per-sample gradients, and where their starts and ends outweigh them
    ("llama, narrow and ragged", _llama(320, 768, 3), 43, 595, 0),
    ("llama, long and ragged", _llama(512, 1408, 4), 8, 1100, 0),
    ("llama, short", _llama(960, 2240, 3), 15, 27, 2),
    ("gpt, short", _gpt(1344, 8), 3, 32, 2),
])
def test_the_faster_way_is_taken(name, shapes, B, T, kernel):
    # (each measured: the other ways take 1.06 to 2.6 times as long)
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc
    g = torch.Generator(device=DEV).manual_seed(T)

    def rows(w):
        return torch.empty(B, T, w, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g)

    layers, acts = [], {}
    for i, (d_in, d_out, group) in enumerate(shapes):
        if i and shapes[i - 1][2] > group:
            acts = {}
        acts.setdefault(group, rows(d_in))
        layers.append(dict(a=acts[group], delta=rows(d_out), provided=True, grad_sum=None))
    got = {}
    for variant in (1, 2, 3):
        with A.Context(0) as ctx:
            ctx.set_tuning("gram_variant", variant)
            ctx.set_tuning("stats_variant", int(variant == 1))
            ps = torch.zeros(B, device=DEV)
            A.adloco_grad_stats(ctx, layers, B, T, A.ADLOCO_BF16, ps, None, new_acc())
            assert ctx.gram_kernel() == (kernel if variant == 1 else variant)
            got[variant] = ps.double()
    for v in (2, 3):
        assert float((got[1] / got[v] - 1).abs().max()) < 1e-4      # fp32 sums in another order


@pytest.mark.parametrize("shapes,B,T,kernel", [(_llama(960, 2240, 3), 15, 27, 2), (_gpt(512, 1), 8, 333, 0)])
def test_the_faster_way_to_form_gradient_sums_is_taken(shapes, B, T, kernel):
    # tiles of the per-sample gradients, or Gram contraction and sum over all rows where most of a chunk would be padding
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV, new_acc
    g = torch.Generator(device=DEV).manual_seed(T)
    layers = [dict(a=torch.empty(B, T, i, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g),
                   delta=torch.empty(B, T, o, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g)) for i, o, _ in shapes]
    got = []
    for stats_variant in (1, 0):
        with A.Context(0) as ctx:
            ctx.set_tuning("stats_variant", stats_variant)
            sums = [torch.zeros(o, i, device=DEV) for i, o, _ in shapes]
            ps = torch.zeros(B, device=DEV)
            A.adloco_grad_stats(ctx, [dict(l, grad_sum=s) for l, s in zip(layers, sums)], B, T, A.ADLOCO_BF16, ps, None, new_acc())
            assert stats_variant == 0 or ctx.gram_kernel() == kernel
            got.append([ps.double()] + [s.double() for s in sums])
    for x, y in zip(*got):
        assert float((x - y).norm() / y.norm()) < 1e-5              # fp32 sums in another order
