"""The tile lists of the statistics serve every batch size and sequence length on the same list of shapes: nothing is built,
allocated or waited for when either changes, so that a call on another batch can be captured and a captured one replays
after it.  Without the memory for a tile route, a call takes the Gram contraction."""
import numpy as np
import pytest

import adloco_synth as synth

pytestmark = pytest.mark.gpu

SHAPES = [(64, 192), (192, 64)]
# element type, gradients supplied, then (B, T): the largest batch first, and smaller ones that take the same route
CASES = [("f32", False, [(6, 40), (4, 33), (1, 40), (5, 24)]),
         ("f16", False, [(6, 100), (4, 77), (1, 96), (5, 64)]),
         ("bf16", True, [(200, 600), (150, 520), (200, 513)]),
         ("f32", True, [(40, 640), (33, 610), (40, 609)])]


def _call(A, ctx, dtype, provided, B, T, seed=0):
    import torch
    from gpu_util import DEV, code_of, new_acc, to_dev
    host = synth.custom_grad_stats_inputs(9000 + B + T + seed, SHAPES, B, T, dtype, std_delta=0.2, rho=0.4)
    layers = [dict(a=to_dev(l["a"]), delta=to_dev(l["delta"]), provided=provided,
                   grad_sum=torch.zeros(l["d_out"], l["d_in"], device=DEV)) for l in host]
    ps, pl, acc = torch.zeros(B, device=DEV), torch.zeros(len(layers), B, device=DEV), new_acc()

    def run():
        A.adloco_grad_stats(ctx, layers, B, T, code_of(dtype), ps, pl, acc)

    return run, [ps, pl, acc] + [l["grad_sum"] for l in layers]


@pytest.mark.parametrize("dtype,provided,batches", CASES)
def test_other_batches_build_nothing_and_can_be_captured(dtype, provided, batches):
    import torch
    import paper_2508_18182_amd as A
    ctx = A.Context(0)
    calls = [_call(A, ctx, dtype, provided, B, T) for B, T in batches]
    want = []
    for (B, T), (run, outs) in zip(batches, calls):          # each on a context of its own
        own = A.Context(0)
        one, o = _call(A, own, dtype, provided, B, T)
        own.set_tuning("profile", 1)
        one()
        torch.cuda.synchronize()
        assert own.profile_read("tile_stats")[1] == 1
        want.append([t.clone() for t in o])
        own.close()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        calls[0][0]()
    torch.cuda.synchronize()
    builds = ctx.table_builds()
    graphs = []
    for run, outs in calls[1:]:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            run()
        graphs.append(g)
    for rep in range(3):
        for g, (run, outs), w in zip(graphs, calls[1:], want[1:]):
            for t in outs:
                t.fill_(-1)
            g.replay()
            torch.cuda.synchronize()
            for a, b in zip(outs if not provided else outs[:3], w):
                assert torch.equal(a, b)
            calls[0][0]()                                    # eager work on the first batch in between
            torch.cuda.synchronize()
            for a, b in zip(calls[0][1] if not provided else calls[0][1][:3], want[0]):
                assert torch.equal(a, b)
    assert ctx.table_builds() == builds
    ctx.close()


def test_without_memory_for_the_tiles():
    # fp32: the partial tiles of the list take 16 MiB, everything else less than the limit
    import torch
    import paper_2508_18182_amd as A
    got = []
    for limit in (0, 256):
        ctx = A.Context(0)
        ctx.set_tuning("scratch_limit_kb", limit)
        ctx.set_tuning("profile", 1)
        run, outs = _call(A, ctx, "f32", False, 3000, 4)
        run()
        torch.cuda.synchronize()
        assert (ctx.profile_read("tile_stats")[1], ctx.profile_read("gram")[1]) == ((1, 0) if limit == 0 else (0, 1))
        got.append([t.double().cpu().numpy() for t in outs])
        ctx.close()
    for a, b in zip(got[0][:2], got[1][:2]):
        assert np.max(np.abs(a - b) / np.abs(b)) < 1e-4
    for a, b in zip(got[0][3:], got[1][3:]):
        assert np.max(np.abs(a - b)) < 1e-4 * np.sqrt(np.mean(b * b))


def test_inner_products_keep_the_list_of_either_tile_width():
    # {768 -> 2304}, B 8: 64-wide tiles up to T 64, 128-wide ones from T 100 on; what belongs to B and T is one table
    import torch
    import paper_2508_18182_amd as A
    from gpu_util import DEV
    B, g = 8, torch.Generator().manual_seed(77)
    calls = []
    for T in (64, 128):
        layers = [dict(a=torch.randn(B, T, 768, generator=g).cuda(), delta=torch.randn(B, T, 2304, generator=g).cuda(),
                       grad_sum=torch.randn(2304, 768, generator=g).cuda())]
        calls.append((T, layers))
    ctx, seen = A.Context(0), []
    for _ in range(3):
        for T, layers in calls:
            dots, acc = torch.zeros(B, device=DEV), torch.zeros(4, dtype=torch.float64, device=DEV)
            builds = ctx.table_builds()
            A.adloco_inner_products(ctx, layers, B, T, A.ADLOCO_F32, dots, None, acc)
            seen.append(ctx.table_builds() - builds)
            want = torch.stack([(layers[0]["delta"][i].double().t() @ layers[0]["a"][i].double() *
                                 layers[0]["grad_sum"].double()).sum() for i in range(B)])
            assert float((dots.double() - want).norm() / want.norm()) < 1e-5
    assert seen[2:] == [1, 1, 1, 1]
    ctx.close()
