"""What this library is timed on: the calls that a training program makes of it, over the sizes it meets.

A program holds one context per GPU and, batch after batch, fresh activations and output gradients, its
parameters and optimizer state; every case goes through the package's public functions on such tensors.

Families (key "family" of a case):
  tiny    statistics, norm test and outer step of one very small layer: launches and host time only
  stats   adloco_grad_stats + adloco_norm_test over the blocks of a transformer
  train   a worker's inner step: gradient sum of a micro-batch (ADLOCO_SUM_ONLY), then fused AdamW
  ip      adloco_inner_products + adloco_inner_product_test
  outer   outer step over M instances, then the merge of all of them; instances as fp32 vectors or as
          bf16 drifts (packed first)
  round   adloco_round: one whole outer step of Algorithm 3 with a batch callback
"""
import math

import torch

import paper_2508_18182_amd as A

_DTYPES = {"f32": (torch.float32, A.ADLOCO_F32), "bf16": (torch.bfloat16, A.ADLOCO_BF16),
           "f16": (torch.float16, A.ADLOCO_F16)}
_RHO = 0.5             # share of every sample that the whole batch has in common
_STD_DELTA = 1e-2
_ETA, _B_CAP = 0.3, 256
_VOCAB = 50257
_contexts = {}


def listed():
    return [
        # The smallest workload of the benchmark: nothing but latency, launches and the read-back of the test.
        dict(name="tiny_f32", family="tiny", d_in=64, d_out=32, B=8, T=16, dtype="f32", M=2, N=10_000),
        # One micro-batch of the 350M round with the weight gradients supplied by the framework's backward:
        # the largest statistics call, and the one the benchmark times.
        dict(name="provided_350m", family="stats", layout="gpt", d=1024, ff=4096, blocks=24, B=32, T=1024,
             dtype="bf16", provided=True, aux=False, accumulate=False),
        # Llama-1B widths, q/k/v and gate/up reading one activation tensor, on sequences of twice the usual length.
        dict(name="provided_llama_long", family="stats", layout="llama", d=2048, ff=5632, blocks=2, B=16, T=2048,
             dtype="bf16", provided=True, aux=False, accumulate=False),
        # All 148 parameter blocks of GPT-2-small, gradient sums formed by the library: biases, normalisation
        # vectors and embedding tables next to the linear weights.
        dict(name="formed_gpt2_all_blocks", family="stats", layout="gpt", d=768, ff=3072, blocks=12, B=32, T=512,
             dtype="bf16", provided=False, aux=True, accumulate=False),
        # A small micro-batch of unpadded sequences in the paper's fp16, added to an accumulated batch: neither
        # T nor B * T is a multiple of anything.
        dict(name="formed_ragged_f16", family="stats", layout="gpt", d=768, ff=3072, blocks=12, B=5, T=1001,
             dtype="f16", provided=False, aux=False, accumulate=True),
        # Full precision activations (debugging, small models): the same path without 16-bit storage.
        dict(name="formed_f32", family="stats", layout="gpt", d=768, ff=3072, blocks=4, B=8, T=256,
             dtype="f32", provided=False, aux=False, accumulate=False),
        # What a worker does in every other inner step: the accumulated micro-batch's gradient sum and AdamW.
        dict(name="train_350m", family="train", layout="gpt", d=1024, ff=4096, blocks=24, B=32, T=1024, dtype="bf16"),
        # The inner-product tests on the GPT-2-small linears.
        dict(name="ip_gpt2", family="ip", layout="gpt", d=768, ff=3072, blocks=12, B=32, T=512, dtype="bf16"),
        # ... and where neither the type nor the sequence length suits the matrix cores.
        dict(name="ip_ragged_f32", family="ip", layout="gpt", d=768, ff=3072, blocks=1, B=4, T=250, dtype="f32"),
        # Outer step and merge of the 350M round: eight fp32 instances.
        dict(name="outer_350m_m8", family="outer", N=350_000_000, M=8, storage="f32", broadcast=False),
        # The same on bf16 drifts, 124M parameters and one more so that no vector is a multiple of four.
        dict(name="outer_drift_124m_m4", family="outer", N=124_000_001, M=4, storage="bf16", broadcast=False),
        # One outer step of Algorithm 3 on a small model: three trainers with different batches (one of them in
        # switch mode), two workers each, a merge; many short calls from the native driver.
        dict(name="round_small_f16", family="round", k=3, M=2, H=3, d=256, ff=1024, blocks=4, T=128, dtype="f16",
             b0=2, b1=24, b2=5, b3=0, b_max=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _widths(rng, lo, hi, odd):
    """Model width: mostly a multiple of 64, sometimes of 8, sometimes (odd) anything."""
    d = _log_int(rng, lo, hi)
    if odd:
        return d | 1
    u = 64 if rng.random() < 0.8 and d >= 64 else 8
    return max(u, d // u * u)


def _tokens(rng, lo, hi):
    T = _log_int(rng, lo, hi)
    p = rng.random()
    if p < 0.4 and T >= 128:
        return T // 128 * 128
    if p < 0.6 and T >= 32:
        return T // 32 * 32
    return T


def draw(rng):
    family = rng.choice(["tiny", "stats", "stats", "stats", "train", "ip", "outer", "round"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    if family == "tiny":
        return dict(family=family, d_in=_log_int(rng, 8, 256), d_out=_log_int(rng, 8, 256), B=rng.randint(2, 16),
                    T=rng.randint(1, 64), dtype=dtype, M=rng.randint(1, 4), N=_log_int(rng, 1000, 100_000))
    if family == "outer":
        M = rng.randint(1, 16)
        N = min(_log_int(rng, 10_000, 350_000_000), 3_500_000_000 // (M + 2))
        return dict(family=family, N=N, M=M, storage=rng.choice(["f32", "bf16"]), broadcast=rng.random() < 0.3)
    if family == "round":
        k = rng.randint(1, 4)
        b = [_log_int(rng, 1, 48) if i < k else 0 for i in range(4)]
        d = _widths(rng, 64, 512, rng.random() < 0.1)
        return dict(family=family, k=k, M=rng.randint(1, 3), H=rng.randint(1, 4), d=d, ff=4 * d,
                    blocks=rng.randint(1, 6), T=_tokens(rng, 16, 256), dtype=dtype, b0=b[0], b1=b[1], b2=b[2], b3=b[3],
                    b_max=rng.choice([4, 8, 16]))
    layout = rng.choice(["gpt", "gpt", "llama"])
    odd = rng.random() < 0.15
    d = _widths(rng, 128, 2048, odd)
    ff = 4 * d if layout == "gpt" else (_widths(rng, 2 * d, 3 * d, odd))
    c = dict(family=family, layout=layout, d=d, ff=ff, blocks=_log_int(rng, 1, 24), B=_log_int(rng, 1, 64),
             T=_tokens(rng, 32, 4096), dtype=dtype)
    if family == "stats":
        c.update(provided=rng.random() < 0.5, aux=layout == "gpt" and rng.random() < 0.3, accumulate=rng.random() < 0.3)
    # no drawn case costs more than the largest listed one, on the slow paths (fp32, rows that are not
    # 16-byte aligned, for the inner products also ragged sequences) no more than they can take
    slow = dtype == "f32" or d % 8 or ff % 8
    flops = 3e11 if slow else 1.6e13
    if family == "ip":
        flops = 2e10 if slow or c["T"] % 32 else 2.7e12
    while 2 * c["B"] * c["T"] * _params(c) > flops or work(c)["bytes"] > 2.4e10:
        key = "blocks" if c["blocks"] > 1 else "B" if c["B"] > 1 else "T"
        c[key] = max(1, c[key] // 2)
    return c


# ---- shapes --------------------------------------------------------------------------------------------

def _linears(case):
    """(activation group, d_in, d_out) of the linear layers of one transformer block; layers with the same group
    read the same activation tensor."""
    d, ff = case["d"], case["ff"]
    if case.get("layout", "gpt") == "gpt":
        return [("h", d, 3 * d), ("o", d, d), ("f", d, ff), ("p", ff, d)]
    return [("h", d, d), ("h", d, d), ("h", d, d), ("o", d, d), ("f", d, ff), ("f", d, ff), ("p", ff, d)]


def _aux_vectors(case):
    """Number of normalisation layers (each a gain and a bias of width d) of the model."""
    return 2 * case["blocks"] + 1


def _params(case):
    return case["blocks"] * sum(i * o for _, i, o in _linears(case))


def _all_params(case):
    n = _params(case)
    if case.get("aux"):
        n += case["blocks"] * sum(o for _, _, o in _linears(case)) + 2 * _aux_vectors(case) * case["d"]
        n += (_VOCAB + case["T"]) * case["d"]
    return n


def _input_elements(case):
    """Elements of a and delta per token, every distinct tensor once."""
    block = {}
    for g, i, _ in _linears(case):
        block[g] = i
    n = case["blocks"] * (sum(block.values()) + sum(o for _, _, o in _linears(case)))
    if case.get("aux"):
        n += 2 * _aux_vectors(case) * case["d"] + case["d"]
    return n


# ---- inputs --------------------------------------------------------------------------------------------

class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, shape, std, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=self.g)

    def rows(self, B, T, d, std, dtype):
        """[B, T, d] with a component that the samples of the batch share."""
        x = self.normal((B, T, d), std * math.sqrt(1 - _RHO * _RHO), dtype)
        return x.add_(self.normal((1, T, d), std * _RHO, dtype))

    def ids(self, B, T):
        """Token ids with a Zipf-like profile: few ids many times, most ids hardly ever."""
        u = torch.rand((B, T), device="cuda", generator=self.g)
        rank = torch.exp(u * math.log(_VOCAB)).to(torch.int64) - 1
        return ((rank * 7919) % _VOCAB).to(torch.int32)


def _context():
    """The context that a program keeps for its GPU."""
    dev = torch.cuda.current_device()
    if dev not in _contexts:
        _contexts[dev] = A.Context(dev)
    return _contexts[dev]


def _layers(case, r):
    """Layer list with all inputs, gradient sums laid out back to back in one vector."""
    tdt, _ = _DTYPES[case["dtype"]]
    B, T, d = case["B"], case["T"], case["d"]
    G = torch.zeros(_all_params(case), device="cuda")
    if case.get("provided"):
        # what the framework's backward holds: of the size that B * T such products add up to
        G.copy_(r.normal(G.shape, _STD_DELTA * math.sqrt(B * T)))
    layers, at = [], 0

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return G[at - n:at].view(*shape)

    for _ in range(case["blocks"]):
        acts = {}
        for g, i, o in _linears(case):
            if g not in acts:
                acts[g] = r.rows(B, T, i, 1.0, tdt)
            delta = r.rows(B, T, o, _STD_DELTA, tdt)
            layers.append(dict(a=acts[g], delta=delta, grad_sum=take(o, i), provided=bool(case.get("provided"))))
            if case.get("aux"):
                layers.append(dict(kind="vector", delta=delta, grad_sum=take(o), provided=bool(case["provided"])))
    if case.get("aux"):
        for _ in range(_aux_vectors(case)):
            x, delta = r.rows(B, T, d, 1.0, tdt), r.rows(B, T, d, _STD_DELTA, tdt)
            for gain in (True, False):
                layers.append(dict(kind="vector", x=x if gain else None, delta=delta, grad_sum=take(d),
                                   provided=bool(case["provided"])))
        delta = r.rows(B, T, d, _STD_DELTA, tdt)
        pos = torch.arange(T, dtype=torch.int32, device="cuda").expand(B, T).contiguous()
        layers.append(dict(kind="embed", ids=r.ids(B, T), vocab=_VOCAB, delta=delta, grad_sum=take(_VOCAB, d)))
        layers.append(dict(kind="embed", ids=pos, vocab=T, delta=delta, grad_sum=take(T, d)))
    assert at == G.numel()
    return layers, G


def _acc(n=2):
    return torch.zeros(n, dtype=torch.float64, device="cuda")


def prepare(case, seed):
    r = _Draw(seed)
    s = dict(case=dict(case), ctx=_context())
    f = case["family"]
    if f in ("stats", "train", "ip"):
        s["layers"], s["G"] = _layers(case, r)
        s["dt"] = _DTYPES[case["dtype"]][1]
        s["per_sample"] = torch.zeros(case["B"], device="cuda")
        s["per_layer"] = torch.zeros(len(s["layers"]), case["B"], device="cuda")
        s["acc"] = _acc()
    if f == "ip":
        # G and S1 of the batch, from the statistics that come before the inner products
        A.adloco_grad_stats(s["ctx"], s["layers"], case["B"], case["T"], s["dt"], s["per_sample"], None, s["acc"])
        s["ip"], s["ip_acc"] = torch.zeros(case["B"], device="cuda"), _acc(4)
    elif f == "train":
        n = s["G"].numel()
        s.update(theta=r.normal((n,), 0.02), m=r.normal((n,), 1e-4), v=r.normal((n,), 1e-4).square_(), step=100)
    elif f == "tiny":
        tdt, s["dt"] = _DTYPES[case["dtype"]]
        B, T, i, o = case["B"], case["T"], case["d_in"], case["d_out"]
        s["G"] = torch.zeros(o * i, device="cuda")
        s["layers"] = [dict(a=r.rows(B, T, i, 1.0, tdt), delta=r.rows(B, T, o, 1.0, tdt), grad_sum=s["G"].view(o, i))]
        s["per_sample"], s["acc"] = torch.zeros(B, device="cuda"), _acc()
    if f in ("tiny", "outer"):
        N, M = case["N"], case["M"]
        s["theta"], s["mom"] = r.normal((N,), 0.02), r.normal((N,), 1e-4)
        s["inst"] = [s["theta"] - r.normal((N,), 1e-3) for _ in range(M)]
        if case.get("storage") == "bf16":
            s["drift"] = [torch.zeros(N, dtype=torch.bfloat16, device="cuda") for _ in range(M)]
            s["rep"] = s["theta"].clone()
    if f == "round":
        s["round"] = _round_state(case, r)
    return s


def _round_state(case, r):
    tdt, dt = _DTYPES[case["dtype"]]
    T, d = case["T"], case["d"]
    blocks = []
    for _ in range(case["blocks"]):
        for _, i, o in _linears(case):
            blocks += [dict(d_in=i, d_out=o), dict(kind="vector", d_out=o)]
        blocks += [dict(kind="vector", d_out=d), dict(kind="vector", d_out=d)]
    N = sum(b.get("d_in", 1) * b["d_out"] for b in blocks)
    b_max = case["b_max"]
    trainers = []
    for i in range(case["k"]):
        theta = r.normal((N,), 0.02)
        trainers.append(dict(
            uid=i, b_req=case["b%d" % i], theta_outer=theta, momentum=r.normal((N,), 1e-4), acc=_acc(),
            per_sample_sqnorm=torch.zeros(b_max * 2, device="cuda"),
            workers=[dict(theta=torch.zeros(N, device="cuda"), exp_avg=r.normal((N,), 1e-4), grad=torch.zeros(N, device="cuda"),
                          exp_avg_sq=r.normal((N,), 1e-4).square_(), step=10) for _ in range(case["M"])]))
    # what the model leaves behind for one batch of the largest size; a smaller batch takes its first samples
    data = []
    for _ in range(case["blocks"]):
        for _, i, o in _linears(case):
            a, delta = r.rows(b_max, T, i, 1.0, tdt), r.rows(b_max, T, o, _STD_DELTA, tdt)
            data += [dict(a=a, delta=delta), dict(x=None, delta=delta)]
        x, delta = r.rows(b_max, T, d, 1.0, tdt), r.rows(b_max, T, d, _STD_DELTA, tdt)
        data += [dict(x=x, delta=delta), dict(x=None, delta=delta)]
    cfg = dict(T=T, dtype=dt, inner_steps=case["H"], n_switch=2, merge_w=2 if case["k"] > 2 else 0, nesterov=1, b_max=b_max,
               b_cap=64, eta=_ETA, lr_inner=4e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.1, lr_outer=0.5, mu_outer=0.9)
    return dict(trainers=trainers, blocks=blocks, cfg=cfg, data=data, N=N)


# ---- one pass ------------------------------------------------------------------------------------------

def _test_outputs(t):
    """The norm test's answer: figures, and decisions."""
    figures = [t["S1"], t["S2"], t["batch_grad_sqnorm"], t["variance"], t["stat"]]
    return dict(figures=figures, b_req=t["b_req"], b_micro=t["b_micro"], accum_steps=t["accum_steps"], n=t["n_samples"])


def run(s):
    c, ctx, f = s["case"], s["ctx"], s["case"]["family"]
    if f == "round":
        return _run_round(s)
    out = {}
    if f in ("stats", "tiny"):
        flags = A.ADLOCO_ACCUMULATE if c.get("accumulate") else 0
        A.adloco_grad_stats(ctx, s["layers"], c["B"], c["T"], s["dt"], s["per_sample"], s.get("per_layer"), s["acc"], flags)
        t = A.adloco_norm_test(ctx, s["layers"], s["acc"], _ETA, c["B"], 32, 2, _B_CAP)
        out = dict(per_sample=s["per_sample"], S1=s["acc"][:1], n=s["acc"].view(torch.int64)[1:2], test=_test_outputs(t))
        if "per_layer" in s:
            out["per_layer"] = s["per_layer"]
        if not c.get("provided"):
            out["G"] = s["G"]
    elif f == "train":
        A.adloco_grad_stats(ctx, s["layers"], c["B"], c["T"], s["dt"], None, None, None, A.ADLOCO_ACCUMULATE | A.ADLOCO_SUM_ONLY)
        A.adloco_inner_step(ctx, s["theta"], s["m"], s["v"], s["G"], s["step"], 4e-4, grad_scale=0.5 / c["B"])
        out = dict(G=s["G"], theta=s["theta"], m=s["m"], v=s["v"])
    elif f == "ip":
        A.adloco_inner_products(ctx, s["layers"], c["B"], c["T"], s["dt"], s["ip"], s["per_sample"], s["ip_acc"])
        t = A.adloco_inner_product_test(ctx, s["layers"], s["acc"], s["ip_acc"], 0.01, 0.3, c["B"], 32, 2, _B_CAP)
        out = dict(ip=s["ip"], per_sample=s["per_sample"], sums=s["ip_acc"][:2], S2=t["S2"], var_ip=t["var_ip"], var_aug=t["var_aug"],
                   b_req_ip=t["b_req_ip"], b_req_aug=t["b_req_aug"], n=t["n_samples"])
    if f in ("tiny", "outer"):
        flags = A.ADLOCO_BROADCAST if c.get("broadcast") else 0
        if c.get("storage") == "bf16":
            for x, q in zip(s["inst"], s["drift"]):
                A.adloco_pack_drift(ctx, s["theta"], x, q)
            A.adloco_merge_drift(ctx, s["rep"], s["drift"][1:], 64.0, [32.0 + j for j in range(c["M"] - 1)])
            A.adloco_outer_step_drift(ctx, s["theta"], s["drift"], s["mom"], 0.7, 0.9, True, flags)
            out.update(theta=s["theta"], mom=s["mom"], rep=s["rep"])
        else:
            A.adloco_outer_step(ctx, s["theta"], s["inst"], s["mom"], 0.7, 0.9, True, flags)
            out.update(theta=s["theta"], mom=s["mom"])
            if f == "outer":
                A.adloco_merge(ctx, s["inst"], [32.0 + j for j in range(c["M"])])
                out["merged"] = s["inst"][-1]
    return out


def _run_round(s):
    q = s["round"]
    # every pass is the outer step of a program whose trainers ask for the case's batches
    trainers = [dict(t, workers=[dict(w) for w in t["workers"]]) for t in q["trainers"]]

    def batch(uid, worker, inner_step, micro_step, b, theta):
        return [{k: v if v is None else v[:b] for k, v in e.items()} for e in q["data"]]

    reports = A.adloco_round(s["ctx"], q["cfg"], trainers, q["blocks"], batch)
    out = dict(left=len(trainers))
    for i, (t, rep) in enumerate(zip(trainers, reports)):
        out["trainer%d" % i] = dict(theta=t["theta_outer"], mom=t["momentum"], uid=t["uid"], b_req=t["b_req"],
                                    grad=t["workers"][-1]["grad"], m=t["workers"][0]["exp_avg"],
                                    v=t["workers"][0]["exp_avg_sq"], test=_test_outputs(rep["test"]))
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------------

def _esize(case):
    return 4 if case["dtype"] == "f32" else 2


def work(case):
    f = case["family"]
    if f == "tiny":
        B, T, i, o = case["B"], case["T"], case["d_in"], case["d_out"]
        return dict(bytes=B * T * (i + o) * _esize(case) + 4 * i * o + 4 * case["N"] * (case["M"] + 4), flops=2 * B * T * i * o)
    if f == "outer":
        N, M = case["N"], case["M"]
        if case["storage"] == "f32":
            step, merge = 4 * (M + 2) + 8, 4 * M + 4 if M > 1 else 0
            return dict(bytes=N * (step + merge + (4 * M if case["broadcast"] else 0)), flops=N * 4 * M)
        pack, step, merge = 10 * M, 16 + 2 * M, 8 + 2 * (M - 1) if M > 1 else 0
        return dict(bytes=N * (pack + step + merge + (2 * M if case["broadcast"] else 0)), flops=N * 4 * M)
    if f == "round":
        P = case["blocks"] * (sum(i * o + o for _, i, o in _linears(case)) + 2 * case["d"])
        tokens, steps = 0, 0
        asked = sorted(case["b%d" % j] for j in range(case["k"]))
        for b in asked[1:] if case["k"] > 2 else asked:      # (of three or more trainers the smallest two merge)
            b_max = case["b_max"]
            samples = -(-b // b_max) * b_max if b > 2 * b_max else min(b, b_max)
            tokens += samples * case["T"] * case["M"] * case["H"]
            steps += case["M"] * case["H"]
        return dict(bytes=steps * P * 28 + tokens * _input_elements(case) * _esize(case), flops=2 * tokens * P)
    B, T, P = case["B"], case["T"], _params(case)
    inputs = B * T * _input_elements(case) * _esize(case)
    if f == "train":
        return dict(bytes=inputs + 8 * P + 28 * P, flops=2 * B * T * P)
    if f == "ip":
        return dict(bytes=inputs + 4 * P, flops=2 * B * T * P)
    if case["provided"]:
        # the cheaper of the Gram identity (symmetric half) and the per-sample gradient itself, layer by layer
        flops = case["blocks"] * B * sum(min(T * (T + 1) * (i + o), 2 * T * i * o) for _, i, o in _linears(case))
    else:
        flops = 2 * B * T * P
    rw = 2 if case["accumulate"] and not case["provided"] else 1
    return dict(bytes=inputs + 4 * rw * _all_params(case), flops=flops)


def tolerance(case):
    """About four times what the path differs by from the same sums in 64 bits (in brackets, measured)."""
    f = case["family"]
    if f == "outer":
        return {"rel": 1e-7}        # fp64 in registers, one rounding to fp32 (2.5e-8)
    if f == "ip":
        return {"rel": 1e-4}        # a variance is a difference of sums of near-equal terms (1.5e-5; the sums: 5e-7)
    if f == "round":
        return {"rel": 2e-5}        # Delta is a difference of parameters twenty times its size
    return {"rel": 1e-5}            # fp32 sums over up to 2^18 token rows (1.0e-6 over 2^15)
