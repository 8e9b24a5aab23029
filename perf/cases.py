"""The work a user of the protected attention layer has it do, as cases to
measure: training steps (forward and backward) of the fused and of the
materialised path, forwards of the allocation-free entry point, the fp32
layer, and the standalone encoder and verifier. Sizes are those of the
layer's workloads (`workloads/`: the single fp32 head, the encoder and
GPT-2 layers, the two large decoders) and generic ones around them.

A case's `op`:
  "step"     ProtectedAttention.forward, then .backward
  "forward"  ProtectedAttention.forward
  "serve"    attn_abft_forward_noalloc
  "guard"    encode_checksums of a matrix, then verify_and_correct of it
Inputs: X and dO from N(0, 1), weights from N(0, w_std^2), as the layer's
workloads draw them, rounded to the storage type.
"""
import math

import torch

from paper_2410_11720_amd import abft

CAPACITY = 256  # events a report holds


def _case(op, batch, seq, hidden, heads, *, dtype="bf16", causal=True, fused=True, block_rows=128,
          sections=abft.SEC_ALL, protect=True, name=None):
    c = dict(op=op, batch=batch, seq=seq, hidden=hidden, heads=heads, dtype=dtype, causal=causal,
             fused=fused, block_rows=block_rows, sections=sections, protect=protect)
    if name:
        c["name"] = name
    return c


def _guard(batch, rows, cols, block_rows, block_cols, dtype, name=None):
    c = dict(op="guard", batch=batch, rows=rows, cols=cols, block_rows=block_rows,
             block_cols=block_cols, dtype=dtype)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one fp32 head of 128 tokens, where launches and latency count
        _case("forward", 1, 128, 64, 1, dtype="f32", causal=False, fused=False,
              name="single_head_f32"),
        # one short prompt through the GPT-2 layer without allocating (serving under graph capture)
        _case("serve", 1, 128, 768, 12, name="serve_prompt"),
        # a full prefill batch of the same layer, the largest its scratch buffer documents
        _case("serve", 8, 1024, 768, 12, name="serve_prefill"),
        # BERT-base encoder layer, one training step
        _case("step", 8, 512, 768, 12, causal=False, name="encoder_step"),
        # GPT-2 layer, one training step: the headline workload
        _case("step", 8, 1024, 768, 12, name="gpt2_step"),
        # the same step on the default path, which stores AS and AP as the paper does
        _case("step", 8, 1024, 768, 12, fused=False, name="gpt2_step_materialised"),
        # the same step on one that the adaptive frequencies leave unchecked
        _case("step", 8, 1024, 768, 12, sections=0, name="gpt2_step_unchecked"),
        # ragged sizes: 864 tokens a sequence in blocks of 32, five heads, three sequences
        _case("step", 3, 864, 320, 5, fused=False, block_rows=32, name="ragged_step"),
        # fp32 training step (the type the materialised path offers for full precision)
        _case("step", 2, 512, 768, 12, dtype="f32", fused=False, name="step_f32"),
        # large decoder layer, head dim 128
        _case("step", 4, 2048, 4096, 32, name="decoder_step"),
        # the longest sequence, one tensor-parallel shard of a wide layer, on the default path
        _case("step", 1, 4096, 5120, 40, fused=False, name="long_step_materialised"),
        # a stored tensor guarded by its own checksums: encoded, later verified
        _guard(8, 1024, 2304, 128, 64, "bf16", name="guard_qkv"),
    ]


STEP_FLOPS = 2.5e12     # below the largest listed step
STEP_FLOPS_F32 = 1.0e11  # fp32 matrix rates are lower
SERVE_BYTES = 60e6      # what the allocation-free forward's buffer holds


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["step", "step", "step", "step", "serve", "serve", "f32", "guard"])
        if kind == "guard":
            rb, cb = rng.choice([32, 64, 128]), rng.choice([64, 128])
            return _guard(_log_int(rng, 1, 16), rb * _log_int(rng, 1, 2048 // rb),
                          cb * _log_int(rng, 1, 5120 // cb), rb, cb, rng.choice(["bf16", "f32"]))
        d = rng.choice([64, 64, 128])
        heads = _log_int(rng, 1, 40)
        dtype = "f32" if kind == "f32" else "bf16"
        fused = dtype == "bf16" and (kind == "serve" or rng.random() < 0.6)
        r = rng.choice([32, 64, 128, 128])
        grain = 128 if fused else r
        seq = grain * _log_int(rng, 1, 4096 // grain)
        if seq > 4096:
            continue
        batch = _log_int(rng, 1, 16)
        c = _case({"f32": rng.choice(["step", "forward"])}.get(kind, kind), batch, seq, heads * d,
                  heads, dtype=dtype, causal=rng.random() < 0.7, fused=fused, block_rows=r,
                  sections=rng.choice([abft.SEC_ALL] * 5 + [0]) if kind == "step" else abft.SEC_ALL)
        t = batch * seq
        if kind == "serve" and t * (8 * c["hidden"] + 32 * heads) + (t // r) * 56 * c["hidden"] > SERVE_BYTES:
            continue
        if work(c)["flops"] > (STEP_FLOPS_F32 if dtype == "f32" else STEP_FLOPS):
            continue
        if not fused and batch * heads * seq * seq > 1.2e9:  # score-shaped tensors in memory
            continue
        return c


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _randn(shape, std, dtype, gen):
    return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = _dtype(case)
    if case["op"] == "guard":
        return dict(C=_randn((case["batch"], case["rows"], case["cols"]), 1.0, dt, gen))
    B, S, H = case["batch"], case["seq"], case["hidden"]
    w_std = 0.02 if H <= 1024 else 0.01
    return dict(X=_randn((B, S, H), 1.0, dt, gen), Wqkv=_randn((H, 3 * H), w_std, dt, gen),
                Wo=_randn((H, H), w_std, dt, gen), dO=_randn((B, S, H), 1.0, dt, gen))


def _zeroed_report():
    report = torch.zeros(abft.attn_abft_report_bytes(CAPACITY), dtype=torch.uint8, device="cuda")
    abft.attn_abft_report_init(report, CAPACITY)
    return report


def prepare(case, seed):
    st = dict(case=case, **_inputs(case, seed))
    if case["op"] == "guard":
        B, M, N = case["batch"], case["rows"], case["cols"]
        rb, cb = case["block_rows"], case["block_cols"]
        st["col"] = torch.empty((B, M // rb, 2, N), dtype=torch.float32, device="cuda")
        st["row"] = torch.empty((B, M, N // cb, 2), dtype=torch.float32, device="cuda")
        st["report"] = _zeroed_report()
        return st
    cfg = abft.LayerConfig(case["batch"], case["seq"], case["hidden"], case["heads"],
                           dtype=case["dtype"], causal=case["causal"],
                           block_rows=case["block_rows"], sections=case["sections"],
                           protect=case["protect"], fused=case["fused"])
    if case["op"] == "serve":
        st.update(cfg=cfg, O=torch.empty_like(st["X"]), report=_zeroed_report())
        return st
    layer = abft.ProtectedAttention(cfg, capacity=CAPACITY)
    layer.report, layer.report_bwd = _zeroed_report(), _zeroed_report()
    st["layer"] = layer
    return st


def run(st):
    case = st["case"]
    if case["op"] == "guard":
        B, M, N = case["batch"], case["rows"], case["cols"]
        rb, cb = case["block_rows"], case["block_cols"]
        dt = abft.FP32 if case["dtype"] == "f32" else abft.BF16
        abft.encode_checksums(st["C"], dt, B, M, N, N, M * N, rb, cb, st["col"], st["row"])
        abft.verify_and_correct(st["C"], dt, B, M, N, N, M * N, rb, cb, st["col"], st["row"],
                                1e10, 1e5, 0.0, abft.OP_ID["O"], st["report"])
        return dict(C=st["C"], col=st["col"], row=st["row"], report=st["report"])
    X, Wqkv, Wo = st["X"], st["Wqkv"], st["Wo"]
    if case["op"] == "serve":
        abft.attn_abft_forward_noalloc(st["cfg"], X, Wqkv, Wo, st["O"], None, 0, st["report"])
        return dict(O=st["O"], report=st["report"])
    layer = st["layer"]
    O = layer.forward(X, Wqkv, Wo)
    if case["op"] == "forward":
        return dict(O=O, report=layer.report)
    dX, dWqkv, dWo = layer.backward(st["dO"], X, Wqkv, Wo)
    return dict(O=O, dX=dX, dWqkv=dWqkv, dWo=dWo, report=layer.report,
                report_bwd=layer.report_bwd)


def _pairs(case):
    S = case["seq"]
    return S * (S + 1) // 2 if case["causal"] else S * S


def work(case):
    es = 4 if case["dtype"] == "f32" else 2
    if case["op"] == "guard":
        n = case["batch"] * case["rows"] * case["cols"]
        chk = 8 * (n // case["block_rows"] + n // case["block_cols"])
        # read to encode, read to verify; checksums written, then read
        return dict(bytes=2 * n * es + 2 * chk, flops=2 * 4 * n)
    T, H = case["batch"] * case["seq"], case["hidden"]
    fwd = 8 * T * H * H + 4 * case["batch"] * H * _pairs(case)
    acts, weights = T * H * es, 4 * H * H * es
    if case["op"] != "step":
        return dict(bytes=2 * acts + weights, flops=fwd)
    # X and dO in, O and dX out; the weights in; their fp32 gradients out
    return dict(bytes=4 * acts + weights + 4 * H * H * 4, flops=3 * fwd)


def tolerance(case):
    """About four times the distance from the 64-bit result: bf16 storage of
    Q, K, V, the probabilities and the gradients between the products; fp32
    sums otherwise."""
    if case["op"] == "guard":
        return {"rel": 1e-6, "max": 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 1.5e-2, "max": 0.3}


def _exact_layer(case, inp):
    B, S, H, nh = case["batch"], case["seq"], case["hidden"], case["heads"]
    d = H // nh
    X, W, Wo, dO = (inp[k].double() for k in ("X", "Wqkv", "Wo", "dO"))
    scale = 1.0 / math.sqrt(d)
    mask = None
    if case["causal"]:
        mask = torch.ones((S, S), dtype=torch.bool, device="cuda").triu(1)
    QKV = (X.view(-1, H) @ W).view(B, S, 3 * H)
    CL = torch.empty((B, S, H), dtype=torch.float64, device="cuda")
    step = case["op"] == "step"
    dCL = (dO.view(-1, H) @ Wo.t().contiguous()).view(B, S, H) if step else None
    dQKV = torch.empty_like(QKV) if step else None
    for b in range(B):
        for h in range(nh):
            q, k, v = (QKV[b, :, i * H + h * d:i * H + (h + 1) * d].contiguous() for i in range(3))
            P = q @ k.t().contiguous()
            P.mul_(scale)
            if mask is not None:
                P.masked_fill_(mask, -math.inf)
            P = torch.softmax(P, dim=1)
            CL[b, :, h * d:(h + 1) * d] = P @ v
            if step:
                g = dCL[b, :, h * d:(h + 1) * d].contiguous()
                dP = g @ v.t().contiguous()
                dP = P * (dP - (P * dP).sum(1, keepdim=True)) * scale
                dQKV[b, :, h * d:(h + 1) * d] = dP @ k
                dQKV[b, :, H + h * d:H + (h + 1) * d] = dP.t().contiguous() @ q
                dQKV[b, :, 2 * H + h * d:2 * H + (h + 1) * d] = P.t().contiguous() @ g
    out = dict(O=(CL.view(-1, H) @ Wo).view(B, S, H), report=None)
    if step:
        g2, x2 = dQKV.view(-1, 3 * H), X.view(-1, H)
        out.update(dX=(g2 @ W.t().contiguous()).view(B, S, H), dWqkv=x2.t().contiguous() @ g2,
                   dWo=CL.view(-1, H).t().contiguous() @ dO.view(-1, H), report_bwd=None)
    return out


def exact(case, seed):
    inp = _inputs(case, seed)
    if case["op"] == "guard":
        B, M, N = case["batch"], case["rows"], case["cols"]
        rb, cb = case["block_rows"], case["block_cols"]
        C = inp["C"].double()
        wr = torch.arange(1, rb + 1, dtype=torch.float64, device="cuda").view(rb, 1)
        wc = torch.arange(1, cb + 1, dtype=torch.float64, device="cuda")
        V, H = C.view(B, M // rb, rb, N), C.view(B, M, N // cb, cb)
        return dict(C=C, col=torch.stack([V.sum(2), (V * wr).sum(2)], 2),
                    row=torch.stack([H.sum(3), (H * wc).sum(3)], 3), report=None)
    return _exact_layer(case, inp)
