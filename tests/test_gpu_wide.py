"""The layer's unbatched products on wide tiles: ragged last tiles in both
directions, every checksum block size, whole and sliced K ranges, one launch
and paired launches, with a fault in the last row and column of each output."""
import pytest
import torch

pytestmark = pytest.mark.gpu

U = 2.0 ** -8       # bf16 rounding
EPS = 2.0 ** -24    # fp32 rounding


def _rows(shape, op, d, H, S, B):
    """Fault coordinates (b, h, row, col) of the last element of op's output."""
    nh = H // d
    if op in ("Q", "K", "V", "dCL"):
        return (B - 1, nh - 1, S - 1, d - 1)
    if op in ("O", "dX"):
        return (B - 1, 0, S - 1, H - 1)
    return (0, 0, H - 1, H - 1)


def _close(name, got, a, b):
    """got against the product a @ b of its stored operands: fp32 sums of K
    terms on both sides (K eps sum|terms| each), then one rounding of got."""
    ref, mag = a.float() @ b.float(), a.float().abs() @ b.float().abs()
    bound = 2 * a.shape[1] * EPS * mag
    if got.dtype == torch.bfloat16:
        bound += U * ref.abs() * (1 + U)
    bad = ((got.float() - ref).abs() > bound + 1e-30).sum().item()
    assert bad == 0, f"{name}: {bad} elements outside the bound"


# batch, seq, hidden, heads, R, fused. The first four reach 256 x 256 and 256
# x 192 tiles (each ragged), the last two 128 x 128 with R = 32 and with K in
# slices of uneven length.
SHAPES = [(1, 1408, 3200, 25, 128, True), (4, 1152, 2880, 45, 128, True),
          (4, 1088, 2816, 22, 64, False), (3, 1408, 2176, 17, 128, True),
          (5, 640, 1088, 17, 32, True), (3, 192, 320, 5, 64, False)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d-S%d-H%d-%dh-R%d-f%d" % s)
@pytest.mark.parametrize("protect", [True, False])
def test_wide_products(shape, protect):
    from paper_2410_11720_amd import abft
    B, S, H, nh, R, fused = shape
    d = H // nh
    cfg = abft.LayerConfig(B, S, H, nh, causal=True, block_rows=R, fused=fused, protect=protect)
    layer = abft.ProtectedAttention(cfg, capacity=256)
    gen = torch.Generator(device="cuda").manual_seed(7)

    def rand(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    X, W, Wo, dO = rand(B, S, H), rand(H, 3 * H, std=0.02), rand(H, H, std=0.02), rand(B, S, H)
    fwd, bwd = ("Q", "K", "V", "O"), ("dCL", "dWO", "dWQ", "dWV", "dX")
    faults = [(op, *_rows(shape, op, d, H, S, B), float("inf")) for op in fwd + bwd] if protect else []
    f = abft.faults_to_device(faults)
    O = layer.forward(X, W, Wo, f)
    dX, dW, dWo = layer.backward(dO, X, W, Wo, f)
    torch.cuda.synchronize()
    for rep, ops in ((layer.report, fwd), (layer.report_bwd, bwd)):
        r = abft.read_report(rep)
        want = [(op, *_rows(shape, op, d, H, S, B), "INF", "RECOMPUTE") for op in ops] if protect else []
        assert sorted(r["events"]) == sorted(want)
        assert r["n_uncorrectable"] == 0

    x2, g2 = X.view(-1, H), dO.view(-1, H)

    def check():
        qkv, cl = layer.tensor("QKV").view(-1, 3 * H), layer.tensor("CL").view(-1, H)
        dcl, dqkv = layer.tensor("dCL").view(-1, H), layer.tensor("dQKV").view(-1, 3 * H)
        _close("QKV", qkv, x2, W)
        _close("O", O.view(-1, H), cl, Wo)
        _close("dCL", dcl, g2, Wo.t().contiguous())
        _close("dWo", dWo, cl.t().contiguous(), g2)
        _close("dWqkv", dW, x2.t().contiguous(), dqkv)
        _close("dX", dX.view(-1, H), dqkv, W.t().contiguous())
    check()
    # the backward's products launched one by one
    for t in (dX, dW, dWo):
        t.fill_(float("nan"))
    for stage in ("dCL", "dWo", "dWqkv", "dX"):
        abft.attn_abft_backward_stages(cfg, dO, X, W, Wo, layer.workspace, dX, dW, dWo, None, 0,
                                       layer.report_bwd, abft.BWD_STAGES[stage])
        assert abft.read_report(layer.report_bwd)["n_events"] == 0
    check()


def test_wide_products_without_root_check():
    """Without the root check a located element is fixed from its checksums;
    two errors in one checksum vector are reported as uncorrectable."""
    from paper_2410_11720_amd import abft
    B, S, H, nh = 1, 1408, 3200, 25
    cfg = abft.LayerConfig(B, S, H, nh, causal=True, fused=True, root_check=False)
    layer = abft.ProtectedAttention(cfg, capacity=256)
    gen = torch.Generator(device="cuda").manual_seed(8)

    def rand(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    X, W, Wo, dO = rand(B, S, H), rand(H, 3 * H, std=0.02), rand(H, H, std=0.02), rand(B, S, H)
    clean = layer.forward(X, W, Wo).clone()
    f = abft.faults_to_device([("O", 0, 0, S - 1, 5, 3e4), ("O", 0, 0, 130, 6, float("nan")),
                               ("O", 0, 0, 3, 7, float("inf")), ("O", 0, 0, 9, 7, float("inf"))])
    O = layer.forward(X, W, Wo, f)
    ev = sorted(abft.read_report(layer.report)["events"])
    assert ev == sorted([("O", 0, 0, S - 1, 5, "NUMERIC", "DELTA"),
                         ("O", 0, 0, 130, 6, "NAN", "RECONSTRUCT"),
                         ("O", 0, 0, 0, 7, "-", "UNCORRECTABLE")])
    # rebuilt from a sum of 128 rounded values: half a step of each, and the
    # DELTA one to a step of the fault's own size (3e4 u)
    rms = clean.float().pow(2).mean().sqrt().item()
    assert abs(O[0, 130, 6].item() - clean[0, 130, 6].item()) <= 128 * U * 4 * rms
    assert abs(O[0, S - 1, 5].item() - clean[0, S - 1, 5].item()) <= 3e4 * U


# batch, seq, hidden, heads, R, dtype: fp32 tiles of 32, 64 and 128 columns,
# and softmax workgroups of 16, 8 and 4 waves (at most 256, 512 and more query
# blocks; R = 16 and 32 leave few rows for a wave); the last two have rows
# above 2048 keys and at least 384 query blocks (column sums added in turn)
@pytest.mark.parametrize("shape", [(2, 512, 512, 8, 128, "f32"), (1, 352, 128, 1, 32, "f32"),
                                   (1, 272, 192, 3, 16, "f32"), (4, 512, 1024, 8, 64, "f32"),
                                   (3, 864, 320, 5, 32, "bf16"), (2, 448, 128, 2, 64, "bf16"),
                                   (4, 512, 768, 12, 32, "bf16"), (1, 2176, 1536, 24, 128, "bf16"),
                                   (1, 2080, 384, 6, 32, "bf16")],
                         ids=lambda s: "B%d-S%d-H%d-%dh-R%d-%s" % s)
def test_materialised_stages(shape):
    """Products of fp32 operands, and the softmax with its checksums, each
    against the stored tensors it reads."""
    from paper_2410_11720_amd import abft
    B, S, H, nh, R, dtype = shape
    d = H // nh
    cfg = abft.LayerConfig(B, S, H, nh, dtype=dtype, causal=True, block_rows=R)
    layer = abft.ProtectedAttention(cfg, capacity=256)
    gen = torch.Generator(device="cuda").manual_seed(9)
    tdt = cfg.torch_dtype

    def rand(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device="cuda") * std).to(tdt)
    X, W, Wo, dO = rand(B, S, H), rand(H, 3 * H, std=0.02), rand(H, H, std=0.02), rand(B, S, H)
    last = [(op, B - 1, nh - 1, S - 1, d - 1) for op in ("V", "CL")] + [("AS", 0, 0, S - 1, S - 1)]
    f = abft.faults_to_device([t + (float("inf"),) for t in last])
    O = layer.forward(X, W, Wo, f)
    ev = abft.read_report(layer.report)["events"]
    assert sorted(ev) == sorted(t + ("INF", "RECOMPUTE") for t in last)
    AS, AP = layer.tensor("AS").double().clone(), layer.tensor("AP").double()
    APc, APr = layer.tensor("APc").double(), layer.tensor("APr").double()
    live = torch.ones(S, S, dtype=torch.bool, device="cuda").tril()
    ref = torch.softmax(AS.masked_fill(~live, float("-inf")) / d ** 0.5, -1)
    AP = torch.where(live, AP, torch.zeros_like(AP))  # masked pairs: unspecified past the tile
    # exp2 and the row sum in fp32: a few units of the argument's rounding
    tol = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -18
    assert ((AP - ref).abs() <= tol * ref + 1e-7).all()
    w = torch.arange(1, R + 1, device="cuda", dtype=torch.float64)
    blocks = AP.view(B, nh, S // R, R, S)
    eps = 2.0 ** -20 * R
    allowed = live.view(S // R, R, S).any(1)  # columns some query of the block may see
    for got, want in ((APc[..., 0, :], blocks.sum(3)), (APc[..., 1, :], (blocks * w.view(R, 1)).sum(3))):
        err = ((got - want).abs() - eps * (want.abs() + 1e-3))[:, :, allowed]
        assert (err <= 0).all()
    cols = AP.view(B, nh, S, S // R, R)
    reach = live.view(S, S // R, R).any(2)
    for got, want in ((APr[..., 0], cols.sum(4)), (APr[..., 1], (cols * w).sum(4))):
        err = ((got - want).abs() - eps * (want.abs() + 1e-3))[:, :, reach]
        assert (err <= 0).all()
    dX, dW, dWo = layer.backward(dO, X, W, Wo)
    assert abft.read_report(layer.report_bwd)["n_events"] == 0
    x2, g2 = X.view(-1, H), dO.view(-1, H)
    dcl, dqkv = layer.tensor("dCL").view(-1, H), layer.tensor("dQKV").view(-1, 3 * H)
    _close("QKV", layer.tensor("QKV").view(-1, 3 * H), x2, W)
    _close("O", O.view(-1, H), layer.tensor("CL").view(-1, H), Wo)
    _close("dCL", dcl, g2, Wo.t().contiguous())
    _close("dWo", dWo, layer.tensor("CL").view(-1, H).t().contiguous(), g2)
    _close("dWqkv", dW, x2.t().contiguous(), dqkv)
    _close("dX", dX.view(-1, H), dqkv, W.t().contiguous())
    # the batched products over the keys or queries, whose K ranges end in a
    # half stage where S % 64 = 32
    qkv, cl, dcl, dqkv = (layer.tensor(t) for t in ("QKV", "CL", "dCL", "dQKV"))
    for t, ap, das in zip(range(B * nh), AP.flatten(0, 1),
                          layer.tensor("dAS").flatten(0, 1).double()):
        b, h = t // nh, t % nh
        das = torch.where(live, das, torch.zeros_like(das))
        q, k, v = (qkv[b, :, i * H + h * d:i * H + (h + 1) * d] for i in range(3))
        g, c = (x[b, :, h * d:(h + 1) * d] for x in (dcl, cl))
        dq, dk, dv = (dqkv[b, :, i * H + h * d:i * H + (h + 1) * d] for i in range(3))
        _close("CL", c, ap, v)
        _close("dV", dv, ap.t().contiguous(), g)
        _close("dQ", dq, das, k)
        _close("dK", dk, das.t().contiguous(), q)
