"""The fused backward at head dim 128: its checks' bound, to the last fp32
bit, and the gradients of its unchecked forms."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

D, NH, S = 128, 2, 256


def _integers(seed):
    """Inputs whose projections, scores and checksums are integers that
    every step holds exactly: the checks then see an injected difference as
    it is, without a rounding of the operands."""
    H = NH * D
    rng = np.random.default_rng(seed)
    X = rng.integers(-1, 2, (1, S, H)) * (rng.random((1, S, H)) < 0.05)
    dO = rng.integers(-1, 2, (1, S, H)) * (rng.random((1, S, H)) < 0.05)
    W, Wo = rng.integers(-2, 3, (H, 3 * H)), rng.integers(-2, 3, (H, H))
    return X, W, Wo, dO


def _faults(op, scores, h, R, e_rel, rng, by_row):
    """One fault per vector of R scores in the last half of the queries, in
    turn the least difference the rule flags and the most that it passes."""
    out, want = [], []
    for n in range(24):
        i = int(rng.integers(S // 2, S))
        j = int(rng.integers(0, S // 2))
        if any((i // R, j) == (a // R, b) if not by_row else (i, j // R) == (a, b // R)
               for _, _, _, a, b, _ in out):
            continue
        s = scores[i, j]
        vec = scores[i // R * R:i // R * R + R, j] if not by_row else scores[i, j // R * R:j // R * R + R]
        rest = np.abs(vec).sum() - abs(s)
        sign = 1 if rng.random() < 0.5 else -1
        k = 1
        while k <= e_rel * (rest + abs(s + sign * k)):  # flagged: |d1| above E
            k += 1
        hit = n % 2 == 0
        out.append((op, 0, h, i, j, float(s + sign * (k if hit else k - 1))))
        if hit:
            want.append((op, 0, h, i, j, "NUMERIC", "RECOMPUTE"))
    assert len(want) >= 6
    return out, want


@pytest.mark.parametrize("R", [32, 64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("stage,ops", [("dQ", ("AS", "dAP")), ("dK", ("AS", "dAP"))])
def test_score_checks_sum_in_fp32(R, causal, stage, ops):
    """With e_rel = 2^-10 the rule's bound lies between two neighbouring
    integers; the differences on either side of it are told apart (sums of
    scores rounded to 16 bits, off by several of them, do not)."""
    from paper_2410_11720_amd import abft
    e_rel, H = 2.0 ** -10, NH * D
    X, W, Wo, dO = _integers(3)
    dev = [torch.from_numpy(a.astype(np.float32)).to("cuda", torch.bfloat16) for a in (X, W, Wo, dO)]
    kw = dict(causal=causal, block_rows=R, fused=True)
    layer = abft.ProtectedAttention(abft.LayerConfig(1, S, H, NH, **kw), capacity=512)
    layer.forward(*dev[:3])
    grads = layer.backward(dev[3], *dev[:3])
    QKV, dCL = (X[0] @ W), (dO[0] @ Wo.T)
    assert np.array_equal(layer.tensor("QKV")[0].double().cpu().numpy(), QKV)
    assert np.array_equal(layer.tensor("dCL")[0].double().cpu().numpy(), dCL)
    w = np.arange(1, R + 1)[:, None]
    assert all(np.abs((w * m[r:r + R]).sum(0)).max() < 2 ** 16 for m in (QKV, dCL)
               for r in range(0, S, R))  # held by the strips' hi/lo pairs
    strict = abft.LayerConfig(1, S, H, NH, e_rel=e_rel, **kw)
    for op in ops:
        for h in range(NH):
            q, k, v = (QKV[:, i * H + h * D:i * H + (h + 1) * D] for i in range(3))
            sc = q @ k.T if op == "AS" else dCL[:, h * D:(h + 1) * D] @ v.T
            faults, want = _faults(op, sc, h, R, e_rel, np.random.default_rng(R + h), stage == "dQ")
            f = abft.faults_to_device(faults)
            abft.attn_abft_backward_stages(strict, dev[3], *dev[:3], layer.workspace, *grads, *f,
                                           layer.report_bwd, abft.BWD_STAGES[stage])
            got = [e for e in abft.read_report(layer.report_bwd)["events"] if e[0] in ("AS", "dAP")]
            assert sorted(got) == sorted(want), (op, h)


@pytest.mark.parametrize("R", [32, 64, 128])
@pytest.mark.parametrize("causal", [True, False])
def test_gradients_of_every_form(R, causal):
    """dQ, dK and dV of the checked, the section-off and the unprotected
    form, each against fp64 products of the stored Q, K, V, CL and dCL:
    within 1e-2 in relative norm (P, dS and the gradients are rounded to
    bf16, 2^-9 each)."""
    from paper_2410_11720_amd import abft
    H = NH * D
    gen = torch.Generator(device="cuda").manual_seed(11)

    def rand(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    B, S3 = 2, 384
    X, W, Wo, dO = rand(B, S3, H), rand(H, 3 * H, std=0.05), rand(H, H, std=0.05), rand(B, S3, H)
    for opt in (dict(), dict(sections=0), dict(protect=False)):
        cfg = abft.LayerConfig(B, S3, H, NH, causal=causal, block_rows=R, fused=True, **opt)
        layer = abft.ProtectedAttention(cfg, capacity=64)
        layer.forward(X, W, Wo)
        layer.backward(dO, X, W, Wo)
        assert abft.read_report(layer.report_bwd)["n_events"] == 0
        qkv, cl, dcl, dqkv = (layer.tensor(t).double() for t in ("QKV", "CL", "dCL", "dQKV"))
        mask = torch.ones(S3, S3, dtype=torch.bool, device="cuda").triu(1) if causal else None
        for b in range(B):
            for h in range(NH):
                q, k, v = (qkv[b, :, i * H + h * D:i * H + (h + 1) * D].contiguous() for i in range(3))
                c, g = (x[b, :, h * D:(h + 1) * D].contiguous() for x in (cl, dcl))
                P = (q @ k.t().contiguous()) / D ** 0.5
                if causal:
                    P = P.masked_fill(mask, float("-inf"))
                P = torch.softmax(P, -1)
                dS = P * (g @ v.t().contiguous() - (c * g).sum(1, keepdim=True)) / D ** 0.5
                ref = (dS @ k, dS.t().contiguous() @ q, P.t().contiguous() @ g)
                for i, name in enumerate(("dQ", "dK", "dV")):
                    got = dqkv[b, :, i * H + h * D:i * H + (h + 1) * D]
                    err = ((got - ref[i]).norm() / ref[i].norm()).item()
                    assert err <= 1e-2, (opt, name, b, h, err)
