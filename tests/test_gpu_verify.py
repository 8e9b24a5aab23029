"""verify_and_correct over slabs of columns: the chunked detection and the
one-vector-per-thread one, ragged last slabs, one and two sides, against the
oracle's verifier on the same faults."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.eec import Verifier, col_checksums, row_checksums
from oracle.numerics import stored_threshold

pytestmark = pytest.mark.gpu


# dtype, rows, cols, ld, block rows, block cols (0: columns only): slabs of 8
# and of 16 chunks, a ragged last slab, a matrix narrower than a slab, an
# unaligned leading dimension, a row block no lane group covers, whole rows
# where the row blocks fill the chip
CASES = [("bf16", 256, 320, 320, 128, 64), ("bf16", 128, 384, 384, 32, 128),
         ("bf16", 96, 200, 208, 32, 8), ("bf16", 64, 8, 8, 64, 8), ("bf16", 256, 200, 208, 128, 0),
         ("bf16", 128, 192, 193, 64, 64), ("bf16", 128, 576, 576, 64, 192),
         ("f32", 128, 160, 160, 64, 32), ("f32", 192, 128, 128, 64, 64), ("f32", 70, 90, 91, 7, 9),
         ("f32", 256, 384, 384, 128, 128), ("bf16", 96, 768, 768, 32, 256),
         ("bf16", 1204, 270, 271, 7, 9)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_verify_slabs(case):
    from paper_2410_11720_amd import abft
    dtype, rows, cols, ld, Rb, Cb = case
    batch, two = 3, Cb > 0
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    e_rel = 2.0 ** -13 if dtype == "f32" else 2.0 ** -4
    rng = np.random.default_rng(rows + cols)
    M = W.to_storage(rng.standard_normal((batch, rows, cols)).astype(np.float32), dtype).astype(np.float64)
    Cc = col_checksums(M, Rb)
    Cr = row_checksums(M, Cb) if two else None
    bad = M.copy()
    # a single error in the first and last slab, a column of two (1C, located
    # by the rows), a row of two (1R, located by the columns)
    hits = [(0, 0, 0, np.inf), (1, rows - 1, cols - 1, np.nan), (2, rows // 2, cols // 2, 1e10)]
    if two and Rb >= 7:
        hits += [(0, 1, cols - 1, np.inf), (0, 3, cols - 1, -1e10)]
        if Cb >= 8:
            hits += [(1, 2, 1, np.inf), (1, 2, 4, np.nan)]
    for b, r, c, v in hits:
        bad[b, r, c] = float(W.to_storage(np.float32([v]), dtype)[0]) if np.isfinite(v) else v
    full = np.zeros((batch, rows, ld))
    full[..., :cols] = bad
    C = torch.from_numpy(full).to("cuda", tdt)
    cc = torch.from_numpy(Cc).to("cuda", torch.float32).contiguous()
    rc = torch.from_numpy(Cr).to("cuda", torch.float32).contiguous() if two else None
    rep = abft.new_report(256)
    args = (abft.FP32 if dtype == "f32" else abft.BF16, batch, rows, cols, ld, rows * ld, Rb,
            Cb or 1, cc, rc, 1e10, 1e5, 0.0, abft.OP_ID["AS"], rep)
    abft.verify_and_correct(C, *args)
    got = abft.read_report(rep)
    ver = Verifier(dtype, e_rel, stored_threshold(1e10, dtype), 1e5)
    ref = bad.copy()
    evs, unc = ver.run(ref, Cc.copy(), Rb, Cr=Cr.copy() if two else None, Cb=Cb if two else None)
    want = [("AS", k, 0, i, j, kind, act) for (k, i, j, kind, act) in evs]
    corrected = [e for e in got["events"] if e[-1] != "UNCORRECTABLE"]
    assert sorted(corrected) == sorted(want)
    assert got["n_uncorrectable"] == len(unc)
    out = C.double().cpu().numpy()
    # rebuilt elements: c1 minus a sum of at most max(Rb, Cb) stored values in fp32
    tol = max(Rb, Cb) * 2.0 ** -22 * 8 + (2.0 ** -8 * 8 if dtype == "bf16" else 0.0)
    ok = np.isfinite(ref)
    assert np.array_equal(ok, np.isfinite(out[..., :cols]))
    assert np.max(np.abs(out[..., :cols] - ref)[ok]) <= tol
    assert np.all(out[..., cols:] == 0)  # the padding is not touched
    # what was corrected is clean
    if not unc:
        abft.attn_abft_report_init(rep, 256)
        abft.verify_and_correct(C, *args)
        assert abft.read_report(rep)["n_events"] == 0
