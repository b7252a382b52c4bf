"""The rows per work item of the prefill kernel (GPU).

The library gives a work item 64, 128 or 256 query rows by how many items
that leaves; with 64 and 128 rows the waves split each key block's keys and
exchange the row maxima.  Every row count is run with every softmax setup and
Q/K format, on ragged tiles (150 query positions: the last tile holds 22 rows
of 64 or 128) and on shapes right at the two limits of the rule."""
import numpy as np
import pytest

import oracle as O
from helpers import ARB_TOL, check_parity, dev_bf16, dev_u8, gpu_dump, lse_arb_tol
from paper_2602_02071_amd import workloads as W

pytestmark = pytest.mark.gpu

CUS = 256
# (D, block, rows per item) -> heads of 150 positions that land there (3 items of 64 rows, 2 of 128, 1 of 256)
HEADS = {(128, 128, 64): 5, (128, 128, 128): 100, (128, 128, 256): 130, (128, 64, 64): 6, (128, 64, 256): 172,
         (64, 64, 64): 7, (64, 64, 256): 260, (64, 128, 64): 5, (64, 128, 256): 172}
SETUPS = ("e2e", "default", "exp2", "even", "fp8", "lambda9")


def on_own_scores(q, k, v, shape, block, rows, o, lse, fp8, **okw):
    """O and lse against the oracle run on the kernel's own dot products alone:
    bit-exact references, O within ARB_TOL.  The FP8 matrix instructions keep
    about 12 bits below the largest product of a step, so no fp32 bound says
    how far their scores lie from exact ones, and short causal rows average
    less of it: the canonical bar of 2e-3 is not a bound for them."""
    B, Hq, Hkv, Sq, Sk, D, causal = shape
    od, ld, acc, gref = gpu_dump(q, k, v, shape, block, rows, fp8=fp8, **okw)
    assert np.array_equal(od, o) and np.array_equal(ld, lse)
    res = O.attention(q, k, v, B, Hq, Hkv, Sq, Sk, D, causal, block, rows=rows,
                      acc=np.where(np.isfinite(acc), acc, 0).astype(np.float32), refs=True, **okw)
    assert np.array_equal(res[-1], gref, equal_nan=True)
    assert np.abs(o - res[0]).max() <= ARB_TOL
    assert np.all(np.abs(lse - res[1]) <= lse_arb_tol(res[1], np.isfinite(acc).sum(axis=1)))


def run(shape, block, label, setup="e2e", heads=None, step=7, own_scores=False):
    import torch
    import paper_2602_02071_amd as baps
    B, Hq, Hkv, Sq, Sk, D, causal = shape
    q, k, v = W.make_qkv(B, Hq, Hkv, Sq, Sk, D, seed=Sq + Hq + D)
    kn, okw, fp8 = {}, {}, None
    qt, kt = dev_bf16(q), dev_bf16(k)
    if setup == "default":
        kn, okw = dict(mode=baps.BAPS_MODE_DEFAULT), dict(mode=O.DEFAULT, pv_bf16=True)
    elif setup == "exp2":
        kn, okw = dict(mode=baps.BAPS_MODE_EXP2_HIF8), dict(mode=O.EXP2_HIF8)
    elif setup == "even":
        kn, okw = dict(tie_mode=baps.BAPS_TIES_EVEN), dict(tie_even=True)
    elif setup == "lambda9":
        kn, okw = dict(lam=9), dict(lam=9)
    elif setup == "fp8":
        fp8 = W.make_qk_fp8(q, k)
        q8, k8, qs, ks = fp8
        qt, kt = dev_u8(q8), dev_u8(k8)
        kn = dict(qk_scales=(qs, ks))
        q, k = O.e4m3_to_bf16(q8), O.e4m3_to_bf16(k8)
        okw = dict(scale_log2=O.fp8_scale_log2(D, qs, ks))
    o = torch.full((B, Hq, Sq, D), float("nan"), dtype=torch.float32, device="cuda:0")
    lse = torch.full((B, Hq, Sq), float("nan"), dtype=torch.float32, device="cuda:0")
    print(f"{label}: {shape} block {block}", flush=True)
    baps.baps_attention_fwd_ex(qt, kt, dev_bf16(v), o, lse, B, Hq, Hkv, Sq, Sk, D, causal, block, **kn)
    torch.cuda.synchronize()
    assert not torch.isnan(o).any() and not torch.isnan(lse).any(), "rows never written"
    heads = sorted({0, Hq // 2, Hq - 1}) if heads is None else heads
    pos = np.array(sorted(set(range(0, Sq, step)) | {min(63, Sq - 1), min(64, Sq - 1), min(127, Sq - 1), Sq - 1}))
    rows = np.concatenate([(b * Hq + h) * Sq + pos for b in range(B) for h in heads])
    o, lse = (x.cpu().numpy().astype(np.float64) for x in (o, lse))
    o, lse = o.reshape(-1, D)[rows], lse.reshape(-1)[rows]
    if own_scores:
        on_own_scores(q, k, v, shape, block, rows, o, lse, fp8, **okw)
    else:
        check_parity(q, k, v, shape, block, o, lse, rows=rows, label=label, fp8=fp8, **okw)


@pytest.mark.parametrize("setup", SETUPS)
@pytest.mark.parametrize("key", sorted(HEADS), ids=lambda k: "d%d-b%d-rows%d" % k)
def test_every_row_count(key, setup):
    D, block, rows = key
    h = HEADS[key]
    per_cu = {4096: 3, 8192: 2, 16384: 1}[D * block]
    want = 64 if 3 * h <= per_cu * CUS else (128 if per_cu == 1 and 2 * h <= CUS else 256)
    assert want == rows                                      # the shape lands where it is meant to
    run((1, h, h, 150, 333, D, setup != "exp2"), block, f"rows {rows} {setup}", setup)


@pytest.mark.parametrize("Sq,rows", [(2048, 64), (2049, 128), (4096, 128), (4097, 256)])
def test_limits_of_the_rule(Sq, rows):
    run((1, 8, 8, Sq, 500, 128, False), 128, f"{rows} rows at {Sq} positions", step=97)


def test_queries_before_the_first_key():
    """Sq > Sk under the causal mask: whole 64-row items see no key (O = 0, lse = -inf), others a few."""
    import torch
    import paper_2602_02071_amd as baps
    B, Hq, Hkv, Sq, Sk, D = 1, 6, 2, 200, 70, 128
    q, k, v = W.make_qkv(B, Hq, Hkv, Sq, Sk, D, seed=3)
    for block in (64, 128):
        o, lse = baps.attention(dev_bf16(q), dev_bf16(k), dev_bf16(v), True, block)
        torch.cuda.synchronize()
        rows = np.arange(0, Hq * Sq, 3)
        check_parity(q, k, v, (B, Hq, Hkv, Sq, Sk, D, True), block, o.cpu().numpy().reshape(-1, D)[rows].astype(np.float64),
                     lse.cpu().numpy().reshape(-1)[rows].astype(np.float64), rows=rows, label="queries before keys")


FOUR_WAVES = [
    # D, block, FP8, causal, positions, heads, keys: 128-row items on four waves
    (128, 64, False, True, 150, 180, 333),
    (128, 64, True, True, 150, 180, 333),
    (64, 64, True, True, 150, 260, 333),
    (64, 128, True, True, 150, 172, 333),
    (64, 128, False, False, 100, 260, 333),      # one round of 128-row items, two of 256-row ones
    (128, 64, False, False, 100, 260, 333),
    (64, 128, False, False, 150, 300, 1100),     # half a second round of 256-row items
    (128, 64, True, False, 150, 300, 600),
]


@pytest.mark.parametrize("key", FOUR_WAVES, ids=lambda k: "-".join(map(str, k)))
def test_four_waves(key):
    D, block, fp8, causal, sq, h, sk = key
    n4, n8 = -(-sq // 128) * h, -(-sq // 256) * h
    assert -(-sq // 64) * h > {4096: 3, 8192: 2}[D * block] * CUS and n8 <= 4 * CUS      # not the 64-row items
    assert causal or -(-n8 // CUS) > -(-n4 // (2 * CUS)) or (CUS < n8 <= 1.5 * CUS and sk >= 8 * block)
    run((1, h, h, sq, sk, D, causal), block, f"four waves {key}", "fp8" if fp8 else "e2e", own_scores=fp8)
