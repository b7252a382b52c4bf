"""The forms of the prefill kernel (GPU): 64, 128 or 256 query rows per work
item on four or eight waves.

With 64 rows, and with 128 on eight waves, the waves split each key block's
keys and exchange the row maxima.  Every form of every head dimension and key
block is run with every softmax setup and Q/K format, causal and not, on
ragged tiles, and the kernel that each call launched is checked, so that a
rule that moves a shape elsewhere cannot leave a form without its test."""
import numpy as np
import pytest

import oracle as O
from helpers import ARB_TOL, check_parity, dev_bf16, dev_u8, gpu_dump, lse_arb_tol
from helpers_form import SETUPS, SIZES, form_of, forms, launched, launched_form, shape_for
from paper_2602_02071_amd import workloads as W

pytestmark = pytest.mark.gpu


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


def run(shape, block, label, setup="e2e", heads=None, step=7, own_scores=False, form=None):
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
    vt = dev_bf16(v)
    _, names = launched(lambda: baps.baps_attention_fwd_ex(qt, kt, vt, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, block,
                                                           **kn))
    want = form_of(shape, block, setup) if form is None else form
    assert launched_form(names) == (D, block) + want, (names, want)
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


EVERY = [(size, setup, causal, form) for size in SIZES for setup in SETUPS for causal in (True, False)
         for form in forms(size, setup, causal)]


@pytest.mark.parametrize("size,setup,causal,form", EVERY,
                         ids=["d%d-b%d-%s-%s-%dx%d" % (s + (t, "causal" if c else "full") + f) for s, t, c, f in EVERY])
def test_every_form(size, setup, causal, form):
    shape = shape_for(size, setup, causal, form)
    assert shape is not None, "no shape takes this form"
    run(shape, size[1], f"form {form} {setup}", setup, step=max(7, shape[3] // 40), own_scores=setup == "fp8", form=form)


@pytest.mark.parametrize("Sq,form", [(2048, (4, 2)), (2049, (8, 2)), (4096, (8, 2)), (4097, (8, 1))])
def test_limits_of_the_rule(Sq, form):
    run((1, 8, 8, Sq, 500, 128, False), 128, f"{form} at {Sq} positions", step=97, form=form)


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
    (128, 64, False, True, 150, 180, 300),
    (128, 64, True, True, 150, 180, 300),
    (64, 64, True, True, 150, 260, 333),
    (64, 128, True, True, 150, 172, 300),
    (64, 128, False, False, 100, 260, 333),      # one round of 128-row items, two of 256-row ones
    (128, 64, False, False, 100, 260, 333),
    (64, 128, False, False, 150, 300, 1100),     # half a second round of 256-row items
    (128, 64, True, False, 150, 300, 600),
]


@pytest.mark.parametrize("key", FOUR_WAVES, ids=lambda k: "-".join(map(str, k)))
def test_four_waves(key):
    D, block, fp8, causal, sq, h, sk = key
    run((1, h, h, sq, sk, D, causal), block, f"four waves {key}", "fp8" if fp8 else "e2e", own_scores=fp8, form=(4, 1))
