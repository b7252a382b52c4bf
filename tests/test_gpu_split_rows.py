"""The split-key path's workgroup shapes (GPU): one or two 16-row tiles per
workgroup, one, two, four or eight waves, block groups within a workgroup, one, two or
four rows per wave in the replay, and runs of dot products that end early.
Every T, P and reference equals the one-pass kernels': O and lse agree with
them to fp32 summation order, the restart counters exactly."""
import numpy as np
import pytest

from helpers import check_parity, dev_bf16, dev_u8, lse_agree
from helpers_form import launched
from paper_2602_02071_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, Hq, Hkv, Sq, Sk, D, causal, block; 16-row tiles and waves of a workgroup
    ((1, 2, 2, 17, 3001, 64, True, 64), (2, 8)),       # 17 rows: one in the second tile
    ((4, 32, 8, 8, 700, 128, True, 32), (2, 8)),       # 32 rows, three and four blocks per split, 8 block groups
    ((1, 6, 2, 11, 5000, 128, True, 128), (2, 8)),     # 33 rows: a workgroup of 32 rows and one of a single row
    ((2, 8, 2, 16, 2500, 64, False, 64), (2, 8)),      # 64 rows
    ((4, 64, 16, 8, 2560, 64, True, 32), (1, 4)),      # 20 blocks per split: 16 rows per workgroup although it has 32
    ((4, 32, 8, 4, 8192, 128, True, 128), (1, 4)),     # 16 rows, 512 workgroups
    ((2, 16, 4, 4, 20000, 64, True, 64), (1, 4)),      # 16 rows on 313 blocks: several windows of 64
    ((1, 8, 8, 6, 9000, 128, True, 32), (1, 4)),       # 6 rows: two per wave
    ((8, 8, 8, 1, 600, 128, False, 64), (1, 4)),       # one row, splits of two blocks
    ((10, 32, 8, 8, 2000, 128, True, 64), (2, 4)),     # 32 rows, more workgroups than CUs
    ((1, 16, 16, 1, 130, 128, True, 32), (1, 1)),      # one block per split, one row: a group of one wave
    ((1, 8, 2, 1, 1000, 64, True, 32), (1, 1)),        # four rows on that wave
    ((4, 8, 8, 2, 300, 64, True, 64), (1, 2)),         # two rows, a group of two waves
    ((1, 6, 2, 1, 650, 128, False, 64), (1, 2)),       # three rows
    ((1, 8, 1, 1, 5000, 64, True, 32), (1, 8)),        # eight rows, one block per split, 157 blocks to replay
    ((1, 16, 16, 1, 600, 64, True, 128), (1, 4)),      # one block per split, whose group has four waves
    ((1, 8, 2, 1, 1050, 64, True, 32), (1, 4)),        # four rows on 33 blocks: past what one wave replays well
    ((1, 4, 4, 1, 3000, 128, True, 32), (1, 1)),       # one row on 94 blocks: one wave again
    ((1, 4, 1, 1, 520, 64, True, 64), (1, 4)),         # four rows on 9 blocks of 64 at D = 64
]
IDS = ["x".join(map(str, s)) for s, _ in SHAPES]


def _inputs(shape, seed):
    B, Hq, Hkv, Sq, Sk, D = shape[:6]
    q, k, v = W.make_qkv(B, Hq, Hkv, Sq, Sk, D, seed=seed, lognormal_k=True)
    return q, k, v


def _pair(qt, kt, vt, shape, block, form=None, **kn):
    """(o, lse, counts) of the split path and of the one-pass kernels."""
    import torch
    import paper_2602_02071_amd as baps
    out = []
    for split in (True, False):
        cnt = torch.zeros((shape[0] * shape[1], 2), dtype=torch.int64, device="cuda:0")
        if split and form:
            (o, lse), names = launched(lambda: baps.attention(qt, kt, vt, shape[6], block, split=True,
                                                              restart_counts=cnt, **kn))
            assert sum("split_pv_kernel<%d, %d, %d, %d>" % ((shape[5], block) + form) in n for n in names) == 1, names
        else:
            o, lse = baps.attention(qt, kt, vt, shape[6], block, split=split, restart_counts=cnt, **kn)
        torch.cuda.synchronize()
        out.append((o.float().cpu().numpy().reshape(-1, shape[5]).astype(np.float64),
                    lse.cpu().numpy().reshape(-1).astype(np.float64), cnt.cpu().numpy()))
    return out


def _agree(pair, rel=2e-5):
    (o, lse, cnt), (o1, lse1, cnt1) = pair
    assert np.abs(o - o1).max() <= rel * max(1.0, np.abs(o1).max())
    assert lse_agree(lse, lse1)
    assert np.array_equal(cnt, cnt1)


@pytest.mark.parametrize("shape,form", SHAPES, ids=IDS)
def test_split_rows(shape, form):
    import paper_2602_02071_amd as baps
    print(f"split rows {shape}", flush=True)
    assert baps.baps_attention_split_workspace(*shape[:6], shape[7]) > 0
    q, k, v = _inputs(shape, sum(shape))
    pair = _pair(dev_bf16(q), dev_bf16(k), dev_bf16(v), shape, shape[7], form)
    _agree(pair)
    rows = np.arange(0, shape[0] * shape[1] * shape[3], 5)
    check_parity(q, k, v, shape[:7], shape[7], pair[0][0][rows], pair[0][1][rows], rows=rows,
                 label=f"split rows {shape}", same_kernels=False)


@pytest.mark.parametrize("shape", [s for s, _ in SHAPES[:4] + SHAPES[9:15]], ids=IDS[:4] + IDS[9:15])
def test_split_rows_knobs(shape):
    """FP8 Q/K, a diagonal B0 block, other thresholds, and bf16 O (one bf16 rounding of nearly equal values)."""
    q, k, v = _inputs(shape, 7)
    q8, k8, qs, ks = W.make_qk_fp8(q, k)
    _agree(_pair(dev_u8(q8), dev_u8(k8), dev_bf16(v), shape, shape[7], qk_scales=(qs, ks)))
    for kn in (dict(b0_last=True), dict(lam=0), dict(lam=8, n_b0=3), dict(lam=-2)):
        _agree(_pair(dev_bf16(q), dev_bf16(k), dev_bf16(v), shape, shape[7], **kn))
    _agree(_pair(dev_bf16(q), dev_bf16(k), dev_bf16(v), shape, shape[7], out_bf16=True), rel=2.0 ** -8)


@pytest.mark.parametrize("lam", [1, -2])
def test_split_replay_below_the_maximum(lam):
    """Steps of the replay whose blocks all lie below the maximum, with and without restarts there (lambda < 0),
    behind a first block that holds it; some of those steps end just above it."""
    shape = (1, 8, 2, 1, 40000, 64, False, 32)
    q, k, v = _inputs(shape, 23)
    k[:, :, :32] += np.uint16(2 << 7)             # bf16 bits: times 4
    k[:, :, 30000] += np.uint16(3 << 7)           # times 8
    _agree(_pair(dev_bf16(q), dev_bf16(k), dev_bf16(v), shape, shape[7], lam=lam))


@pytest.mark.parametrize("delta", [0.02, 0.9, 3.0])
def test_split_replay_of_a_climbing_maximum(delta):
    """Scores that climb by delta log2 units per block: small steps that the
    8-bit test rounds (the guess of the replay is off there), steps of about
    one, and a restart at every block."""
    shape = (1, 8, 2, 8, 6400, 64, False, 64)
    q, k, v = W.make_slow_climb(*shape[:6], delta=delta, block=shape[7], seed=int(100 * delta))
    _agree(_pair(dev_bf16(q), dev_bf16(k), dev_bf16(v), shape, shape[7]))
