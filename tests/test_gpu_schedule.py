"""The prefill kernel's work schedule (GPU).

With D = 128 the kernels of one wave per 32 rows run a persistent grid: at most
one workgroup per resident slot, each taking a sequence of (query tile,
key/value head, batch) items.  These shapes have more items than the GPU holds at once, (batch, key/
value head) counts that are and are not multiples of 8, and ragged last
tiles.  O and lse start as NaN, so an item that is skipped (or a row written
by no item) shows; sampled rows, including the last row of every ragged
tile, are compared with the oracle to the usual bar."""
import numpy as np
import pytest

from helpers import check_parity, dev_bf16
from helpers_form import launched, launched_form
from paper_2602_02071_amd.workloads import make_qkv

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, Hq, Hkv, Sq, Sk, D, causal, block and waves: items = ceil(Sq*G/rows) * B*Hkv, 32 rows per wave
    (3, 6, 3, 5000, 5000, 128, True, 128, 8),  # 9 heads, 40 tiles each (last one 16 rows): 360 items
    (2, 8, 4, 4500, 2100, 128, False, 64, 4),  # 8 heads, 71 tiles of 128 rows each (last one 40): 568 items, two
                                               # workgroups per CU
    (2, 8, 4, 7000, 900, 128, False, 64, 8),   # 8 heads, 55 tiles each (last one 176 rows): 440 items
    (8, 32, 8, 1050, 1050, 128, True, 64, 8),  # 64 heads, 17 tiles each (last one 104 rows): 1088 items
    (1, 40, 8, 3000, 3000, 128, True, 32, 8),  # 8 heads, G = 5 (a tile splits query positions): 472 items
    (1, 32, 8, 4096, 4096, 128, True, 128, 8), # the Llama-3-8B prefill: 512 items, two per workgroup
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_persistent_schedule(shape):
    import torch
    import paper_2602_02071_amd as baps
    B, Hq, Hkv, Sq, Sk, D, causal, block, nw = shape
    G, rows = Hq // Hkv, 32 * nw
    q, k, v = make_qkv(B, Hq, Hkv, Sq, Sk, D, seed=sum(shape[:8]), outliers=True)
    o = torch.full((B, Hq, Sq, D), float("nan"), dtype=torch.float32, device="cuda:0")
    lse = torch.full((B, Hq, Sq), float("nan"), dtype=torch.float32, device="cuda:0")
    cnt = torch.zeros((B * Hq, 2), dtype=torch.int64, device="cuda:0")
    items = -(-Sq * G // rows) * B * Hkv
    print(f"persistent schedule {shape}: {items} items", flush=True)
    assert items > 256 * (8 // nw)                          # more than one round
    qt, kt, vt = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    _, names = launched(lambda: baps.baps_attention_fwd_ex(qt, kt, vt, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, block,
                                                           restart_counts=cnt))
    assert launched_form(names) == (D, block, nw, 1)
    assert not torch.isnan(o).any(), "rows never written"
    assert not torch.isnan(lse).any(), "lse never written"
    # every (row, key block after the first) that a row sees is visited once:
    # an item run twice (or skipped) moves its heads' totals
    r = np.arange(Sq)
    kmax = np.minimum(Sk - 1, r + Sk - Sq) if causal else np.full(Sq, Sk - 1)
    want = int((np.clip(kmax, 0, None) // block).sum())
    assert np.all(cnt[:, 1].cpu().numpy() == want), (cnt[:, 1].cpu().numpy(), want)
    o = o.cpu().numpy().reshape(-1, D).astype(np.float64)
    lse = lse.cpu().numpy().reshape(-1).astype(np.float64)
    # per (batch, head): a few positions, plus the positions of the last
    # flattened row of every tile and the last query position
    last_of_tile = {min(Sq - 1, (t * rows + rows - 1) // G) for t in range(-(-Sq * G // rows))}
    pos = np.array(sorted(set(range(0, Sq, 997)) | last_of_tile | {Sq - 1}), np.int64)
    heads = range(0, Hq, max(1, Hq // 5))
    sel = np.concatenate([(b * Hq + h) * Sq + pos for b in range(B) for h in heads])
    check_parity(q, k, v, (B, Hq, Hkv, Sq, Sk, D, causal), block, o[sel], lse[sel], rows=sel,
                 label=f"persistent {shape}")
