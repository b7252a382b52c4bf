"""The forms of the softmax-block kernel (GPU): the wide one (a workgroup per
row, chunks of 4096 columns) at the edges of its chunks and blocks, aligned
and not, and the row-group and row-per-wave forms that the rule still picks.
Codes, shifts, maxima and flags are bit-exact against the oracle, d within
fp32 summation order (1e-5)."""
import numpy as np
import pytest

import oracle as O
from paper_2602_02071_amd.workloads import random_scores
from helpers_form import launched
from test_gpu_softmax_block import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [64, 128, 256, 512, 1024])
@pytest.mark.parametrize("cols", [4, 60, 1024, 4092, 4096, 4100, 8192, 8196, 12292])
def test_wide_aligned(cols, block):
    print(f"wide {cols} block {block}", flush=True)
    _compare(random_scores(9, cols, seed=cols + block, std=5.0, masked_frac=0.02), block, ld=cols + 8)


@pytest.mark.parametrize("block", [64, 128, 256, 512, 1024])
@pytest.mark.parametrize("cols", [513, 1999, 4095, 4097, 8191, 12289])
def test_wide_unaligned(cols, block):
    _compare(random_scores(7, cols, seed=cols + block, std=5.0, masked_frac=0.02), block)


@pytest.mark.parametrize("lam,n_b0", [(0, 0), (2, 3), (-3, 1), (50, 2), (1, 200)])
def test_wide_knobs_on_climbing_rows(lam, n_b0):
    """Rows whose maximum moves at nearly every block (by small steps, about
    one, and many at once), where the wide form's guess is often off; masked
    rows and a masked start among them."""
    rows, cols = 12, 9000
    s = random_scores(rows, cols, seed=lam + 7, std=0.3)
    s += (np.linspace(0, 1, cols, dtype=np.float32)[None, :] *
          np.array([0, 1, 3, 8, 20, 60, 120, 250, 600, -50, -300, 5], np.float32)[:, None])
    s[3, :5000] = -np.inf
    s[11] = -np.inf
    for block in (64, 256):
        _compare(s, block, lam, n_b0)
        _compare(s[:, :8999], block, lam, n_b0)


@pytest.mark.parametrize("rows,cols,block,kernel", [
    (1500, 4096, 128, "block_wide_kernel<128, true>"),           # several rows per workgroup
    (3000, 300, 64, "block4_kernel<64, 256, 1024>"),       # row groups, 256 threads, wide steps
    (9000, 200, 128, "block4_kernel<128, 256, 256>"),      # row groups, 256 threads
    (16500, 132, 256, "block4_kernel<256, 1024, 256>"),    # row groups, 1024 threads
    (16500, 4100, 256, "block4_kernel<256, 1024, 512>"),   # the same, rows just behind a chunk of the wide form
    (1030, 700, 512, "block_kernel<512>"),                 # a row per wave, aligned rows and a wide block
    (1100, 515, 128, "block_kernel<128>"),                 # a row per wave, unaligned
    (3, 70000, 64, "block4_kernel<64, 256, 1024>"),        # more blocks than the wide form holds
])
def test_every_form(rows, cols, block, kernel):
    s = random_scores(rows, cols, seed=rows, std=4.0, masked_frac=0.01)
    _, names = launched(lambda: _compare(s, block))
    assert len(names) == 1 and "softmax_" + kernel in names[0], names


@pytest.mark.parametrize("rows,cols,block,wide", [
    (16384, 4100, 64, False), (16384, 4100, 256, False), (32768, 4500, 128, False), (4096, 4100, 1024, False),
    (3000, 4100, 512, False), (8192, 4100, 256, False), (4096, 2048, 256, False), (16384, 3000, 256, False),
    (8192, 4100, 64, True), (16384, 8196, 128, True), (16384, 4096, 256, True), (16384, 5200, 64, True),
    (2048, 4100, 1024, True), (2048, 1024, 256, True), (16384, 3000, 128, True),
])
def test_lines_of_the_wide_form(rows, cols, block, wide):
    """Rows that end just behind a chunk, and the other lines of the rule, by the kernel that runs."""
    import torch
    import paper_2602_02071_amd as baps
    nblk = -(-cols // block)
    s = torch.zeros((rows, cols), device="cuda:0")
    codes = torch.empty((rows, cols), dtype=torch.uint8, device="cuda:0")
    shift = torch.empty((rows, nblk), dtype=torch.int32, device="cuda:0")
    m, d = torch.empty(rows, device="cuda:0"), torch.empty(rows, device="cuda:0")
    _, names = launched(lambda: baps.baps_softmax_block(s, rows, cols, cols, block, 1, 1, 0, codes, shift, m, d))
    assert len(names) == 1 and ("wide" in names[0]) == wide, names


def test_wide_rows_that_climb_take_no_settling_one_by_one():
    """Scores that climb by 6 log2 units per block at lambda 8, where the 8-bit cast rounds every few blocks'
    T down to an integer: at most 1.6 times the time of level scores (settled block by block it was 2.6 times)."""
    import torch
    import paper_2602_02071_amd as baps
    rows, cols, block, lam = 16384, 8192, 64, 8
    level = torch.randn((rows, cols), device="cuda:0") * 0.05
    climb = level + 6.2 * (torch.arange(cols, device="cuda:0") // block)
    nblk = cols // block
    codes = torch.empty((rows, cols), dtype=torch.uint8, device="cuda:0")
    shift = torch.empty((rows, nblk), dtype=torch.int32, device="cuda:0")
    m, d = torch.empty(rows, device="cuda:0"), torch.empty(rows, device="cuda:0")

    def fastest(s):
        best = float("inf")
        for _ in range(12):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            baps.baps_softmax_block(s, rows, cols, cols, block, lam, 1, 0, codes, shift, m, d)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    t_level, t_climb = fastest(level), fastest(climb)
    print(f"level {t_level * 1e3:.0f} us, climbing {t_climb * 1e3:.0f} us", flush=True)
    assert t_climb <= 1.6 * t_level


@pytest.mark.parametrize("lam,step", [(1, 0.3), (8, 0.3), (1, 1.03), (1, 1.6), (2, 2.1), (4, 3.1), (8, 6.2), (50, 41.0)])
def test_wide_rows_that_climb(lam, step):
    """Several blocks of a chunk whose T the 8-bit cast rounds down to an integer, more chunks than one and a last
    one that is short; at lambda 50 the cast rounds by up to 4."""
    s = random_scores(6, 9000, seed=lam, std=0.05)
    s += np.float32(step) * (np.arange(9000) // 64).astype(np.float32)
    for block in (64, 128):
        _compare(s, block, lam)
        _compare(s[:, :8999], block, lam)
