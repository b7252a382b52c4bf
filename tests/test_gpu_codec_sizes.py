"""HiF8 codec kernels at the edges of their grids (GPU): fewer elements than a
lane's group, a workgroup's chunk (4096 elements encoding, 2048 decoding) give
or take one, ragged tails, and nothing written past the end."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("even", [False, True])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 2047, 2048, 2049, 4095, 4096, 4097, 8193, 262147])
def test_codec_sizes(n, even):
    import torch
    import paper_2602_02071_amd as baps
    g = np.random.default_rng(n)
    x = (g.standard_normal(n) * np.exp2(g.integers(-26, 18, n))).astype(np.float32)
    x[::5] = np.float32(1.0625)                                # ties
    flags = baps.BAPS_HIF8_SATURATE | (baps.BAPS_HIF8_TIES_EVEN if even else 0)
    codes = torch.full((n + 16,), 0x5A, dtype=torch.uint8, device="cuda:0")
    y = torch.full((n + 16,), -7.0, dtype=torch.float32, device="cuda:0")
    baps.hif8_encode(torch.from_numpy(x).to("cuda:0"), codes, n, flags)
    baps.hif8_decode(codes, y, n)
    torch.cuda.synchronize()
    want = O.hif8_encode(x, ties_even=even)
    assert np.array_equal(codes[:n].cpu().numpy(), want)
    assert np.array_equal(y[:n].cpu().numpy().astype(np.float64), O.hif8_decode(want), equal_nan=True)
    assert bool((codes[n:] == 0x5A).all()) and bool((y[n:] == -7.0).all())
