"""What the compiled kernels take of a CU (CPU only: the notes of the code
objects in the built library).  A SIMD has 512 registers per lane and a CU
160 KiB of LDS: where the design has two workgroups of eight waves share a CU,
a kernel takes at most 128 registers."""
import os
import re

import pytest

from helpers_code_object import READELF, kernel_resources

pytestmark = pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")


def _prefill():
    """(D, block, waves, waves per row, code table, mode, tile, fp8, persistent, ties even, dump) -> resources"""
    out = {}
    for name, res in kernel_resources().items():
        m = re.search(r"baps_attn_fwd_kernel<([^>]*)>", name)
        if m:
            out[tuple(dict(true=True, false=False).get(x, x) if not x.isdigit() else int(x)
                      for x in m.group(1).split(", "))] = res
    return out


def test_two_prefill_workgroups_per_cu():
    """D = 64 with key blocks of up to 64: the eight-wave kernels of the library's calls (tile-level
    restart among them) fit a CU twice."""
    seen = 0
    for key, res in _prefill().items():
        D, block, nw, dump = key[0], key[1], key[2], key[-1]
        if D == 64 and block <= 64 and nw == 8 and not dump:
            seen += 1
            assert res["vgpr"] <= 128, (key, res)
            assert 2 * (res["lds"] + 4 * block * 2 * D) <= 160 << 10, (key, res)
    assert seen >= 10



def test_rows64_workgroups_fit_as_the_rule_counts():
    """prefill_form's LDS per 64-row workgroup is at least the kernel's, and says right how many (of up to three) fit."""
    for (D, block, nw, kw, ct, mode, tile, f8, persist, even, dump), res in _prefill().items():
        if (nw, kw) == (4, 2) and not dump:
            lds = res["lds"] + 4 * block * 2 * D
            counted = 8 * D * block + (16 if even or not ct else 8) * 1024 + 1024 + 256
            assert lds <= counted and min(3, (160 << 10) // lds) == min(3, (160 << 10) // counted), (D, block, ct, mode, even, lds)
