"""The rule that picks the prefill kernel's form (CPU only): shapes on both
sides of its lines, each with the form that measured faster there."""
import pytest

from helpers_form import SETUPS, SIZES, form_of, forms

ROWS64, ROWS128, ROWS256, FOUR = (4, 2), (8, 2), (8, 1), (4, 1)


def _form(heads, Sq, Sk, D, block, causal, setup="e2e", group=1):
    return form_of((1, heads * group, heads, Sq, Sk, D, causal), block, setup)


# ties to even and lambda > 8 hold 16 KiB of table: two 64-row workgroups do not share a CU at D * block = 8192
@pytest.mark.parametrize("heads,Sq,Sk,D,block,causal,setup,want", [
    (80, 256, 256, 64, 128, False, "even", ROWS256),
    (200, 70, 70, 128, 64, True, "even", ROWS256),
    (24, 700, 700, 128, 64, True, "even", ROWS64),
    (64, 256, 256, 64, 128, False, "even", ROWS64),
    (150, 70, 70, 64, 128, False, "lambda9", ROWS256),
    (37, 500, 500, 64, 128, False, "lambda9", ROWS256),
    (128, 256, 256, 128, 64, False, "lambda9", ROWS256),
    (8, 3000, 3000, 64, 128, True, "lambda9", ROWS64),
    (170, 230, 230, 64, 64, False, "lambda9", ROWS256),
    (100, 70, 70, 128, 128, True, "lambda9", ROWS256),
    (16, 1024, 1024, 64, 64, False, "lambda9", ROWS64),
    (80, 256, 256, 64, 128, False, "e2e", ROWS64),
])
def test_larger_tables(heads, Sq, Sk, D, block, causal, setup, want):
    assert _form(heads, Sq, Sk, D, block, causal, setup) == want


# one 256-row item per head on more than half of the CUs reads K/V once
@pytest.mark.parametrize("heads,Sq,Sk,D,block,causal,setup,want", [
    (256, 128, 5000, 64, 128, False, "e2e", ROWS256),
    (256, 70, 1500, 128, 64, True, "fp8", ROWS256),
    (200, 128, 500, 128, 128, True, "e2e", ROWS256),
    (200, 100, 100, 64, 64, False, "default", ROWS256),
    (170, 150, 150, 128, 64, False, "exp2", ROWS256),
    (256, 128, 300, 64, 128, True, "fp8", ROWS256),
    (133, 150, 150, 64, 128, True, "e2e", ROWS64),
    (170, 150, 150, 64, 128, False, "fp8", ROWS64),
    (128, 197, 197, 64, 128, False, "e2e", ROWS64),
    (200, 128, 1500, 128, 128, False, "even", ROWS128),
    (200, 197, 197, 64, 128, True, "fp8", FOUR),
])
def test_one_item_per_head(heads, Sq, Sk, D, block, causal, setup, want):
    assert _form(heads, Sq, Sk, D, block, causal, setup) == want


# a third 64-row workgroup per CU at D = 64, block 64
@pytest.mark.parametrize("heads,Sq,Sk,causal,setup,want", [
    (192, 197, 197, False, "e2e", ROWS256),
    (170, 256, 256, False, "default", ROWS256),
    (85, 500, 500, False, "e2e", ROWS256),
    (109, 400, 400, False, "exp2", ROWS256),
    (65, 512, 6000, True, "e2e", ROWS256),
    (260, 128, 4000, True, "e2e", ROWS256),
    (256, 150, 150, True, "e2e", ROWS256),
    (192, 197, 197, True, "e2e", ROWS64),
    (144, 257, 257, False, "e2e", ROWS64),
    (12, 4096, 4096, False, "e2e", ROWS64),
    (8, 6000, 7500, True, "e2e", ROWS64),
    (340, 70, 70, True, "default", ROWS64),
])
def test_third_workgroup(heads, Sq, Sk, causal, setup, want):
    assert _form(heads, Sq, Sk, 64, 64, causal, setup) == want


# 128 rows on four waves at D * block = 8192 (FP8 at 4096 too): where the longest causal item sets the time, heads
# of few items, padded tiles; not where the 256-row items pair up and fill the GPU
@pytest.mark.parametrize("heads,group,Sq,Sk,D,block,causal,setup,want", [
    (8, 4, 4096, 4096, 128, 64, True, "e2e", ROWS256),
    (8, 4, 2000, 6000, 128, 64, True, "fp8", ROWS256),
    (8, 4, 3500, 9000, 128, 64, True, "fp8", ROWS256),
    (16, 1, 4096, 4096, 128, 64, True, "e2e", FOUR),
    (32, 1, 4096, 4096, 64, 128, True, "fp8", ROWS256),
    (64, 1, 4096, 4096, 128, 64, True, "fp8", ROWS256),
    (48, 1, 2048, 2048, 64, 128, True, "e2e", ROWS256),
    (16, 1, 4096, 4096, 64, 128, True, "fp8", FOUR),
    (96, 1, 1369, 1369, 128, 64, True, "e2e", FOUR),
    (184, 1, 512, 512, 128, 64, True, "fp8", FOUR),
    (96, 1, 577, 577, 64, 128, True, "e2e", FOUR),
    (16, 1, 4096, 4096, 64, 64, True, "fp8", FOUR),
    (64, 4, 2048, 3048, 64, 64, True, "fp8", ROWS256),
    (96, 1, 577, 577, 128, 64, False, "e2e", FOUR),
    (32, 1, 4096, 4096, 128, 64, False, "e2e", ROWS256),
    (16, 1, 4096, 4096, 128, 64, True, "exp2", ROWS256),
])
def test_four_waves(heads, group, Sq, Sk, D, block, causal, setup, want):
    assert _form(heads, Sq, Sk, D, block, causal, setup, group) == want


def test_only_forms_that_are_built():
    """Every form that the rule can return is one that the library builds (over a grid of shapes)."""
    for size in SIZES:
        for setup in SETUPS:
            for causal in (True, False):
                for heads in (1, 3, 8, 24, 64, 130, 200, 400, 1100):
                    for Sq in (1, 65, 130, 200, 500, 1369, 4096):
                        for Sk in (0, 1, 64, 500, 5000):
                            f = _form(heads, Sq, Sk, *size, causal, setup)
                            assert f in forms(size, setup, causal), (size, setup, causal, heads, Sq, Sk, f)
