"""The rule that picks the prefill kernel's form (CPU only): shapes on both
sides of its lines, each with the form that measured faster there."""
import pytest

from helpers_code_object import READELF, kernel_resources
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
