"""Host-side checks of the dispatch rules (no GPU needed), at sizes on both sides
of each line, against the kernel that was measured the faster one there."""
import os

import pytest

from paper_2606_29094_amd import dlm

pytestmark = pytest.mark.skipif(not os.path.exists(dlm.LIB_PATH), reason="libdlm.so not built")

SHARED, SHARED4, HEAD32X4, HEAD64X2, HEAD32X2 = range(5)
GQA, MHA = (28, 4, 128), (32, 32, 128)


# heads, (requests, rows of each, keys of each), kernel, key splits
ATTENTION = [
    # grouped queries of at most 32 rows fill shared-tile blocks at any batch
    (GQA, (20, 32, 1280), SHARED, 1), (GQA, (32, 32, 1280), SHARED, 1),
    (GQA, (48, 16, 320), SHARED, 1), (GQA, (64, 16, 1280), SHARED, 1),
    ((32, 8, 128), (24, 32, 1280), SHARED, 1), ((32, 16, 128), (10, 16, 320), SHARED, 1),
    # key splits: equal ranges that make at most a block per CU
    (GQA, (3, 64, 1024), SHARED, 4), (GQA, (8, 48, 1280), SHARED, 2),
    (GQA, (1, 64, 900), SHARED, 8), (MHA, (1, 32, 517), SHARED, 5),
    (MHA, (3, 16, 2304), SHARED, 3), (MHA, (4, 32, 1280), SHARED, 2),
    # multi-head, at most 32 rows: short sequences; one, two, more rounds of per-head blocks
    (MHA, (8, 32, 640), SHARED, 1), (MHA, (8, 32, 1280), HEAD32X4, 1),
    (MHA, (9, 32, 1280), SHARED, 1), (MHA, (12, 32, 1280), SHARED, 1),
    (MHA, (15, 16, 2400), SHARED, 1), (MHA, (16, 32, 1280), SHARED, 1),
    (MHA, (17, 32, 1280), HEAD32X4, 1),
    # head_dim 64
    ((32, 32, 64), (8, 32, 320), SHARED, 1), ((32, 32, 64), (12, 32, 700), HEAD32X2, 1),
    ((32, 32, 64), (20, 32, 1280), HEAD32X2, 1), ((32, 32, 64), (8, 32, 2304), HEAD32X4, 1),
    ((32, 32, 64), (1, 32, 2304), SHARED, 8), ((32, 32, 64), (20, 64, 1280), SHARED4, 1),
    ((32, 32, 64), (16, 64, 1280), SHARED, 1), ((32, 32, 64), (2, 200, 1280), HEAD64X2, 1),
    ((32, 8, 64), (24, 32, 1280), SHARED, 1),
    # more rows: one to five key tiles, then one round of per-head blocks, then shared tiles
    (MHA, (1, 64, 64), SHARED, 1), (MHA, (4, 64, 320), SHARED, 1), (MHA, (1, 128, 128), HEAD64X2, 1),
    (MHA, (1, 160, 160), SHARED, 1), (MHA, (1, 200, 200), HEAD64X2, 1),
    (MHA, (1, 256, 256), HEAD32X4, 1), (MHA, (1, 512, 512), HEAD64X2, 1),
    (MHA, (1, 513, 513), SHARED, 1), (MHA, (1, 1024, 1024), SHARED, 1),
    (GQA, (1, 512, 512), HEAD64X2, 1), (GQA, (1, 600, 600), SHARED, 1),
    (GQA, (16, 64, 1024), SHARED, 1), ((8, 8, 128), (2, 1024, 1024), HEAD64X2, 1),
]


@pytest.mark.parametrize("heads,batch,kernel,splits", ATTENTION)
def test_attention_plan(heads, batch, kernel, splits):
    n, rows, keys = batch
    got = dlm.debug_attention_plan(*heads, [rows] * n, [keys] * n, 1 << 30)
    assert got == (kernel, splits)


def test_attention_plan_stays_within_the_scratch():
    hq, hkv, dh = GQA
    one = 64 * hq * (dh + 2) * 4                       # one split's partials of 64 rows
    for room in range(10):
        kernel, splits = dlm.debug_attention_plan(hq, hkv, dh, [64], [2304], room * one + room)
        assert splits <= max(room, 1) and (splits == 1 or kernel == SHARED)
    assert dlm.debug_attention_plan(hq, hkv, dh, [64], [2304], 8 * one)[1] > 4


def test_attention_plan_of_a_smaller_chip():
    # the lines are multiples of the CUs: half of them, half the requests
    for n in (4, 5, 8, 9):
        assert dlm.debug_attention_plan(*MHA, [32] * n, [1280] * n, 0, 128) == \
            dlm.debug_attention_plan(*MHA, [32] * 2 * n, [1280] * 2 * n, 0, 256)
