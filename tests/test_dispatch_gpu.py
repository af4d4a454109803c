"""GPU parity at the edges of the launch rules: sizes where a call passes from
one kernel variant to another, each against the fp64 oracle."""

import numpy as np
import pytest

from tests.test_decode_gpu import cache_case, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,G,C", [("bf16", 128, 16, 8192), ("bf16", 128, 7, 7937), ("bf16", 64, 5, 7681),
                                         ("f32", 128, 4, 7680), ("bf16", 64, 4, 8200)])
def test_combine_many_records(dtype, d, G, C):
    """31 to 34 split-K records per head, around the record count from which
    the merge of a call without an append is dealt to several blocks; heads
    that fill all, some and one of the records, with and without residuals."""
    Hkv, Rcap = 3, 200
    res = [[0, 200, 3]]
    main = [[C, 700, C - 3]]
    shape, q, kc, vc, logc = cache_case(40 + G, 1, G * Hkv, Hkv, d, dtype, C, Rcap, res, main)
    check(dtype, shape, q, kc, vc, logc, res, main)
