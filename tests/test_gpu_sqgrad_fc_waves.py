"""The FC statistic either side of the rules by which rows of any length go through LDS or a wave at a time: 511 and 512 tiles of
64 x 64, 32 and 33 rows, batches of 63 and 64, and 8 and 9 rows of bfloat16; and beyond one tile in both directions."""
import pytest

import test_gpu_sqgrad_fc_rows as rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("want_g", [False, True])
@pytest.mark.parametrize("B,J,C", [(63, 1, 64 * 511), (63, 1, 64 * 511 + 1), (64, 1, 64 * 511 + 1), (7, 64 * 512 - 1, 32), (64, 64 * 512 - 1, 32),
                                   (5, 33, 64 * 512 - 1), (1, 67, 33), (8, 67, 33), (9, 67, 33), (8, 129, 191)])
def test_either_kernel(B, J, C, want_g, bf16):
    rows.test_any_row_length(B, J, C, want_g, bf16)
