"""The float32 FC statistic at the edges of its two block tiles, of its staged chunks of 16 samples and of the fallback's
requests ahead, against the float64 oracle."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W
from test_gpu_sqgrad import _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_1802_06058_amd import vgc
    assert torch.cuda.is_available()
    vgc.load()
    return torch.device("cuda:0")


@pytest.mark.parametrize("want_g", [False, True])
@pytest.mark.parametrize("B,J,C", [
    (16, 64, 64), (17, 68, 60), (1, 4, 132), (33, 132, 4),            # 64 x 64: one tile, ragged tiles, one chunk and more
    (31, 2888, 2884), (16, 4100, 2052),                               # 529 and 561 tiles of 128 x 128: the larger tile, ragged
    (256, 2888, 2884), (273, 2948, 2820),                             # the larger tile's form for long sums: an even and an odd number of chunks
    (15, 2816, 2944),                                                 # 22 x 23 = 506 of them: still the smaller tile
    (16, 33, 31), (17, 65, 10), (1, 1, 1), (48, 129, 67),             # rows that are not whole 16-byte pieces: the fallback
])
def test_fc_f32(dev, B, J, C, want_g):
    from paper_1802_06058_amd import vgc
    X, D = W.fc_inputs(23, (B, J, C), B, J, C, "normal", True, 0.02)
    c = 1.0 / B
    g, s = _run(vgc.FC, X, D, c, dev, False, want_g=want_g)
    g64, s64 = O.sqgrad_fc(X, D, c)
    # products and sums in float32: at most B + 3 roundings of 2^-24 of the magnitudes summed, which for s are s itself
    assert np.all(np.abs(s - s64) <= (B + 3) * 2.0 ** -24 * s64)
    if want_g:
        mag = np.abs(X).astype(np.float64).T @ np.abs(D).astype(np.float64) * c
        assert np.all(np.abs(g - g64) <= (B + 3) * 2.0 ** -24 * mag)
