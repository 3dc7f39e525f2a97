"""The FC statistic on rows of any length (not whole 16-byte pieces), float32 and bfloat16, at the edges of tiles, of chunks and
of the matrices' last piece, against the float64 oracle.  What lies behind the operands is NaN, what lies behind the outputs
must stay."""
import numpy as np
import pytest

from oracle import vgc_oracle as O

pytestmark = pytest.mark.gpu


def _behind(torch, a, dtype):
    """a on the GPU, in a buffer that goes on with NaN."""
    buf = torch.full((a.size + 64,), float("nan"), dtype=dtype, device="cuda")
    buf[:a.size] = torch.from_numpy(a.ravel()).cuda().to(dtype)
    return buf[:a.size].view(a.shape)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("want_g", [False, True])
@pytest.mark.parametrize("B,J,C", [(1, 1, 1), (1, 3, 2), (2, 5, 7), (15, 63, 65), (16, 65, 63), (17, 66, 1), (33, 129, 127), (48, 1, 131), (100, 62, 4), (5, 2947, 2941), (273, 2945, 2943)])
def test_any_row_length(B, J, C, want_g, bf16):
    import torch
    from paper_1802_06058_amd import vgc
    rng = np.random.default_rng(B * J + C)
    X, D = rng.standard_normal((B, J), dtype=np.float32), rng.standard_normal((B, C), dtype=np.float32)
    dtype = torch.bfloat16 if bf16 else torch.float32
    Xd, Dd = _behind(torch, X, dtype), _behind(torch, D, dtype)
    X, D = Xd.float().cpu().numpy(), Dd.float().cpu().numpy()
    out = [torch.full((J * C + 64,), -7.0, device="cuda") for _ in range(2)]
    c = 1.0 / B
    vgc.sqgrad(vgc.FC, Xd, Dd, c, out[0], out[1] if want_g else None)
    g64, s64 = O.sqgrad_fc(X, D, c)
    s, g = (t[:J * C].view(J, C).cpu().numpy() for t in out)
    # float32 products and sums, also of bfloat16 inputs: at most B + 3 roundings of 2^-24 of the magnitudes summed
    assert np.all(np.abs(s - s64) <= (B + 3) * 2.0 ** -24 * s64)
    if want_g:
        mag = np.abs(X).astype(np.float64).T @ np.abs(D).astype(np.float64) * c
        assert np.all(np.abs(g - g64) <= (B + 3) * 2.0 ** -24 * mag)
    assert all(bool((t[J * C if i == 0 or want_g else 0:] == -7.0).all()) for i, t in enumerate(out))
