"""The float32 conv statistic on the bf16 matrix cores (three bf16 pieces per element): every block tile, input mode and
remainder of its kernel against the float64 oracle; that no bit of a float32 input is lost over the range of exponents;
that the sums are not biased although the matrix instruction truncates; and sums that are not finite."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from test_gpu_sqgrad_conv2d import _patches, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_1802_06058_amd import vgc
    assert torch.cuda.is_available()
    vgc.load()
    return torch.device("cuda:0")


SHAPES = [  # B, H, W, Cin, C, k, stride, pad          tile, input mode
    (4, 4, 8, 60, 60, 1, 1, 0),                      # 64 x 64, 32 positions: one whole chunk
    (5, 3, 11, 64, 68, 1, 1, 0),                     # 64 x 128 with a ragged column tile, 33 positions
    (4, 31, 1, 132, 64, 1, 1, 0),                    # 128 x 64, 31 positions, output one column wide
    (6, 7, 7, 24, 132, 3, 1, 1),                     # 128 x 128, 49 positions, ragged in both directions
    (4, 9, 14, 36, 128, 3, 2, 1),                    # general mode: stride 2
    (4, 8, 37, 16, 64, 3, 1, 1),                     # W = 37: a period of 37 chunks does not fit the mask
    (5, 10, 32, 16, 64, 3, 1, 1),                    # W = 32: a period of one chunk
    (4, 66, 33, 12, 12, 3, 1, 1),                    # the positions split over workgroups
    (4, 40, 41, 8, 132, 2, 1, 0),                    # even kernel, output narrower than the input
    (40, 3, 5, 256, 1024, 1, 1, 0),                  # several samples per workgroup
    (4, 4, 4, 60, 60, 1, 1, 0),                      # at most 16 positions, where two products share an MFMA: 64 x 64, 16 of them
    (6, 1, 1, 200, 200, 1, 1, 0),                    # 128 x 128, one position
    (4, 7, 8, 12, 200, 3, 2, 1),                     # 128 x 128, stride 2
    (4, 2, 2, 200, 60, 2, 1, 1),                     # 128 x 64, 9 positions
    (35, 3, 4, 60, 200, 1, 1, 0),                    # 64 x 128, 12 positions, an odd number of samples
    (4, 1, 17, 60, 60, 1, 1, 0),                     # 17: no longer
]


@pytest.mark.parametrize("want_g", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_shapes(dev, shape, want_g):
    import torch
    from paper_1802_06058_amd import vgc
    B, H, W, Cin, C, k, st, pad = shape
    rng = np.random.default_rng(B * H + W + C)
    A = rng.standard_normal((B, H, W, Cin)).astype(np.float32)
    Ho, Wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    D = (rng.standard_normal((B, Ho, Wo, C)) * 1e-3).astype(np.float32)
    U = _patches(A, k, k, (st, st), (pad, pad), Ho, Wo).astype(np.float64)
    E = D.reshape(B, Ho * Wo, C).astype(np.float64)
    G = np.matmul(U.transpose(0, 2, 1), E)
    c = np.float32(1.0 / B)
    g64, s64 = G.sum(0) * float(c), (G * G).sum(0) * float(c) ** 2
    mag = np.matmul(np.abs(U).transpose(0, 2, 1), np.abs(E)).sum(0) * float(c)
    runs = [_run(A, D, k, k, (st, st), (pad, pad), float(c), dev, want_g, use_ws) for use_ws in (True, False)]
    X = torch.from_numpy(np.ascontiguousarray(U.astype(np.float32))).to(dev)
    Dd = torch.from_numpy(np.ascontiguousarray(D.reshape(B, Ho * Wo, C))).to(dev)
    s = torch.empty(U.shape[2], C, device=dev)
    g = torch.empty(U.shape[2], C, device=dev) if want_g else None
    vgc.sqgrad(vgc.CONV, X, Dd, float(c), s, g)                      # the patch matrix, no workspace
    runs.append((g.cpu().numpy() if want_g else None, s.cpu().numpy()))
    for gv, sv in runs:
        # |G_z - exact| <= about (P / 32 + 8) roundings of 2^-24 of the magnitudes summed; s doubles it.  The outputs are sums
        # over at least four samples, so s does not cancel below a hundredth of the magnitudes squared.
        assert np.all(np.abs(sv - s64) <= 1e-5 * s64)
        if want_g:
            assert np.all(np.abs(gv - g64) <= 1e-6 * mag)


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("positions", [1, 20])
@pytest.mark.parametrize("exponent", [-145, -130, -126, -112, -104, -100, -60, -1, 0, 60, 126])
def test_every_bit_of_the_inputs_counts(dev, exponent, positions, swap):
    """One sample, one position (or one and zeros): g is the product of two floats, one with mantissas that are the hardest to cut, the other
    around one.  A power of two is a piece of its own, so the other operand must come back bit for bit.  In general the
    products of pieces that are left out stay below 2^-24 of the product (mid below 2^-8, lo below 2^-17 of the leading bit,
    mid lo and lo mid), the last addition is cut off at 2^-23 of it, and the five before it at 2^-31."""
    rng = np.random.default_rng(exponent + 200)
    n = 64
    hard = [1 + 2.0 ** -23, 2 - 2.0 ** -23, 1 + 2.0 ** -16, 1 + 2.0 ** -8, 1.0077972, 1.0038986, 1 + 2.0 ** -8 + 2.0 ** -23]
    x = np.ldexp(rng.uniform(1, 2, n), exponent).astype(np.float32)
    x[:len(hard)] = np.ldexp(np.array(hard), exponent).astype(np.float32)
    x[len(hard):2 * len(hard)] = -x[:len(hard)]
    up = np.float32(2.0 ** max(0, -60 - exponent))                  # tiny (and subnormal) elements: a product in the normal range
    d = rng.uniform(0.5, 1, n).astype(np.float32)
    d[:5] = [1.0, 1 - 2.0 ** -24, 1.0077972, 0.25, 1.0038986]
    if exponent == 126:
        d[2], d[4] = 0.50389862, 0.5019608
        x[20] = np.float32(3.4028235e38)                            # the largest float: it rounds up to infinity in 16 bits
    d *= up
    a, b = (d, x) if swap else (x, d)
    at = lambda v: np.concatenate([v, np.zeros((positions - 1) * n, np.float32)]).reshape(1, 1, positions, n)
    g, _ = _run(at(a), at(b), 1, 1, (1, 1), (0, 0), 1.0, dev)
    want = np.outer(a.astype(np.float64), b.astype(np.float64))
    assert np.all(np.abs(g - want) <= (2.0 ** -24 + 2.0 ** -23 + 5 * 2.0 ** -31) * np.abs(want))
    g = g.T if swap else g
    assert np.array_equal(g[:, 0], x * up) and np.array_equal(g[:, 3], x * (up / 4))


def test_sums_are_not_biased(dev):
    """The mean error of g over many outputs: each output errs by at most 1e-6 of its magnitudes, and if the truncation of the
    matrix instruction did not cancel, all would err to the same side (1e-7 of the magnitudes at 1600 positions)."""
    rng = np.random.default_rng(5)
    B, H, Cin, C = 8, 40, 64, 64
    A = rng.standard_normal((B, H, H, Cin)).astype(np.float32)
    D = rng.standard_normal((B, H, H, C)).astype(np.float32)
    g, _ = _run(A, D, 1, 1, (1, 1), (0, 0), 1.0, dev, use_workspace=False)
    U, E = A.reshape(-1, Cin).astype(np.float64), D.reshape(-1, C).astype(np.float64)
    err = g - U.T @ E
    assert abs(err.mean()) <= 2e-9 * (np.abs(U).T @ np.abs(E)).mean()


def _float32_results(U, E, c):
    """g and s from patches U [B, P, J] and gradients E [B, P, C]: which outputs are not finite as float32 arithmetic has it
    (0 * inf and inf - inf are NaN, what leaves the range is infinite), the finite ones' values in 64 bits."""
    with np.errstate(all="ignore"):
        G, G64 = np.einsum("zpj,zpc->zjc", U, E), np.einsum("zpj,zpc->zjc", U.astype(np.float64), E.astype(np.float64))
        g, s = G.sum(0), (G * G).sum(0)
        return np.where(np.isfinite(g), G64.sum(0), g) * float(c), np.where(np.isfinite(s), (G64 * G64).sum(0), s) * float(c) ** 2


@pytest.mark.parametrize("want_g", [False, True])
@pytest.mark.parametrize("shape", SHAPES + [(4, 6, 6, 16, 16, 1, 1, 0), (3, 64, 48, 8, 8, 3, 1, 1)], ids=lambda s: "x".join(map(str, s)))
def test_sums_that_are_not_finite(dev, shape, want_g):
    """Infinities, NaN and products beyond the range of float32: each output is what float32 arithmetic makes of the inputs it
    depends on, whatever the elements are cut into, and no other output sees them."""
    import torch
    from paper_1802_06058_amd import vgc
    B, H, W, Cin, C, k, st, pad = shape
    rng = np.random.default_rng(B + H + W + C)
    Ho, Wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    A = rng.standard_normal((B, H, W, Cin)).astype(np.float32)
    D = rng.standard_normal((B, Ho, Wo, C)).astype(np.float32)
    A[0, 0, 0, 1], A[-1, -1, -1, 2], A[B // 2, H // 2, W // 2, 3] = np.inf, -np.inf, np.nan
    A[1, H - 1, 0, 1] = np.inf                                      # beside the first: inf + inf or inf - inf
    D[0, 0, 0, 3], D[-1, -1, -1, 2] = np.inf, np.nan
    A[1, 0, 0, 4], D[1, 0, 0, 4] = 1.7 * 2.0 ** 100, -1.3 * 2.0 ** 100
    D[1, Ho // 2, Wo // 2, 5], A[..., 5] = 3.4028235e38, 1.0         # in range as a product, not as a square
    D[2, 0, 0, 6] = 3.4028235e38                                     # rounds up to infinity in 16 bits
    A[2, :, :, 6] = 2.0 ** -100
    c = np.float32(1.0 / B)
    U = _patches(A, k, k, (st, st), (pad, pad), Ho, Wo)
    E = D.reshape(B, Ho * Wo, C)
    g64, s64 = _float32_results(U, E, c)
    runs = [_run(A, D, k, k, (st, st), (pad, pad), float(c), dev, want_g, use_ws) for use_ws in (True, False)]
    X, Dd = torch.from_numpy(np.ascontiguousarray(U)).to(dev), torch.from_numpy(np.ascontiguousarray(E)).to(dev)
    s = torch.empty(U.shape[2], C, device=dev)
    g = torch.empty(U.shape[2], C, device=dev) if want_g else None
    nb = vgc.sqgrad_workspace_bytes(vgc.CONV, vgc.F32, B, Ho * Wo, U.shape[2], C)
    ws = torch.empty(nb, dtype=torch.uint8, device=dev) if nb else None
    vgc.sqgrad(vgc.CONV, X, Dd, float(c), s, g, workspace=ws)
    runs.append((g.cpu().numpy() if want_g else None, s.cpu().numpy()))
    assert np.isinf(s64).any() and np.isnan(s64).any() and np.isfinite(s64).any()
    for gv, sv in runs:
        for got, want, rtol in ((sv, s64, 1e-5), (gv, g64, None)):
            if got is None:
                continue
            assert np.array_equal(np.isnan(got), np.isnan(want))
            inf = np.isinf(want)
            assert np.array_equal(got[inf], want[inf].astype(np.float32))
            fin = np.isfinite(want)
            assert np.isfinite(got[fin]).all()
            if rtol:
                assert np.all(np.abs(got[fin] - want[fin]) <= rtol * want[fin])
