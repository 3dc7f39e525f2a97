"""The float32 conv statistic of 3 x 3 layers with unit stride and padding 1 that stages every input pixel once for all nine taps
(k_conv_taps_f32): at the edges of its ring, its groups of samples and its parts of positions, against float64 and against the
general kernel on the patch matrix; and sums that are not finite."""
import numpy as np
import pytest

from test_gpu_sqgrad_conv2d import _patches, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_1802_06058_amd import vgc
    assert torch.cuda.is_available()
    vgc.load()
    return torch.device("cuda:0")


SHAPES = [  # B, H, W, Cin, C
    (12, 9, 28, 192, 88),       # two pixels beyond a sample's last block, samples in two parts, ragged columns
    (8, 68, 6, 236, 76),        # three such pixels, three parts, a ragged channel block
    (5, 3, 78, 188, 220),       # the widest rows that fit the ring
    (12, 47, 6, 152, 68),       # rows much shorter than a block
    (32, 14, 14, 256, 256),     # one such pixel; groups of two samples
    (16, 34, 11, 256, 204),     # four such pixels, one sample a group
    (9, 17, 17, 320, 320),      # an odd number of groups
    (32, 7, 7, 512, 512),       # groups of eight samples: g is summed by groups as well
]


def _inputs(shape):
    B, H, W, Cin, C = shape
    rng = np.random.default_rng(sum(shape))
    return rng.standard_normal((B, H, W, Cin)).astype(np.float32), (rng.standard_normal((B, H, W, C)) * 1e-3).astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_shapes(dev, shape):
    _check_shape(dev, shape, (True,))


# Layers whose results the kernel scales and writes itself: their samples are not split (without a workspace), or in two and g is asked
# for, when the first half's sums of g wait in g's own buffer from four samples on.  And layers that would have so few groups of
# samples that sums in a row grow longer than in the general kernel.  (The host check states the splits.)
@pytest.mark.parametrize("shape", [(9, 7, 7, 512, 1024), (8, 7, 7, 512, 1024), (5, 14, 14, 1024, 512), (6, 7, 7, 512, 1024),
                                   (16, 7, 7, 1024, 1024), (57, 13, 13, 456, 464)], ids=lambda s: "x".join(map(str, s)))
def test_few_groups(dev, shape):
    _check_shape(dev, shape, (True, False) if shape[4] == 1024 or shape[3] == 1024 else (True,))


def _check_shape(dev, shape, workspaces):
    import torch
    from paper_1802_06058_amd import vgc
    B, H, W, Cin, C = shape
    A, D = _inputs(shape)
    c = float(np.float32(1.0 / B))
    P, J = H * W, 9 * Cin
    U = torch.from_numpy(_patches(A, 3, 3, (1, 1), (1, 1), H, W)).to(dev)
    E = torch.from_numpy(D.reshape(B, P, C)).to(dev)
    g64, s64, mag = (torch.zeros(J, C, dtype=torch.float64, device=dev) for _ in range(3))
    for z in range(B):
        u, e = U[z].double().t().contiguous(), E[z].double()
        G = u @ e
        g64 += G * c
        s64 += G * G * c * c
        mag += (u.abs() @ e.abs()) * c
    g64, s64, mag = g64.cpu().numpy(), s64.cpu().numpy(), mag.cpu().numpy()
    norm = lambda x: np.sqrt((x.astype(np.float64) ** 2).sum())
    for use_workspace in workspaces:
        g, s = _run(A, D, 3, 3, (1, 1), (1, 1), c, dev, True, use_workspace)
        _, s_only = _run(A, D, 3, 3, (1, 1), (1, 1), c, dev, False, use_workspace)
        assert np.array_equal(s_only, s)
        # as for the general kernel: |G_z - exact| <= about (P / 32 + 8) roundings of 2^-24 of the magnitudes summed, s doubles it, and
        # sums over at least five samples do not cancel below a hundredth of the magnitudes squared
        assert np.all(np.abs(s - s64) <= 1e-5 * s64)
        assert np.all(np.abs(g - g64) <= 1e-6 * mag)
        s_gen, g_gen = torch.empty(J, C, device=dev), torch.empty(J, C, device=dev)
        nb = vgc.sqgrad_workspace_bytes(vgc.CONV, vgc.F32, B, P, J, C) if use_workspace else 0
        vgc.sqgrad(vgc.CONV, U, E, c, s_gen, g_gen, workspace=torch.empty(nb, dtype=torch.uint8, device=dev) if nb else None)
        s_gen, g_gen = s_gen.cpu().numpy(), g_gen.cpu().numpy()
        assert not np.array_equal(s_gen, s)                          # another kernel, or this file tests nothing
        assert np.all(np.abs(s - s_gen) <= 2 * 1e-5 * s64)
        # no further from float64 than the general kernel by more than the spread between inputs
        assert norm(s - s64) <= 1.15 * norm(s_gen - s64)
        assert norm(g - g64) <= 1.15 * norm(g_gen - g64)


@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[3], SHAPES[4]], ids=lambda s: "x".join(map(str, s)))
def test_sums_that_are_not_finite(dev, shape):
    """Infinities, NaN and products beyond float32 at the corners of samples, beside which the ring holds another sample's pixels:
    each output is what float32 arithmetic makes of the inputs it depends on, and no other output sees them."""
    B, H, W, Cin, C = shape
    A, D = _inputs(shape)
    D *= 1e3
    A[0, 0, 0, 1], A[-1, -1, -1, 2], A[B // 2, H // 2, W // 2, 3] = np.inf, -np.inf, np.nan
    A[1, H - 1, 0, 1], A[2, 0, W - 1, 0], A[2, H - 1, W - 1, 7] = np.inf, np.inf, -np.inf
    D[0, 0, 0, 3], D[-1, -1, -1, 2], D[3, 0, W - 1, 1] = np.inf, np.nan, -np.inf
    A[1, 0, 0, 4], D[1, 0, 0, 4] = 1.7 * 2.0 ** 100, -1.3 * 2.0 ** 100
    D[2, 0, 0, 6] = 3.4028235e38                                     # rounds up to infinity in 16 bits
    A[2, :, :, 6] = 2.0 ** -100
    c = np.float32(1.0 / B)
    U, E = _patches(A, 3, 3, (1, 1), (1, 1), H, W), D.reshape(B, H * W, C)
    with np.errstate(all="ignore"):
        G = np.matmul(np.ascontiguousarray(U.transpose(0, 2, 1)), E)
        G64 = np.stack([U[z].T.astype(np.float64) @ E[z].astype(np.float64) for z in range(B)])
        want = []
        for x, x64, scale in (((G * G).sum(0), (G64 * G64).sum(0), float(c) ** 2), (G.sum(0), G64.sum(0), float(c))):
            want.append(np.where(np.isfinite(x), x64, x) * scale)
    s64, g64 = want
    assert np.isinf(s64).any() and np.isnan(s64).any() and np.isfinite(s64).any()
    for want_g in (False, True):
        g, s = _run(A, D, 3, 3, (1, 1), (1, 1), float(c), dev, want_g)
        for got, ref, rtol in ((s, s64, 1e-5), (g, g64, None)):
            if got is None:
                continue
            assert np.array_equal(np.isnan(got), np.isnan(ref))
            inf, fin = np.isinf(ref), np.isfinite(ref)
            assert np.array_equal(got[inf], ref[inf].astype(np.float32)) and np.isfinite(got[fin]).all()
            if rtol:
                assert np.all(np.abs(got[fin] - ref[fin]) <= rtol * ref[fin])


@pytest.mark.parametrize("shape", [(32, 14, 14, 256, 256), (8, 7, 7, 512, 1024), (4, 14, 14, 1024, 512)], ids=lambda s: "x".join(map(str, s)))
def test_s_is_the_same_with_g_beside_sums_that_are_not_finite(dev, shape):
    """A workgroup has two groups of samples with g and one without.  Where one group's sums are not finite they are formed again, and
    finite ones share their tiles: s is the same bits whether g is asked for or not.  Infinities in the first, the second and in both
    groups of a pair, a NaN, and a group whose sum alone overflows."""
    B, H, W, Cin, C = shape
    A, D = _inputs(shape)
    D *= 1e3
    A[0, 0, 0, 1], A[B // 4 - 1, H // 2, 3, 40], A[B // 2, 1, 1, 70], A[-1, 2, 2, 100], D[1, 3, 3, 20] = np.inf, -np.inf, np.inf, np.inf, np.nan
    A[B // 2 + 1, 4, 4, 130], D[B // 2 + 1, 4, 4, 200] = 2.0 ** 80, 2.0 ** 20
    c = float(np.float32(1.0 / B))
    for use_workspace in (True, False):
        _, s = _run(A, D, 3, 3, (1, 1), (1, 1), c, dev, False, use_workspace)
        _, s_with_g = _run(A, D, 3, 3, (1, 1), (1, 1), c, dev, True, use_workspace)
        assert np.isnan(s).any() and np.isinf(s).any() and np.isfinite(s).any()
        np.testing.assert_array_equal(s_with_g, s)
