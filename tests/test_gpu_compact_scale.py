"""The compact decoder against the plain one for scales of either sign, zero and at the ends of the range, on a buffer that holds
zeros of both signs: bytes that end no element must leave every bit of it as it is.  Bit-exact."""
import numpy as np
import pytest

from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [0.5, 6.0], ids=["dense", "two-byte-gaps"])
@pytest.mark.parametrize("scale", [0.25, -0.25, 0.0, -0.0, 1e-37, -3e38])
def test_scale_and_signed_zeros(scale, alpha):
    import torch
    from paper_1802_06058_amd import vgc
    sizes = [2048 * 9 + 77, 3, 2048 * 3, 700]
    groups, n = W.groups_from_sizes(sizes), sum(sizes)
    gen = torch.Generator(device="cuda").manual_seed(5)
    plan = vgc.Plan(groups, "cuda")
    g = torch.randn(n, generator=gen, device="cuda") * torch.exp2(torch.randint(-4, 5, (n,), generator=gen, device="cuda").float())
    s, r, v = torch.full((n,), 1.0, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    scratch, status = plan.new_scratch(), plan.new_status()
    vgc.accumulate_select(g, s, r, v, plan, alpha, 0.999, scratch)
    words, hdrs = torch.zeros(n, dtype=torch.int32, device="cuda"), plan.new_headers()
    vgc.pack(plan, scratch, words, hdrs, status)
    stream, tile_bytes = torch.zeros(2 * n, dtype=torch.uint8, device="cuda"), torch.zeros(plan.n_tiles, dtype=torch.int16, device="cuda")
    runs, chdrs = torch.zeros(plan.n_runs, dtype=torch.int64, device="cuda"), plan.new_headers()
    vgc.pack_compact(plan, scratch, stream, tile_bytes, runs, chdrs, status)
    n_bytes, _ = vgc.read_status(status)
    zeros = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.5, -0.0, 0.0)
    dense = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.5, zeros, torch.randn(n, generator=gen, device="cuda"))
    a, b = dense.clone(), dense.clone()
    vgc.unpack_add_batch([words], [n], [hdrs], plan, scale, a)
    vgc.unpack_compact_add_batch([stream], [n_bytes], [tile_bytes], [runs], [chdrs], plan, scale, b)
    a, b = a.cpu().numpy().view(np.uint32), b.cpu().numpy().view(np.uint32)
    nan = np.isnan(a.view(np.float32))
    assert np.array_equal(np.isnan(b.view(np.float32)), nan) and np.array_equal(a[~nan], b[~nan])
    assert scale == 0 or np.any(a != dense.cpu().numpy().view(np.uint32))
