"""vgc_pack against the oracle where its scans are divided: either side of what one launch takes, parts of a group either side
of their size, groups either side of a segment.  Bit-exact."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu
T = 2048


@pytest.mark.parametrize("sizes", [
    [2048 * T],                                                # the largest of the one launch, one group
    [2048 * T + 1],                                            # one tile more
    [1000] * 511 + [T * 5 + 9],                                # most groups of the one launch
    [1000] * 512 + [T * 5 + 9],                                # one more
    [1024 * T, 3, 1024 * T + 1, 700, 2048 * T],                # one part and two, small groups between them
    [2048 * T, 9, 2048 * T + 1],                               # two parts and three
    [5, 8192 * T, 8192 * T + 1, 17],                           # one segment and two
], ids=["2048-tiles", "2049-tiles", "512-groups", "513-groups", "parts", "three-parts", "segments"])
def test_pack_matches_oracle(sizes):
    import torch
    from paper_1802_06058_amd import vgc
    groups, n = W.groups_from_sizes(sizes), sum(sizes)
    rng = np.random.default_rng(len(sizes))
    # a scale per part of 1024 tiles and one per tile: parts and tiles differ in their exponents, whole tiles fall away
    scale = np.exp2(rng.integers(-6, 3, n // (1024 * T) + 1)).astype(np.float32).repeat(1024 * T)[:n]
    scale *= np.exp2(rng.integers(-9, 1, n // T + 1)).astype(np.float32).repeat(T)[:n]
    g = rng.standard_normal(n, dtype=np.float32) * scale
    z = np.zeros(n, np.float32)
    s = (scale * scale * rng.random(n, dtype=np.float32)).astype(np.float32)
    r_acc, _, _, send = O.accumulate_select(g, s, z, z, 2.0, 0.999)
    words, hdrs, _ = O.pack(r_acc, send, groups)

    plan = vgc.Plan(groups, "cuda")
    r, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    scratch, status = plan.new_scratch().fill_(0xAB), plan.new_status()
    out, gh = torch.full((words.size + 64,), -1, dtype=torch.int32, device="cuda"), plan.new_headers()
    vgc.accumulate_select(torch.from_numpy(g).cuda(), torch.from_numpy(s).cuda(), r, v, plan, 2.0, 0.999, scratch)
    for _ in range(2):                                         # a second call finds the records as the first one left them
        vgc.pack(plan, scratch, out[:words.size], gh, status)
    assert vgc.read_status(status) == (words.size, 0)
    assert vgc.read_headers(gh) == hdrs
    got = out.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:words.size], words) and np.all(got[words.size:] == 0xFFFFFFFF)
