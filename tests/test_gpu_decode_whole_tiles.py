"""The plain decoders where every group is whole tiles, either side of the rule by which a workgroup takes a tile: 512 tiles, and
above them few or many words; and the largest set with a ragged group that is decoded so.  Bit-exact."""
import numpy as np
import pytest

import test_gpu_decode_by_tile as by_tile
from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu
T = 2048


@pytest.mark.parametrize("sizes", [[500 * T, 12 * T], [500 * T, 13 * T], [1000 * T - 5, 280 * T]], ids=["512-tiles", "513-tiles", "1280-ragged"])
@pytest.mark.parametrize("rhos", [(0.0004, "tiles", 0.1), (0.9, 0.3, 0.0), (0.125, "tiles", 0.13)], ids=["sparse", "dense", "between"])
def test_decoders_at_the_rules_edge(sizes, rhos):
    import torch
    from paper_1802_06058_amd import vgc
    by_tile.test_decoders_at_the_rules_edge(sizes, rhos)
    # momentum SGD
    groups, n, rng = W.groups_from_sizes(sizes), sum(sizes), np.random.default_rng(3)
    x = rng.standard_normal(n, dtype=np.float32)
    msgs = [O.pack(x, rng.random(n, dtype=np.float32) < (0.05 if rho == "tiles" else rho), groups)[:2] for rho in rhos]
    words = [torch.from_numpy(np.append(w, np.uint32(5)).view(np.int32)).cuda() for w, _ in msgs]
    hdrs = [torch.from_numpy(np.array(h, dtype=vgc.HDR_DTYPE).view(np.uint8)).cuda() for _, h in msgs]
    w, m = x.copy(), x * np.float32(0.1)
    dw, dm = torch.from_numpy(w).cuda(), torch.from_numpy(m).cuda()
    w, m = O.unpack_apply(msgs, groups, 0.3, n, "momentum_sgd", w, m, lr=0.05, mu=0.9)
    vgc.unpack_apply(words, [a.size for a, _ in msgs], hdrs, vgc.Plan(groups, "cuda"), 0.3, dw, dm, kind=vgc.MOMENTUM_SGD, lr=0.05, momentum=0.9)
    assert np.array_equal(dw.cpu().numpy().view(np.uint32), w.view(np.uint32)) and np.array_equal(dm.cpu().numpy().view(np.uint32), m.view(np.uint32))
