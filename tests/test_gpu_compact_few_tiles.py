"""vgc_pack_compact on either side of the line between its two forms (at most 2048 tiles and 512 groups: two kernels whose workgroups
read all tile records; beyond: scans), against the oracle, bit for bit, also where the stream does not fit."""
import numpy as np
import pytest

import test_gpu_compact as compact
from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W
from streams import sample_stream

pytestmark = pytest.mark.gpu
T = 2048
SETS = {
    "tiles-2048": [T * 2000 + 1, 5, T * 45 + 1],
    "tiles-2049": [T * 2000 + 1, 5, T * 46 + 1],
    "groups-512": [40, 3, 2500, 1] * 128,
    "groups-513": [40, 3, 2500, 1] * 128 + [70],
    "five-tiles": [T, 1, T * 2, 9],
    "runs": [T * 64, T * 65, T * 63 + 1, T * 128 + 1],
}


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_1802_06058_amd import vgc
    vgc.load()
    return torch.device("cuda:0")


@pytest.mark.parametrize("alpha", [0.5, 6.0])
@pytest.mark.parametrize("name", list(SETS))
def test_both_forms_match_the_oracle(dev, name, alpha):
    import torch
    from paper_1802_06058_amd import vgc
    groups = W.groups_from_sizes(SETS[name])
    plan = vgc.Plan(groups, dev)
    g, s = sample_stream(74, (len(name),), plan.n, 16, "normal", sigma=0.1)
    g[groups[-2][0]:] = 0                                      # the last two groups send nothing
    scratch = compact._select(plan, g, s, alpha, dev)
    words, hdrs = compact._oracle_message(g, s, groups, alpha)
    stream, tile_bytes, runs, chdrs = O.pack_compact(words, hdrs, groups)
    assert stream.size > 2
    for cap in (2 * plan.n, stream.size, stream.size - 1, stream.size // 2, 1, 0):
        msg = compact.CompactMessage(plan, dev, cap)
        vgc.pack_compact(plan, scratch, msg.stream[:cap], msg.tile_bytes, msg.run_offsets, msg.hdrs, msg.status)
        torch.cuda.synchronize()
        assert vgc.read_status(msg.status) == (stream.size, int(stream.size > cap)) and vgc.read_headers(msg.hdrs) == chdrs
        got, most = msg.stream.cpu().numpy(), min(cap, stream.size)
        assert np.array_equal(got[:most], stream[:most]) and np.all(got[most:] == 0xEE)
        assert np.array_equal(msg.tile_bytes.cpu().numpy().view(np.uint16), tile_bytes)
        assert np.array_equal(msg.run_offsets.cpu().numpy().view(np.uint64), runs)
