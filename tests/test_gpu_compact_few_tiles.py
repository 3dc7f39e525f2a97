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


@pytest.mark.parametrize("alpha", [0.5, 40.0])
def test_two_tiles_a_wave(dev, alpha):
    """From 65536 tiles on a wave encodes two, which may belong to different runs and groups; the number is odd.  Against the plain
    encoder's message: decoded the same, and the directory adds up."""
    import torch
    from paper_1802_06058_amd import vgc
    sizes = [T * 64 * 500 + 7, 3, T * 65, T * 33466 + 1, 2 * T, 1]
    groups, n = W.groups_from_sizes(sizes), sum(sizes)
    plan = vgc.Plan(groups, dev)
    assert plan.n_tiles >= 65536 and plan.n_tiles % 2 == 1
    gen = torch.Generator(device=dev).manual_seed(int(alpha))
    g = torch.randn(n, generator=gen, device=dev)
    g *= torch.exp2(torch.randint(-3, 4, (n,), generator=gen, device=dev).float())
    g[T * 1000:T * 1100] = 0                                   # tiles without any
    s, r, v = torch.full((n,), 1.0, device=dev), torch.zeros(n, device=dev), torch.zeros(n, device=dev)
    scratch, status = plan.new_scratch(), plan.new_status()
    vgc.accumulate_select(g, s, r, v, plan, alpha, 0.999, scratch)
    words, hdrs = torch.zeros(n, dtype=torch.int32, device=dev), plan.new_headers()
    vgc.pack(plan, scratch, words, hdrs, status)
    count, _ = vgc.read_status(status)
    msg = compact.CompactMessage(plan, dev, 2 * n)
    vgc.pack_compact(plan, scratch, msg.stream[:msg.cap], msg.tile_bytes, msg.run_offsets, msg.hdrs, msg.status)
    total, overflow = vgc.read_status(msg.status)
    tile_bytes = msg.tile_bytes.long()
    begin = tile_bytes.cumsum(0) - tile_bytes
    first, runs = 0, []
    for size in sizes:
        tiles = (size + T - 1) // T
        runs += range(first, first + tiles, 64)
        first += tiles
    assert overflow == 0 and count <= total == int(tile_bytes.sum()) and torch.equal(begin[torch.tensor(runs, device=dev)], msg.run_offsets)
    assert [h[:2] for h in vgc.read_headers(msg.hdrs)] == [h[:2] for h in vgc.read_headers(hdrs)]
    # streams that end inside a wave's second tile, between its two, inside the first, where a run begins, and before the first byte
    wave = plan.n_tiles // 4
    at = {k: int(begin[2 * wave + k]) for k in (0, 1, 2)}
    assert at[0] + 2 < at[1] < at[2] - 2
    want = [x.clone() for x in (msg.stream, msg.tile_bytes, msg.run_offsets)]
    run = int(msg.run_offsets[plan.n_runs // 2])
    for cap in (total, total - 1, at[2] - 1, at[1] + 1, at[1], at[0] + 1, run, run - 1, 1, 0):
        for x, fill in ((msg.stream, 0xEE), (msg.tile_bytes, -1), (msg.run_offsets, -1)):
            x.fill_(fill)
        vgc.pack_compact(plan, scratch, msg.stream[:cap], msg.tile_bytes, msg.run_offsets, msg.hdrs, msg.status)
        assert vgc.read_status(msg.status) == (total, int(total > cap))
        assert torch.equal(msg.stream[:cap], want[0][:cap]) and bool((msg.stream[cap:] == 0xEE).all())
        assert torch.equal(msg.tile_bytes, want[1]) and torch.equal(msg.run_offsets, want[2])
    msg.stream.copy_(want[0])
    a, b = g, s                                                # (buffers whose contents are no longer needed)
    vgc.unpack_add_batch([words], [count], [hdrs], plan, 0.5, a, overwrite=True)
    vgc.unpack_compact_add_batch([msg.stream], [total], [msg.tile_bytes], [msg.run_offsets], [msg.hdrs], plan, 0.5, b, overwrite=True)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32)) and bool((msg.stream[msg.cap:] == 0xEE).all())
