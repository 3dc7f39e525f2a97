"""vgc_pack and vgc_pack_compact where their scans go from chunk to chunk: 1024 segments or runs at a time, parts of large groups
among many small ones, several parts and segments of a group in the compact format; buffers too small and plans of another
group list beyond what the one-launch packer takes.  Bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W

T = 2048


def _small(n_groups):
    return np.random.default_rng(n_groups).integers(1, 3000, n_groups).tolist()


SETS = {
    "1024-groups": _small(1024),
    "1025-groups": _small(1025),
    "2100-groups": _small(2100),
    "large-among-small": [700] * 1500 + [3 * 1024 * T + 5] + [3] * 40 + [1024 * T + 1, 9, 8193 * T],
    "2049-tiles": [2048 * T + 1],
    "parts": [1024 * T, 3, 1024 * T + 1, 700, 2048 * T],
    "three-parts": [2048 * T, 9, 2048 * T + 1],
    "segments": [5, 8192 * T, 8192 * T + 1, 17],
}


def _compact(words, hdrs, groups):
    """O.pack_compact without a loop over elements (held against it below)."""
    size = np.array([s for _, s in groups])
    tiles = (size + T - 1) // T
    first_tile = np.cumsum(tiles) - tiles
    group = np.repeat(np.arange(len(groups)), [c for _, c, _ in hdrs])
    index = (words & np.uint32(0x0FFFFFFF)).astype(np.int64)
    tile, pos = first_tile[group] + index // T, index % T
    before = np.full(index.size, -1)
    before[1:] = np.where(tile[1:] == tile[:-1], pos[:-1], -1)
    gap = pos - before - 1
    two = gap >= 8
    behind = np.cumsum(1 + two)
    stream = np.zeros(int(behind[-1]) if index.size else 0, np.uint8)
    stream[behind - 1 - two] = np.where(two, 0x80, 0) | (gap & 7) << 4 | (words >> np.uint32(28)).astype(np.int64)
    stream[behind[two] - 1] = gap[two] >> 3
    tile_bytes = np.bincount(tile, weights=1 + two, minlength=int(tiles.sum())).astype(np.uint16)
    begin = np.cumsum(tile_bytes, dtype=np.uint64) - tile_bytes
    runs = np.concatenate([np.arange(f, f + t, 64) for f, t in zip(first_tile, tiles)])
    return stream, tile_bytes, begin[runs], [(e, c, int(begin[f])) for (e, c, _), f in zip(hdrs, first_tile)]


def _step(sizes):
    """g, s of a step and the oracle's message: scales differ from part to part and from tile to tile, whole tiles and (among
    small ones) groups fall away."""
    groups, n = W.groups_from_sizes(sizes), sum(sizes)
    rng = np.random.default_rng(len(sizes))
    scale = np.exp2(rng.integers(-6, 3, n // (1024 * T) + 1)).astype(np.float32).repeat(1024 * T)[:n]
    scale *= np.exp2(rng.integers(-9, 1, n // T + 1)).astype(np.float32).repeat(T)[:n]
    g = rng.standard_normal(n, dtype=np.float32) * scale
    for k in range(0, len(groups), 7):
        if groups[k][1] < T:
            g[groups[k][0]:groups[k][0] + groups[k][1]] = 0
    z = np.zeros(n, np.float32)
    s = (scale * scale * rng.random(n, dtype=np.float32)).astype(np.float32)
    r_acc, _, _, send = O.accumulate_select(g, s, z, z, 2.0, 0.999)
    return groups, g, s, O.pack(r_acc, send, groups)[:2]


def _selected(groups, g, s):
    import torch
    from paper_1802_06058_amd import vgc
    plan = vgc.Plan(groups, "cuda")
    r, v = torch.zeros(g.size, device="cuda"), torch.zeros(g.size, device="cuda")
    scratch = plan.new_scratch().fill_(0xAB)
    vgc.accumulate_select(torch.from_numpy(g).cuda(), torch.from_numpy(s).cuda(), r, v, plan, 2.0, 0.999, scratch)
    return plan, scratch


@pytest.mark.parametrize("sizes", [_small(40), [T * 65 + 7, 3, T], [1]])
def test_the_reference_without_loops(sizes):
    groups, _, _, (words, hdrs) = _step(sizes)
    want, got = O.pack_compact(words, hdrs, groups), _compact(words, hdrs, groups)
    assert all(np.array_equal(a, b) for a, b in zip(want[:3], got[:3])) and want[3] == got[3]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(SETS))
def test_both_formats_match_oracle(name):
    import torch
    from paper_1802_06058_amd import vgc
    groups, g, s, (words, hdrs) = _step(SETS[name])
    plan, scratch = _selected(groups, g, s)
    status, gh = plan.new_status(), plan.new_headers()
    out = torch.full((words.size + 64,), -1, dtype=torch.int32, device="cuda")
    vgc.pack(plan, scratch, out[:words.size], gh, status)
    assert vgc.read_status(status) == (words.size, 0) and vgc.read_headers(gh) == hdrs
    got = out.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:words.size], words) and np.all(got[words.size:] == 0xFFFFFFFF)

    stream, tile_bytes, run_offsets, chdrs = _compact(words, hdrs, groups)
    cs = torch.full((stream.size + 64,), 0xEE, dtype=torch.uint8, device="cuda")
    tb = torch.full((plan.n_tiles,), -1, dtype=torch.int16, device="cuda")
    ro = torch.full((plan.n_runs,), -1, dtype=torch.int64, device="cuda")
    for _ in range(2):                                         # a second call finds the records as the first one left them
        vgc.pack_compact(plan, scratch, cs[:stream.size], tb, ro, gh, status)
    assert vgc.read_status(status) == (stream.size, 0) and vgc.read_headers(gh) == chdrs
    assert np.array_equal(tb.cpu().numpy().view(np.uint16), tile_bytes)
    assert np.array_equal(ro.cpu().numpy().view(np.uint64), run_offsets)
    got = cs.cpu().numpy()
    assert np.array_equal(got[:stream.size], stream) and np.all(got[stream.size:] == 0xEE)


@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [[2048 * T + 1], [700] * 513 + [5 * T]], ids=["2049-tiles", "514-groups"])
def test_capacity_overflow_is_reported_not_written(sizes):
    import torch
    from paper_1802_06058_amd import vgc
    groups, g, s, (words, hdrs) = _step(sizes)
    plan, scratch = _selected(groups, g, s)
    status, gh = plan.new_status(), plan.new_headers()
    stream, _, _, chdrs = _compact(words, hdrs, groups)
    tb = torch.empty(plan.n_tiles, dtype=torch.int16, device="cuda")
    ro = torch.empty(plan.n_runs, dtype=torch.int64, device="cuda")
    for cap in (0, words.size // 2 + 1, words.size - 1):
        out = torch.full((words.size,), -1, dtype=torch.int32, device="cuda")
        vgc.pack(plan, scratch, out[:cap], gh, status)
        assert vgc.read_status(status) == (words.size, 1) and vgc.read_headers(gh) == hdrs
        got = out.cpu().numpy().view(np.uint32)
        assert np.array_equal(got[:cap], words[:cap]) and np.all(got[cap:] == 0xFFFFFFFF)
    for cap in (0, stream.size // 2 + 1, stream.size - 1):
        cs = torch.full((stream.size,), 0xEE, dtype=torch.uint8, device="cuda")
        vgc.pack_compact(plan, scratch, cs[:cap], tb, ro, gh, status)
        assert vgc.read_status(status) == (stream.size, 1) and vgc.read_headers(gh) == chdrs
        got = cs.cpu().numpy()
        assert np.array_equal(got[:cap], stream[:cap]) and np.all(got[cap:] == 0xEE)


@pytest.mark.gpu
@pytest.mark.parametrize("of,used", [([2049 * T, T], [2048 * T, 2 * T]), ([2 * T] + [T] * 600, [T] * 600 + [2 * T])], ids=["2050-tiles", "601-groups"])
def test_plan_of_another_group_list(of, used):
    """As many groups, tiles and elements, but other sizes: nothing is computed, the message is empty, the status says why."""
    import torch
    from paper_1802_06058_amd import vgc
    groups, g, s, (words, hdrs) = _step(used)
    plan, scratch = _selected(groups, g, s)
    other = vgc.Plan(W.groups_from_sizes(of), "cuda")
    assert (other.n, other.n_groups, other.n_tiles) == (plan.n, plan.n_groups, plan.n_tiles)
    plan.plan = other.plan                                     # host list of one, device tables of the other
    status, gh = plan.new_status(), plan.new_headers().fill_(0xEE)
    out = torch.full((words.size,), -1, dtype=torch.int32, device="cuda")
    vgc.pack(plan, scratch, out, gh, status)
    with pytest.raises(vgc.VgcError, match="not built from the group list"):
        vgc.read_status(status)
    assert bool((out == -1).all()) and set(vgc.read_headers(gh)) == {(0, 0, 0)}
    tb, ro = torch.full((plan.n_tiles,), -1, dtype=torch.int16, device="cuda"), torch.full((plan.n_runs,), -1, dtype=torch.int64, device="cuda")
    status, gh = plan.new_status(), plan.new_headers().fill_(0xEE)
    vgc.pack_compact(plan, scratch, out.view(torch.uint8), tb, ro, gh, status)
    with pytest.raises(vgc.VgcError, match="not built from the group list"):
        vgc.read_status(status)
    assert bool((out == -1).all()) and set(vgc.read_headers(gh)) == {(0, 0, 0)}

    # the decoders add nothing
    hd = torch.from_numpy(np.array(hdrs, dtype=vgc.HDR_DTYPE).view(np.uint8)).cuda()
    wd = torch.from_numpy(words.view(np.int32)).cuda()
    dense, m = torch.full((plan.n,), 7.0, device="cuda"), torch.zeros(plan.n, device="cuda")
    vgc.unpack_add_batch([wd], [words.size], [hd], plan, 1.0, dense, overwrite=True)
    vgc.unpack_apply([wd], [words.size], [hd], plan, 1.0, dense, m, kind=vgc.MOMENTUM_SGD, lr=1.0, momentum=0.5)
    assert bool((dense == 7.0).all()) and bool((m == 0.0).all())
