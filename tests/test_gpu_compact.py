"""The compressed index format on the GPU (vgc_pack_compact, vgc_unpack_compact_add_batch) against the oracle:
stream bytes, per-tile byte counts, run offsets and headers bit for bit; decoded dense sums bit for bit equal to the
oracle's decode of the plain message, messages in order."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W
from streams import sample_stream

pytestmark = pytest.mark.gpu

F32 = np.float32
U32 = np.uint32


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_1802_06058_amd import vgc
    assert torch.cuda.is_available()
    vgc.load()
    return torch.device("cuda:0")


def _dev(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def _bits(a):
    return np.ascontiguousarray(a).view(U32)


class CompactMessage:
    def __init__(self, plan, dev, cap):
        import torch
        self.stream = torch.full((cap + 64,), 0xEE, dtype=torch.uint8, device=dev)         # 64 canary bytes
        self.cap = cap
        self.tile_bytes = torch.full((plan.n_tiles,), -1, dtype=torch.int16, device=dev)
        self.run_offsets = torch.full((plan.n_runs,), -1, dtype=torch.int64, device=dev)
        self.hdrs, self.status = plan.new_headers(), plan.new_status()


def _select(plan, g, s, alpha, dev):
    import torch
    from paper_1802_06058_amd import vgc
    n = plan.n
    r = torch.zeros(n, dtype=torch.float32, device=dev); v = torch.zeros(n, dtype=torch.float32, device=dev)
    scratch = plan.new_scratch()
    vgc.accumulate_select(_dev(g, dev), _dev(s, dev), r, v, plan, alpha, 0.999, scratch)
    return scratch


def _oracle_message(g, s, groups, alpha):
    z = np.zeros(g.size, F32)
    r_acc, _, _, send = O.accumulate_select(g, s, z, z, alpha, 0.999)
    words, hdrs, _ = O.pack(r_acc, send, groups)
    return words, hdrs


GROUP_SETS = {
    "mixed": [1000, 1, 37, 5000, 64, 2048, 4099, 3, 6144, 10],
    "runs": [2048 * 70 + 5, 3, 5000, 2048 * 130, 1],
    "one_partial": [777],
}


@pytest.mark.parametrize("name", list(GROUP_SETS))
@pytest.mark.parametrize("alpha", [0.0, 1.0, 4.0, 12.0])
def test_pack_compact_matches_oracle(dev, name, alpha):
    import torch
    from paper_1802_06058_amd import vgc
    sizes = GROUP_SETS[name]
    groups = W.groups_from_sizes(sizes)
    plan = vgc.Plan(groups, dev)
    n = plan.n
    g, s = sample_stream(71, (len(name), int(alpha)), n, 16, "student", sigma=0.01)
    if name == "runs":
        g[: 2048 * 3] = 0                                      # leading tiles without any element
    scratch = _select(plan, g, s, alpha, dev)
    words, hdrs = _oracle_message(g, s, groups, alpha)
    stream, tile_bytes, run_offsets, chdrs = O.pack_compact(words, hdrs, groups)
    msg = CompactMessage(plan, dev, 2 * n)
    vgc.pack_compact(plan, scratch, msg.stream[:msg.cap], msg.tile_bytes, msg.run_offsets, msg.hdrs, msg.status)
    # the plain encoder reads the same staged result, before or after
    plain = torch.empty(n, dtype=torch.int32, device=dev)
    ph, ps = plan.new_headers(), plan.new_status()
    vgc.pack(plan, scratch, plain, ph, ps)
    torch.cuda.synchronize()
    total, overflow = vgc.read_status(msg.status)
    assert overflow == 0 and total == stream.size
    got = msg.stream.cpu().numpy()
    assert np.array_equal(got[:total], stream)
    assert np.all(got[msg.cap:] == 0xEE)
    assert np.array_equal(msg.tile_bytes.cpu().numpy().view(np.uint16), tile_bytes)
    assert np.array_equal(msg.run_offsets.cpu().numpy().view(np.uint64), run_offsets)
    assert vgc.read_headers(msg.hdrs) == chdrs
    assert vgc.read_status(ps) == (words.size, 0) and np.array_equal(plain[:words.size].cpu().numpy().view(U32), words)
    if words.size >= plan.n_tiles:
        assert total + 2 * plan.n_tiles + 8 * plan.n_runs <= 4 * words.size


def test_pack_compact_capacity_overflow_is_reported_not_written(dev):
    from paper_1802_06058_amd import vgc
    import torch
    groups = W.groups_from_sizes([2048 * 5 + 9, 3000])
    plan = vgc.Plan(groups, dev)
    g, s = sample_stream(72, (0,), plan.n, 16, "normal", sigma=0.1)
    scratch = _select(plan, g, s, 1.0, dev)
    stream = O.pack_compact(*_oracle_message(g, s, groups, 1.0), groups)[0]
    cap = stream.size // 2
    msg = CompactMessage(plan, dev, cap)
    vgc.pack_compact(plan, scratch, msg.stream[:cap], msg.tile_bytes, msg.run_offsets, msg.hdrs, msg.status)
    torch.cuda.synchronize()
    assert vgc.read_status(msg.status) == (stream.size, 1)
    got = msg.stream.cpu().numpy()
    assert np.array_equal(got[:cap], stream[:cap]) and np.all(got[cap:] == 0xEE)


@pytest.mark.parametrize("p,overwrite", [(0, True), (1, False), (3, True), (8, False), (11, True)])
def test_unpack_compact_batch_equals_plain_decode_in_order(dev, p, overwrite):
    import torch
    from paper_1802_06058_amd import vgc
    sizes = [2048 * 70 + 5, 3, 5000, 2048 * 130, 1]
    groups = W.groups_from_sizes(sizes)
    plan = vgc.Plan(groups, dev)
    n = plan.n
    rng = np.random.default_rng(p)
    dense0 = rng.standard_normal(n).astype(F32)
    expect = np.zeros(n, F32) if overwrite else dense0.copy()
    dense = _dev(dense0, dev)
    scale = 1.0 / 3.0
    msgs, nbytes = [], []
    for w in range(p):
        g, s = sample_stream(73, (p, w), n, 16, "student", sigma=10.0 ** rng.uniform(-3, 0))
        alpha = [0.0, 1.0, 4.0, 12.0][w % 4]
        if w == 2:
            g[: 2048 * 70 + 5] = 0                             # a whole group absent from this message
        words, hdrs = _oracle_message(g, s, groups, alpha)
        O.unpack_add(words, hdrs, groups, scale, expect)
        # the GPU's own encoder makes the message (checked against the oracle's bytes above)
        scratch = _select(plan, g, s, alpha, dev)
        msg = CompactMessage(plan, dev, 2 * n)
        vgc.pack_compact(plan, scratch, msg.stream[:msg.cap], msg.tile_bytes, msg.run_offsets, msg.hdrs, msg.status)
        torch.cuda.synchronize()
        total, _ = vgc.read_status(msg.status)
        assert total == O.pack_compact(words, hdrs, groups)[0].size
        msgs.append(msg); nbytes.append(total)
    vgc.unpack_compact_add_batch([m.stream for m in msgs], nbytes, [m.tile_bytes for m in msgs], [m.run_offsets for m in msgs],
                                 [m.hdrs for m in msgs], plan, scale, dense, overwrite=overwrite)
    torch.cuda.synchronize()
    got = dense.cpu().numpy()
    assert np.array_equal(_bits(got), _bits(expect)), f"{np.flatnonzero(_bits(got) != _bits(expect))[:10]}"


def test_unpack_compact_from_oracle_bytes_with_long_gaps(dev):
    """A hand-made sparse message straight from the oracle's encoder: two-byte elements across the 64-byte rounds of
    the decoder (an element's first byte in lane 63), an element at the last position of a partial tile."""
    import torch
    from paper_1802_06058_amd import vgc
    sizes = [2048 * 2 + 100, 2048]
    groups = W.groups_from_sizes(sizes)
    plan = vgc.Plan(groups, dev)
    n = plan.n
    idx0 = np.concatenate([np.arange(0, 2048, 9), 2048 + np.arange(0, 2048, 31), [4096 + 99]])   # gaps of 8 and 30: two bytes each
    idx1 = np.array([0, 1, 2, 2047])
    mk = lambda idx, seed: ((np.random.default_rng(seed).integers(0, 16, idx.size).astype(np.uint64) << 28) | idx.astype(np.uint64)).astype(U32)
    words = np.concatenate([mk(idx0, 1), mk(idx1, 2)])
    hdrs = [(140, idx0.size, 0), (100, idx1.size, idx0.size)]
    stream, tile_bytes, run_offsets, chdrs = O.pack_compact(words, hdrs, groups)
    assert stream.size > 2 * 64 and tile_bytes[0] == 2 * 228 - 1
    expect = np.zeros(n, F32)
    O.unpack_add(words, hdrs, groups, 0.25, expect)
    dense = torch.zeros(n, dtype=torch.float32, device=dev)
    vgc.unpack_compact_add_batch([_dev(stream, dev)], [stream.size], [_dev(tile_bytes.view(np.int16), dev)],
                                 [_dev(run_offsets.view(np.int64), dev)],
                                 [_dev(np.array(chdrs, dtype=vgc.HDR_DTYPE).view(np.uint8), dev)], plan, 0.25, dense, overwrite=True)
    torch.cuda.synchronize()
    assert np.array_equal(_bits(dense.cpu().numpy()), _bits(expect))


@pytest.mark.parametrize("case", ["dense", "all_two_byte", "alternating", "one_byte", "two_bytes", "seven_bytes", "small_exponent", "run_end"])
def test_unpack_compact_at_the_edges_of_a_lane_and_a_round(dev, case):
    """A lane decodes 8 bytes, a round 512: elements cut by either, tiles of more than one round, streams shorter than a
    lane's access, exponent fields below the largest code, the tiles around the end of a run; three messages, the second
    of them shifted so that its bytes begin at other alignments.  Bit-exact against the oracle's decode."""
    import torch
    from paper_1802_06058_amd import vgc
    sizes = [2048 * 66 + 300, 700] if case == "run_end" else [3 * 2048 + 5, 2048]
    groups = W.groups_from_sizes(sizes)
    plan = vgc.Plan(groups, dev)
    rng = np.random.default_rng(len(case))
    field = 5 if case == "small_exponent" else 120
    scale = 1.0 if case == "small_exponent" else 1.0 / 3.0
    expect = np.zeros(plan.n, F32)
    streams, nb, tb, ro, hd = [], [], [], [], []
    for w in range(3):
        idx = []
        for _, size in groups:
            if case in ("dense", "small_exponent", "run_end"):
                i = np.flatnonzero(rng.random(size) < [0.9, 0.4, 0.05][w])
            elif case == "all_two_byte":
                i = np.arange(w, size, 9 + w)
            elif case == "alternating":                          # one- and two-byte elements by turns
                i = np.cumsum(np.tile([1 + w, 9 + 250 * w], size))
                i = i[i < size]
            else:                                                # one to seven bytes in all, in the first group only
                few = {"one_byte": [3], "two_bytes": [2047], "seven_bytes": [0, 1, 2, 3, 1000, 1001]}[case]
                i = np.array(few if size > 2048 else [], dtype=np.int64) + (w if case == "seven_bytes" else 0)
            idx.append(i)
        code = lambda k: (rng.integers(0, 2, k) << 3 | rng.integers(0, min(8, field), k)).astype(np.uint64)   # d < field: decodable
        words = np.concatenate([(code(i.size) << np.uint64(28) | i.astype(np.uint64)).astype(U32) for i in idx])
        counts = [i.size for i in idx]
        hdrs = [(field if c else 0, c, sum(counts[:k])) for k, c in enumerate(counts)]
        stream, tile_bytes, run_offsets, chdrs = O.pack_compact(words, hdrs, groups)
        O.unpack_add(words, hdrs, groups, scale, expect)
        shift = 5 * w                                            # the stream at an odd address, canary bytes around it
        whole = np.full(stream.size + 32, 0xFF, np.uint8)
        whole[shift:shift + stream.size] = stream
        streams.append(_dev(whole, dev)[shift:shift + stream.size]); nb.append(stream.size)
        tb.append(_dev(tile_bytes.view(np.int16), dev)); ro.append(_dev(run_offsets.view(np.int64), dev))
        hd.append(_dev(np.array(chdrs, dtype=vgc.HDR_DTYPE).view(np.uint8), dev))
    if case == "one_byte":
        assert nb[0] == 1
    if case == "seven_bytes":
        assert nb[0] == 7
    dense = torch.zeros(plan.n, dtype=torch.float32, device=dev)
    vgc.unpack_compact_add_batch(streams, nb, tb, ro, hd, plan, scale, dense, overwrite=True)
    torch.cuda.synchronize()
    got = dense.cpu().numpy()
    assert np.array_equal(_bits(got), _bits(expect)), np.flatnonzero(_bits(got) != _bits(expect))[:10]


def _compact(words, hdrs, groups, dev):
    from paper_1802_06058_amd import vgc
    stream, tile_bytes, run_offsets, chdrs = O.pack_compact(words, hdrs, groups)
    return (_dev(np.append(stream, np.zeros(32, np.uint8)), dev)[:stream.size], stream.size, _dev(tile_bytes.view(np.int16), dev),
            _dev(run_offsets.view(np.int64), dev), _dev(np.array(chdrs, dtype=vgc.HDR_DTYPE).view(np.uint8), dev))


def _message(idx, group_size, rng, field=120):
    """Words and headers of a model of one group whose elements idx are sent."""
    code = rng.integers(0, 16, idx.size).astype(U32)
    return code << U32(28) | idx.astype(U32), [(field if idx.size else 0, idx.size, 0)]


def test_short_messages_beside_dense_ones(dev):
    """A worker may send nothing, or a handful of bytes (fewer than a lane reads at once): its message is decoded right
    wherever it stands among dense ones, and so are they."""
    import torch
    from paper_1802_06058_amd import vgc
    rng = np.random.default_rng(0)
    n, scale = 2048 * 70 + 100, 0.125
    groups = W.groups_from_sizes([n])
    plan = vgc.Plan(groups, dev)
    few = {0: [], 1: [5], 7: [1, 2, 3, 4, 5, 6, 7], 9: [n - 9 + k for k in range(8)], 5: [2048 * 66 + 9, 2048 * 67, 2048 * 69 + 9]}
    dense_msgs = [_message(np.flatnonzero(rng.random(n) < rho), n, rng) for rho in (0.3, 0.9, 0.04)]
    for k, idx in few.items():
        short = _message(np.array(idx, np.int64), n, rng)
        for at in (0, 1, 3):
            msgs = dense_msgs[:at] + [short] + dense_msgs[at:]
            streams, nb, tb, ro, hd = zip(*(_compact(*m, groups, dev) for m in msgs))
            assert nb[at] == k
            dense = torch.zeros(n, dtype=torch.float32, device=dev)
            vgc.unpack_compact_add_batch(streams, nb, tb, ro, hd, plan, scale, dense, overwrite=True)
            torch.cuda.synchronize()
            expect = np.zeros(n, F32)
            for w, h in msgs:
                O.unpack_add(w, h, groups, scale, expect)
            assert np.array_equal(_bits(dense.cpu().numpy()), _bits(expect)), (k, at)
