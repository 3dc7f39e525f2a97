"""The compact decoder on messages of a few bytes a tile, which it decodes several at once: an eighth, a quarter or half of a
wave each, by the longest that a tile has.  Bit for bit against the oracle, which adds them in order; elements that no message
has keep their bits (signalling NaNs)."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W
from test_gpu_compact_forms import _encode

pytestmark = pytest.mark.gpu
T = 2048


def _tile(rng, n_bytes, room):
    """Positions and whether each takes two bytes (also where one would do), n_bytes in all."""
    while True:
        twice = int(rng.integers(0, n_bytes // 2 + 1))
        long = rng.permutation(np.arange(n_bytes - twice) < twice)
        gap = np.where(long, rng.integers(0, 13, long.size), rng.integers(0, 8, long.size))
        if rng.random() < 0.3 and long.any():
            gap[np.flatnonzero(long)[0]] += 200
        pos = np.cumsum(gap + 1) - 1
        if not pos.size or pos[-1] < room:
            return pos, long


@pytest.mark.parametrize("tiles", [1, 16])
@pytest.mark.parametrize("p,top", [(8, 64), (8, 65), (5, 128), (7, 129), (2, 256), (3, 256), (8, 257), (9, 128), (11, 20)])
def test_several_messages_a_round(p, top, tiles):
    import torch
    from paper_1802_06058_amd import vgc
    lib = vgc.load()
    inner = lib.vgc_tiles_unpack_compact_add_batch
    inner.restype, inner.argtypes = vgc.C.c_int, lib.vgc_unpack_compact_add_batch.argtypes + [vgc.C.c_uint32]
    rng = np.random.default_rng([p, top, tiles])
    nt, last = 11, 1900
    sizes = [(nt - 1) * T + last, 12 * T, 777]                 # nothing is sent of the second group
    groups, scale = W.groups_from_sizes(sizes), -0.3
    plan = vgc.Plan(groups, "cuda")
    n = plan.n
    longest = rng.integers(0, p, nt + 1)                       # the message that has `top` bytes in a tile
    x = rng.standard_normal(n, dtype=np.float32)
    touched, parts = np.zeros(n, bool), []
    dev = lambda a: torch.from_numpy(a).cuda()
    for w in range(p):
        field = (120, 8, 5, 254, 0)[w % 5] if w else 130       # (5: some codes are too small; 0: no element can be decoded)
        stream, tile_bytes, runs, hdrs, words, kept = [], [], [], [], [], []
        at = lost = 0
        for g, (off, size) in enumerate(groups):
            runs.append(at)
            first = at
            idx, long = np.zeros(0, np.int64), np.zeros(0, bool)
            tiles_g = (size + T - 1) // T
            for t in range(tiles_g if g != 1 else 0):
                b = top if longest[t if g == 0 else nt] == w else int(rng.choice([0, 1, 2, 7, 8, 9, top // 2, top - 1, top]))
                pos, two = _tile(rng, b, min(T, size - t * T))
                idx, long = np.concatenate([idx, t * T + pos]), np.concatenate([long, two])
            count = np.zeros(tiles_g, np.uint16)
            code = rng.integers(0, 16, idx.size).astype(np.uint32)
            if idx.size:
                s, c, behind = _encode(idx, code, long)
                count[:c.size] = c
                lost = int(w == p - 1 and g == 2)              # the last message is cut inside its last element, or before it
                there = (behind <= s.size - lost) & ((code & 7) < field)
                stream.append(s); at += s.size
                words.append(code[there] << np.uint32(28) | idx[there].astype(np.uint32))
                touched[off + idx[there]] = True
                kept.append((field, int(there.sum()), sum(v.size for v in words[:-1])))
            else:
                kept.append((field, 0, 0))
            tile_bytes.append(count)
            hdrs.append((field, idx.size, first))
        parts.append((np.concatenate(stream + [np.zeros(8, np.uint8)]), at - lost, np.concatenate(tile_bytes), np.array(runs, np.int64),
                      np.array(hdrs, dtype=vgc.HDR_DTYPE).view(np.uint8), np.concatenate(words), kept))
    assert all(8 <= part[1] <= 200 * plan.n_tiles for part in parts)         # (such a call, and no stream under eight bytes)
    x.view(np.uint32)[~touched] = 0x7F800001 + rng.integers(0, 1000, (~touched).sum()).astype(np.uint32)
    want = x.copy()
    for part in parts:
        O.unpack_add(part[5], part[6], groups, scale, want)
    streams, counts, runs, hdrs = [dev(q[0]) for q in parts], [dev(q[2].view(np.int16)) for q in parts], [dev(q[3]) for q in parts], [dev(q[4]) for q in parts]
    dense = dev(x)
    public = lib.vgc_unpack_compact_add_batch
    try:
        lib.vgc_unpack_compact_add_batch = lambda *args: inner(*args, tiles)
        vgc.unpack_compact_add_batch(streams, [q[1] for q in parts], counts, runs, hdrs, plan, scale, dense)
    finally:
        lib.vgc_unpack_compact_add_batch = public
    got = dense.cpu().numpy().view(np.uint32)
    wrong = np.flatnonzero(got != want.view(np.uint32))
    assert wrong.size == 0, (wrong[:10], wrong.size)
