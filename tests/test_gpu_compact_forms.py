"""The compact decoder on streams that this library's encoder does not write: gaps below 8 in the two-byte form, streams cut
inside an element; and on a buffer with signalling NaNs, which only an element's own addition may change.  Bit-exact."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu
T = 2048


def _encode(idx, code, long):
    """Stream and tile_bytes of one group whose elements idx (ascending) carry `code`; `long`: two bytes whatever the gap.
    Also, per element, the stream offset behind its last byte."""
    stream, tile_bytes, behind = [], np.zeros((idx[-1] + T) // T, np.uint16), []
    prev_tile, prev = -1, -1
    for i, c, two in zip(idx.tolist(), code.tolist(), long.tolist()):
        tile, pos = divmod(i, T)
        gap = pos - (prev if tile == prev_tile else -1) - 1
        prev_tile, prev = tile, pos
        b = [0x80 | (gap & 7) << 4 | c, gap >> 3] if two or gap >= 8 else [gap << 4 | c]
        stream += b
        tile_bytes[tile] += len(b)
        behind.append(len(stream))
    return np.array(stream, np.uint8), tile_bytes, np.array(behind)


@pytest.mark.parametrize("field", [120, 8, 5])
@pytest.mark.parametrize("rho,two", [(0.6, 0.5), (0.6, 1.0), (0.05, 0.3), (0.2, 0.0)])
def test_any_form_decodes_and_nothing_else_changes(rho, two, field):
    import torch
    from paper_1802_06058_amd import vgc
    rng = np.random.default_rng([field, int(100 * rho), int(10 * two)])
    n, scale = 2 * T + 300, 0.5
    groups = W.groups_from_sizes([n])
    plan = vgc.Plan(groups, "cuda")
    send = rng.random(n) < rho
    send[-1] = True                                            # (the last tile has elements)
    idx = np.flatnonzero(send)
    code = rng.integers(0, 16, idx.size).astype(np.uint32)
    stream, tile_bytes, behind = _encode(idx, code, rng.random(idx.size) < two)
    words = code << np.uint32(28) | idx.astype(np.uint32)
    decoded = (code & 7) < field
    x = rng.standard_normal(n, dtype=np.float32)
    quiet = np.ones(n, bool)
    quiet[idx[decoded]] = False
    x.view(np.uint32)[quiet] = 0x7F800001 + rng.integers(0, 1000, quiet.sum()).astype(np.uint32)     # signalling NaNs
    dev = lambda a: torch.from_numpy(a).cuda()
    # whole, cut inside the last tile, inside the one before, and by a byte
    for cut in (0, 1, 2, 3, 4, 5, 6, 7, 8, 9, int(tile_bytes[2]) + 3, int(tile_bytes[2]) + 4, int(tile_bytes[2]) + 5):
        left = stream.size - cut
        there = behind <= left
        want = x.copy()
        O.unpack_add(words[there & decoded], [(field, int((there & decoded).sum()), 0)], groups, scale, want)
        hdrs = np.array([(field, idx.size, 0)], dtype=vgc.HDR_DTYPE).view(np.uint8)
        dense = dev(x)
        vgc.unpack_compact_add_batch([dev(stream)], [left], [dev(tile_bytes.view(np.int16))], [dev(np.zeros(1, np.int64))], [dev(hdrs)],
                                     plan, scale, dense)
        got = dense.cpu().numpy().view(np.uint32)
        wrong = np.flatnonzero(got != want.view(np.uint32))
        assert wrong.size == 0, (cut, wrong[:10], idx.size)
