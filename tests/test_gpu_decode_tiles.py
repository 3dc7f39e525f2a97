"""The batched decoders with more than one tile per wave.  How many a wave takes follows from the size of the parameter set
(up to a run of 64 beyond 10^9 parameters); here it is given, so that what a wave carries from tile to tile (cursors, requests
ahead, the compact format's directory in blocks of eight tiles, the tile's place in LDS) is checked on sets small enough for
the oracle.  The checks are those of the other decoder tests, bit for bit against the oracle."""
import pytest

import test_gpu_compact as compact
import test_gpu_select_pack as plain
import test_gpu_update as update

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_1802_06058_amd import vgc
    assert torch.cuda.is_available()
    vgc.load()
    return torch.device("cuda:0")


@pytest.fixture(params=[1, 2, 16, 64])
def calls(request, monkeypatch):
    """The library's decoders with the tiles per wave given; how often each was called."""
    from paper_1802_06058_amd import vgc
    lib, seen = vgc.load(), {}
    for name in ("unpack_add_batch", "unpack_apply", "unpack_compact_add_batch"):
        public, inner = getattr(lib, "vgc_" + name), getattr(lib, "vgc_tiles_" + name)
        inner.restype, inner.argtypes = public.restype, public.argtypes + [vgc.C.c_uint32]

        def call(*args, inner=inner, name=name):
            seen[name] = seen.get(name, 0) + 1
            return inner(*args, request.param)
        monkeypatch.setattr(lib, "vgc_" + name, call)
    return seen


@pytest.mark.parametrize("rhos", [(0.05,), (0.0, 0.17, 0.01), (0.2, 1.0, 0.3, 0.6, "tiles"), ("tiles", 0.03) * 16 + (0.0,)])
def test_plain_messages(dev, calls, rhos):
    plain.test_batch_decoder_at_the_edges_of_its_requests(dev, rhos)
    assert calls == {"unpack_add_batch": 2, "unpack_apply": 1}


def test_adam(dev, calls):
    update.test_adam_steps_match_oracle(dev, 3)
    update.test_update_on_unaligned_views(dev)
    assert calls["unpack_apply"] > 1


@pytest.mark.parametrize("p,overwrite", [(1, False), (3, True), (8, False), (11, True)])
def test_compact_messages(dev, calls, p, overwrite):
    compact.test_unpack_compact_batch_equals_plain_decode_in_order(dev, p, overwrite)
    assert calls["unpack_compact_add_batch"]


@pytest.mark.parametrize("case", ["dense", "alternating", "seven_bytes", "run_end"])
def test_compact_messages_at_the_edges(dev, calls, case):
    compact.test_unpack_compact_at_the_edges_of_a_lane_and_a_round(dev, case)
    compact.test_unpack_compact_from_oracle_bytes_with_long_gaps(dev)
    if case == "run_end":
        compact.test_short_messages_beside_dense_ones(dev)
    assert calls["unpack_compact_add_batch"]


def test_other_numbers_are_refused(dev):
    from paper_1802_06058_amd import vgc
    lib = vgc.load()
    for name, n_args in (("unpack_add_batch", 12), ("unpack_apply", 14), ("unpack_compact_add_batch", 14)):
        inner = getattr(lib, "vgc_tiles_" + name)
        inner.restype, inner.argtypes = vgc.C.c_int, getattr(lib, "vgc_" + name).argtypes + [vgc.C.c_uint32]
        assert len(inner.argtypes) == n_args + 1
        zero = [0.0 if t is vgc.C.c_float else 0 if t in (vgc.C.c_uint32, vgc.C.c_uint64, vgc.C.c_int) else None for t in inner.argtypes[:-1]]
        for tiles in (3, 128):
            assert inner(*zero, tiles) == -6
