"""One message into a buffer of 2^27 elements: either side of the number of words from which on it is added tile by tile, a twelfth of
the elements where groups begin anywhere or the buffer does so itself, else a sixteenth.  Bit-exact: one float32 multiply and one add per word."""
import pytest

from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 1 << 27


@pytest.mark.parametrize("first,shift,part", [(5, 0, 12), (8, 1, 12), (8, 0, 16)], ids=["groups-anywhere", "buffer-anywhere", "neither"])
@pytest.mark.parametrize("below", [1, 0], ids=["below", "at"])
def test_one_message_at_the_rules_edge(first, shift, part, below):
    import torch
    from paper_1802_06058_amd import vgc
    gen = torch.Generator(device="cuda").manual_seed(first + below)
    groups = W.groups_from_sizes([first, N // 2, N // 2 - first])
    plan = vgc.Plan(groups, "cuda")
    at = torch.cat([torch.randint(0, N, (N // part - 100,), generator=gen, device="cuda"), torch.arange(N - 64, N, device="cuda")]).unique()
    starts = torch.tensor([o for o, _ in groups], device="cuda")
    group = torch.searchsorted(starts, at, right=True) - 1
    code = torch.randint(0, 16, at.shape, generator=gen, device="cuda")
    field = torch.randint(110, 125, (3,), generator=gen, device="cuda")
    words = torch.zeros(N // part, dtype=torch.int32, device="cuda")                    # n_words may be an upper bound
    words[:at.numel()] = ((at - starts[group]) | (code << 28)).to(torch.int32)
    count = torch.bincount(group, minlength=3)
    hdrs = torch.stack([(count << 32) | field, count.cumsum(0) - count], 1).view(torch.uint8).flatten()
    dense = torch.randn(N + 4, generator=gen, device="cuda")[shift:shift + N]
    value = (((field[group] - (code & 7)) << 23) | ((code >> 3) << 31)).to(torch.int32).view(torch.float32)
    want = dense.clone()
    want[at] += value * 0.3
    vgc.unpack_add(words, words.numel() - below, hdrs, plan, 0.3, dense)
    assert torch.equal(dense.view(torch.int32), want.view(torch.int32))
