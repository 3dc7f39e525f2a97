"""One message into a buffer either side of 2^27 elements, from which on messages of a sixteenth of the elements (below it: an
eighth) are added tile by tile instead of word by word.  Bit-exact: one float32 multiply and one add per word."""
import pytest

from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 1 << 27


@pytest.mark.parametrize("n", [N - 1, N, N + 1])
@pytest.mark.parametrize("below", [1, 0], ids=["below-a-sixteenth", "a-sixteenth"])
def test_one_message_at_the_rules_edge(n, below):
    import torch
    from paper_1802_06058_amd import vgc
    gen = torch.Generator(device="cuda").manual_seed(n + below)
    sizes = [8, (1 << 24) - 4] + [1 << 24] * 7                 # (all begin at a multiple of 16 bytes)
    sizes[-1] += n - sum(sizes)
    groups = W.groups_from_sizes(sizes)
    plan = vgc.Plan(groups, "cuda")
    at = torch.cat([torch.randint(0, n, (n // 17,), generator=gen, device="cuda"), torch.arange(n - 64, n, device="cuda")]).unique()
    starts = torch.tensor([o for o, _ in groups], device="cuda")
    group = torch.searchsorted(starts, at, right=True) - 1
    code = torch.randint(0, 16, at.shape, generator=gen, device="cuda")
    field = torch.randint(110, 125, (len(groups),), generator=gen, device="cuda")
    words = torch.zeros(n // 16, dtype=torch.int32, device="cuda")                    # n_words may be an upper bound
    words[:at.numel()] = ((at - starts[group]) | (code << 28)).to(torch.int32)
    count = torch.bincount(group, minlength=len(groups))
    hdrs = torch.stack([(count << 32) | field, count.cumsum(0) - count], 1).view(torch.uint8).flatten()
    dense = torch.randn(n, generator=gen, device="cuda")
    value = (((field[group] - (code & 7)) << 23) | ((code >> 3) << 31)).to(torch.int32).view(torch.float32)
    want = dense.clone()
    want[at] += value * 0.3
    vgc.unpack_add(words, words.numel() - below, hdrs, plan, 0.3, dense)
    assert torch.equal(dense.view(torch.int32), want.view(torch.int32))
