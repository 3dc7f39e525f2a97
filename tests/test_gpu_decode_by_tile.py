"""The plain decoders either side of the parameter set up to which a workgroup takes a tile (1280 tiles; a wave takes tiles
above it), with messages whose tiles hold more words than their group's mean leads to request.  Bit-exact."""
import numpy as np
import pytest

from oracle import vgc_oracle as O
from paper_1802_06058_amd import workloads as W

pytestmark = pytest.mark.gpu
T = 2048


@pytest.mark.parametrize("sizes", [[1000 * T, 280 * T], [1000 * T + 1, 280 * T]], ids=["1280-tiles", "1281-tiles"])
@pytest.mark.parametrize("rhos", [(0.0004, "tiles", 0.1), (0.2, 0.0, "tiles", 0.5, 0.3, 0.01, 0.2, 0.2, 0.1)], ids=["sparse", "dense"])
def test_decoders_at_the_rules_edge(sizes, rhos):
    import torch
    from paper_1802_06058_amd import vgc
    groups, n, rng = W.groups_from_sizes(sizes), sum(sizes), np.random.default_rng(len(rhos))
    x = rng.standard_normal(n, dtype=np.float32)
    msgs = []
    for rho in rhos:
        if rho == "tiles":                                     # whole tiles, here and there
            send = (rng.random(n // T + 1) < 0.05).repeat(T)[:n]
        else:
            send = rng.random(n, dtype=np.float32) < rho
        msgs.append(O.pack(x, send, groups)[:2])
    words = [torch.from_numpy(np.concatenate([w, w[:1]]).view(np.int32)).cuda() if w.size else torch.zeros(1, dtype=torch.int32, device="cuda") for w, _ in msgs]
    hdrs = [torch.from_numpy(np.array(h, dtype=vgc.HDR_DTYPE).view(np.uint8)).cuda() for _, h in msgs]
    plan, counts = vgc.Plan(groups, "cuda"), [w.size for w, _ in msgs]
    bits = lambda t: (t.cpu().numpy() if hasattr(t, "cpu") else t).view(np.uint32)

    for overwrite in (True, False):
        want = np.zeros(n, np.float32) if overwrite else x.copy()
        for w, h in msgs:
            O.unpack_add(w, h, groups, 0.3, want)
        dense = torch.from_numpy(x.copy()).cuda()
        vgc.unpack_add_batch(words, counts, hdrs, plan, 0.3, dense, overwrite=overwrite)
        assert np.array_equal(bits(dense), bits(want))
    hyper = dict(lr=0.01, beta1=0.9, beta2=0.999, eps=1e-8)
    ghat = np.zeros(n, np.float32)
    for w, h in msgs:
        O.unpack_add(w, h, groups, 0.3, ghat)
    param, m, v = x.copy(), (x * np.float32(0.1)), (x * x)
    want = O.adam_step(ghat, param, m, v, hyper["lr"], hyper["beta1"], hyper["beta2"], hyper["eps"], 3)
    got = [torch.from_numpy(a.copy()).cuda() for a in (param, m, v)]
    vgc.unpack_apply(words, counts, hdrs, plan, 0.3, *got, kind=vgc.ADAM, step=3, **hyper)
    for a, b in zip(got, want):
        assert np.array_equal(bits(a), bits(b))
