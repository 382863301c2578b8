"""Encoding calls of many items: every item equals its encoding in a call of its
own, at the edges of the launch sizes, with outputs that hold the slots (in
place, or another item's) and with the integers returned for some items."""
import numpy as np
import pytest

import paper_2605_17222_amd as H
import workload as W
from gpu_common import gpu_params, log

pytestmark = pytest.mark.gpu


def _slots(count, n, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    z = torch.empty((count, n // 2, 2), dtype=torch.float64, device="cuda").uniform_(-1.0, 1.0, generator=g)
    return torch.view_as_complex(z)


def _encode(P, slots, rots, outs, limbs, coefs=None):
    import torch
    wsb = H.ckks_encode_workspace_size(P, len(slots))
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    H.ckks_encode(P, slots, rots, 2.0 ** 30, 0, limbs, outs, ws, wsb, coefs=coefs)
    torch.cuda.synchronize()


@pytest.mark.parametrize("log_n,count", [(12, 1), (12, 64), (12, 65), (12, 130), (13, 33), (14, 65), (16, 3)])
def test_many_items_equal_single_ones(log_n, count):
    import torch
    log("encode batch", log_n, count)
    prm = W.params_toy() if log_n == 12 else W.params_paper_set("A") if log_n == 13 else W.params_n16(log_n)
    P, n = gpu_params(prm), prm.n
    limbs = min(4, prm.alpha + len(prm.q))
    z = _slots(count, n, 100 + count)
    rots = [(-7 * i) % 50 for i in range(count)]
    ref = H.empty((count, limbs, n))
    for i in range(count):
        _encode(P, [z[i]], [rots[i]], [ref[i]], limbs)
    got, coef = H.empty((count, limbs, n)), H.empty((count, n))
    _encode(P, list(z), rots, list(got), limbs)
    assert torch.equal(got, ref)
    got.zero_()
    _encode(P, list(z), rots, list(got), limbs, coefs=[coef[i] if i % 3 else None for i in range(count)])
    assert torch.equal(got, ref)
    # the slots inside an output of the same call: each item's own, then the
    # next item's (within the first 32, which share a launch)
    for shift in (0, 1):
        m = min(count, 32)
        buf = H.empty((m, limbs, n))
        zs = []
        for i in range(m):
            home = buf[(i + shift) % m, 0].view(torch.complex128)
            home.copy_(z[i])
            zs.append(home)
        _encode(P, zs, rots[:m], list(buf), limbs)
        assert torch.equal(buf, ref[:m])
