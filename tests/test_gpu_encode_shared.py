"""Encoding calls whose buffers share bytes in the ways that items of 32 a launch,
one launch after the other, allow: one output for every item of a caller that
wants only the integers, integers in the output itself, outputs and integers
shared by items 32 apart, integers in a later item's output.  Every result equals
a call of its own."""
import pytest

import paper_2605_17222_amd as H
import workload as W
from gpu_common import gpu_params, log

pytestmark = pytest.mark.gpu


def _encode(P, slots, rots, outs, limbs, coefs=None):
    import torch
    wsb = H.ckks_encode_workspace_size(P, len(slots))
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    H.ckks_encode(P, slots, rots, 2.0 ** 30, 0, limbs, outs, ws, wsb, coefs=coefs)
    torch.cuda.synchronize()


@pytest.mark.parametrize("log_n", [12, 13, 14])
def test_buffers_that_share_bytes(log_n):
    import torch
    log("encode, shared buffers", log_n)
    prm = W.params_toy() if log_n == 12 else W.params_paper_set("A") if log_n == 13 else W.params_n16(log_n)
    P, n, limbs, count = gpu_params(prm), prm.n, 3, 70
    g = torch.Generator(device="cuda")
    g.manual_seed(31)
    z = list(torch.view_as_complex(torch.empty((count, n // 2, 2), dtype=torch.float64, device="cuda").uniform_(
        -1.0, 1.0, generator=g)))
    rots = [-3 * i % 40 for i in range(count)]
    ref, ref_m = H.empty((count, limbs, n)), H.empty((count, n))
    for i in range(count):
        _encode(P, [z[i]], [rots[i]], [ref[i]], limbs, coefs=[ref_m[i]])
    # one output, the integers wanted
    one, m = H.empty((limbs, n)), H.empty((count, n))
    _encode(P, z, rots, [one] * count, limbs, coefs=list(m))
    assert torch.equal(m, ref_m)
    # outputs that overlap by a limb within a launch: the integers again
    buf = H.empty((count + limbs, n))
    m.zero_()
    _encode(P, z, rots, [buf[i:i + limbs] for i in range(count)], limbs, coefs=list(m))
    assert torch.equal(m, ref_m)
    # the integers in the output itself, for one limb
    got = H.empty((count, 1, n))
    _encode(P, z, rots, list(got), 1, coefs=[x[0] for x in got])
    assert torch.equal(got[:, 0], ref[:, 0])
    # outputs of items 32 apart: the later one's stays
    got = H.empty((32, limbs, n))
    _encode(P, z, rots, [got[i % 32] for i in range(count)], limbs)
    for i in range(32):
        assert torch.equal(got[i], ref[max(j for j in range(i, count, 32))])
    # integers of items 32 apart
    got, m = H.empty((count, limbs, n)), H.empty((32, n))
    _encode(P, z, rots, list(got), limbs, coefs=[m[i % 32] for i in range(count)])
    assert torch.equal(got, ref)
    # the first items' integers in outputs of the next launch
    got = H.empty((count, limbs, n))
    _encode(P, z, rots, list(got), limbs, coefs=[got[i + 32, 0] if i < 32 else None for i in range(count)])
    assert torch.equal(got, ref)
