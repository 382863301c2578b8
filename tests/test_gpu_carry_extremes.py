"""The fused middle layer's 128-bit sums over operands whose products carry at
every place (halves of all ones, of one bit and of none, residues at q - 1),
for integer-path primes at both ends of their sizes: accumulators of up to 64
such products and key-switch sums of two, against the oracle's Algorithm 2."""
import numpy as np
import pytest

import oracle as O
import paper_2605_17222_amd as H
import workload as W
from gpu_common import gpu_params, log

pytestmark = pytest.mark.gpu


def _extreme(g, q, n):
    hi = q >> 32
    vals = [0, 1, q - 1, q - 2, 2 ** 32 - 1, 2 ** 32, 2 ** 31, ((hi - 1) << 32) | 0xffffffff, hi << 32, (hi // 2) << 32]
    return g.choice(np.array(vals, dtype=np.uint64), n, p=[.05, .05, .3, .05, .1, .05, .05, .25, .05, .05])


@pytest.mark.parametrize("split,zero_keys", [((1, 40, 2), True), ((1, 33, 1), False), ((2, 20, 4), False)])
def test_sums_that_carry_everywhere(split, zero_keys):
    import torch
    log("carry extremes", split, zero_keys)
    two_n = 1 << 13
    p61 = W.ntt_primes(61, 2, two_n)
    one = lambda bits: W.ntt_primes(bits, 1, two_n)[0]
    prm = W.Params(log_n=12, q=(p61[0], one(60), one(54), one(47)), p=(p61[1], one(58)), dnum=2, log_delta=30, h=64)
    o = O.Oracle(prm)
    P, n, level = gpu_params(prm), prm.n, prm.max_level
    pq = [int(q) for q in o.pq]
    g = np.random.Generator(np.random.PCG64(97))
    limbs = lambda mods: np.stack([_extreme(g, q, n) for q in mods])
    # the ciphertext whose multiple by P holds the chosen words
    pinv = [pow(prm.p[0] * prm.p[1], -1, q) for q in prm.q]
    ct = np.stack([np.stack([np.array([int(x) * i % q for x in row], dtype=np.uint64)
                             for row, i, q in zip(limbs(prm.q), pinv, prm.q)]) for _ in range(2)])
    rots = W.th_rotations(*split)
    kshape = (2, 2, len(pq), n)
    keys = {r: np.zeros(kshape, dtype=np.uint64) if zero_keys else
            np.stack([np.stack([limbs(pq) for _ in range(2)]) for _ in range(2)]) for r in rots}
    pts = [limbs(pq) for _ in range(split[0] * split[1] * split[2])]
    ref = o.lt_th(level, ct, split, pts, keys)
    dpts = [H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    dct = [H.to_device(np.ascontiguousarray(c)) for c in ct]
    wsb = H.ckks_lt_workspace_size(P, level, split, dpts, H.CKKS_LT_TH_BSGS)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    o0, o1 = H.empty((level, n)), H.empty((level, n))
    delta = 2.0 ** prm.log_delta
    H.ckks_lt_eval(P, level, delta, dct[0], dct[1], split, dpts, delta, dkeys, H.CKKS_LT_TH_BSGS, o0, o1, ws, wsb)
    torch.cuda.synchronize()
    assert np.array_equal(np.stack([H.to_host(o0), H.to_host(o1)]), ref)
