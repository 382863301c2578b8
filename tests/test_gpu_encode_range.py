"""Encodings at the ends of the coefficient range, whose first coefficient (every
output's sum starts with it) makes the transform's values largest, over primes at
the top of every class of lazy integers, against the oracle."""
import numpy as np
import pytest

import oracle as O
import paper_2605_17222_amd as H
import workload as W
from gpu_common import gpu_params, log

pytestmark = pytest.mark.gpu

TOP = 2.0 ** 62


@pytest.mark.parametrize("log_n", [12, 13, 14, 15, 16])
def test_first_coefficient_at_the_end_of_the_range(log_n):
    import torch
    log("encoded integers, ends of the range", log_n)
    two_n = 2 << log_n
    one = lambda bits: W.ntt_primes(bits, 1, two_n)[0]
    prm = W.Params(log_n=log_n, q=(one(58), one(57), one(61), one(60), one(54)), p=(W.ntt_primes(58, 2, two_n)[1], one(46)),
                   dnum=3, log_delta=30, h=64)
    o = O.Oracle(prm)
    P = gpu_params(prm)
    K, n = len(o.pq), prm.n
    g = torch.Generator(device="cuda")
    g.manual_seed(23)
    noise = torch.view_as_complex(torch.empty((n // 2, 2), dtype=torch.float64, device="cuda").uniform_(-1.0, 1.0,
                                                                                                     generator=g))
    wsb = H.ckks_encode_workspace_size(P, 1)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    # a constant slot vector is its first coefficient alone; noise of 2^-20 of it
    # gives the others about 2^35, noise of its size coefficients up to 2^57
    for c0, amount in ((1.0, 0.0), (0.95, 0.0), (-1.0, 0.0), (0.999, 2.0 ** -20), (0.95, 1.0)):
        z = torch.full((n // 2,), c0, dtype=torch.complex128, device="cuda") + amount * noise
        out, coef = H.empty((K, n)), H.empty((n,))
        H.ckks_encode(P, [z], [0], TOP, 0, K, [out], ws, wsb, coefs=[coef])
        torch.cuda.synchronize()
        m = coef.cpu().numpy()
        assert abs(abs(int(m[0])) / TOP - abs(c0)) < 0.04 and abs(int(m[0])) <= 2 ** 62
        assert np.array_equal(H.to_host(out), o.poly_from_signed(m, range(K)))
