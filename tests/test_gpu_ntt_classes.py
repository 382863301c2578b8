"""The transforms for every class of prime (how far values may grow within 64
bits differs below 2^58, 2^60 and 2^61; below 2^46 they run in FP64), at the
top of each class and with the residues that make values largest, for the
one-kernel transforms (N <= 2^13) and the two-pass ones, against the oracle; and
the one-kernel transform's two thread shapes against each other."""
import numpy as np
import pytest

import oracle as O
import paper_2605_17222_amd as H
import workload as W
from gpu_common import gpu_params, limbs_tensor, log, random_limbs

pytestmark = pytest.mark.gpu


def _params(log_n):
    two_n = 2 << log_n
    one = lambda bits: W.ntt_primes(bits, 1, two_n)[0]
    return W.Params(log_n=log_n, q=(one(61), one(60), one(58), one(46), one(47), one(30), one(59)),
                    p=(W.ntt_primes(61, 2, two_n)[1], one(54)), dnum=4, log_delta=30, h=64)


@pytest.mark.parametrize("log_n", [12, 13, 14, 15, 16])
def test_every_prime_class(log_n):
    log("ntt prime classes", log_n)
    prm = _params(log_n)
    o = O.Oracle(prm)
    P = gpu_params(prm)
    K, n = len(o.pq), prm.n
    top = np.repeat(np.array([[q - 1] for q in o.pq], dtype=np.uint64), n, axis=1)
    alternating = top.copy()
    alternating[:, 1::2] = 0
    halves = top.copy()
    halves[:, n // 2:] = 1
    for x in (random_limbs(3, o.pq, n), top, alternating, halves, np.zeros_like(top)):
        d = H.empty((K, n))
        H.ckks_op_ntt(P, True, 0, K, limbs_tensor(x), d)
        f = H.to_host(d)
        assert np.array_equal(f, o.ntt(x, range(K)))
        H.ckks_op_ntt(P, False, 0, K, limbs_tensor(x), d)
        assert np.array_equal(H.to_host(d), o.intt(x, range(K)))
        H.ckks_op_ntt(P, False, 0, K, limbs_tensor(f), d)
        assert np.array_equal(H.to_host(d), x)


def test_one_kernel_transform_shapes_agree():
    """At N = 2^13 a launch of more than 256 limbs runs another thread shape
    than a smaller one: 12 LTs as one batch (Decompose and ModDown launches of
    300 to 700 limbs) equal each LT alone (at most 100 limbs a launch), and the
    oracle for one."""
    import torch
    log("one-kernel transform shapes")
    prm = W.params_paper_set("A")
    o = O.Oracle(prm)
    o.keygen(5)
    delta = 2.0 ** prm.log_delta
    split, level = (2, 2, 4), prm.max_level
    keys = {r: o.rotkey(r) for r in W.th_rotations(*split)}
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    P = gpu_params(prm)
    items, alone = [], []
    for t in range(12):
        diags = W.banded_diagonals(60 + t, prm.slots, range(16))
        ct = o.encrypt(level, W.input_vector(60 + t, prm.slots), delta, seed=60 + t)
        pts = o.th_plaintexts(diags, *split, delta)
        dpts = [H.to_device(f) for f in pts]
        dct = [H.to_device(ct[0]), H.to_device(ct[1])]
        out = [H.empty((level, prm.n)) for _ in range(4)]
        wsb = H.ckks_lt_workspace_size(P, level, split, dpts, H.CKKS_LT_TH_BSGS)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        H.ckks_lt_eval(P, level, delta, dct[0], dct[1], split, dpts, delta, dkeys, H.CKKS_LT_TH_BSGS, out[0], out[1],
                       ws, wsb)
        torch.cuda.synchronize()
        alone.append(np.stack([H.to_host(out[0]), H.to_host(out[1])]))
        items.append(H.BatchItem(level, delta, dct[0], dct[1], split, dpts, delta, dkeys, out[2], out[3]))
        if t == 0:
            assert np.array_equal(alone[0], o.lt_th(level, ct, split, pts, keys))
    wsb = H.ckks_lt_batch_workspace_size(P, items, H.CKKS_LT_TH_BSGS)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    assert H.ckks_lt_eval_batch(P, items, H.CKKS_LT_TH_BSGS, ws, wsb) == H.CKKS_OK
    torch.cuda.synchronize()
    for it, ref in zip(items, alone):
        assert np.array_equal(np.stack([H.to_host(it.out0), H.to_host(it.out1)]), ref)


@pytest.mark.parametrize("log_n", [12, 13, 14, 16])
def test_encoded_integers_every_prime_class(log_n):
    """The transform of an encoding's signed integers for every class of prime:
    ordinary ones, and ones clamped at the ends of the range (+-2^62)."""
    import torch
    log("encoded integers, prime classes", log_n)
    prm = _params(log_n)
    o = O.Oracle(prm)
    P = gpu_params(prm)
    K, n = len(o.pq), prm.n
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    z = torch.view_as_complex(torch.empty((n // 2, 2), dtype=torch.float64, device="cuda").uniform_(-1.0, 1.0,
                                                                                                 generator=g))
    wsb = H.ckks_encode_workspace_size(P, 1)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for scale in (2.0 ** 30, 2.0 ** 66, 2.0 ** 200):
        out, coef = H.empty((K, n)), H.empty((n,))
        H.ckks_encode(P, [z], [3], scale, 0, K, [out], ws, wsb, coefs=[coef])
        torch.cuda.synchronize()
        m = coef.cpu().numpy()
        if scale > 2.0 ** 100:
            assert m.max() == 2 ** 62 and m.min() == -2 ** 62
        assert np.array_equal(H.to_host(out), o.poly_from_signed(m, range(K)))  # (in NTT form)
