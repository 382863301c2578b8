"""The middle key switch fused with the plaintext multiply-accumulate
(Algorithm 2, lines 8-14 in one kernel: the rotated products exist only in
registers) against the oracle's Algorithm 2 and against the unfused kernels
(more accumulators than a fused launch holds run the separate key-switch and
MAC launches), with packed keys and plaintexts as well, bit for bit,
alone and as the items of a batch sharing every key.  The splits cover one
and several fused launches (more than 16 terms), a middle step of one
((n1, 1, n3) runs as (1, n1, n3)), and more accumulators than one fused
launch holds (not fused)."""
import numpy as np
import pytest

import oracle as O
import paper_2605_17222_amd as H
import workload as W
from gpu_common import gpu_params, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    prm = W.params_toy()
    o = O.Oracle(prm)
    o.keygen(23)
    delta = 2.0 ** prm.log_delta
    level = prm.max_level
    diags = W.banded_diagonals(31, prm.slots, range(32))
    v = W.input_vector(31, prm.slots)
    ct = o.encrypt(level, v, delta, seed=37)
    return dict(prm=prm, o=o, delta=delta, level=level, diags=diags, v=v, ct=ct, keys={})


def _keys(c, split):
    for r in W.th_rotations(*split):
        if r not in c["keys"]:
            c["keys"][r] = c["o"].rotkey(r)
    return {r: c["keys"][r] for r in W.th_rotations(*split)}


def _single(c, split, dpts, dkeys, dct):
    import torch
    prm, level = c["prm"], c["level"]
    P = gpu_params(prm)
    wsb = H.ckks_lt_workspace_size(P, level, split, dpts, H.CKKS_LT_TH_BSGS)
    ws = torch.empty(max(wsb, 8), dtype=torch.uint8, device="cuda")
    o0, o1 = H.empty((level, prm.n)), H.empty((level, prm.n))
    H.ckks_lt_eval(P, level, c["delta"], dct[0], dct[1], split, dpts, c["delta"], dkeys, H.CKKS_LT_TH_BSGS,
                   o0, o1, ws, wsb)
    torch.cuda.synchronize()
    return np.stack([H.to_host(o0), H.to_host(o1)])


def _shared_pair(c, split, dpts, dkeys, dct):
    import torch
    prm, level = c["prm"], c["level"]
    P = gpu_params(prm)
    items = [H.BatchItem(level, c["delta"], dct[0], dct[1], split, dpts, c["delta"], dkeys,
                         H.empty((level, prm.n)), H.empty((level, prm.n))) for _ in range(2)]
    wsb = H.ckks_lt_batch_workspace_size(P, items, H.CKKS_LT_TH_BSGS)
    ws = torch.empty(max(wsb, 8), dtype=torch.uint8, device="cuda")
    code = H.ckks_lt_eval_batch(P, items, H.CKKS_LT_TH_BSGS, ws, wsb)
    torch.cuda.synchronize()
    assert code == H.CKKS_OK and all(it.status == H.CKKS_OK for it in items)
    return [np.stack([H.to_host(it.out0), H.to_host(it.out1)]) for it in items]


@pytest.mark.parametrize("split", [(2, 4, 4), (1, 8, 4), (2, 16, 1), (1, 32, 1), (4, 1, 8), (1, 2, 16)])
def test_fused_middle_layer_equals_oracle_and_unfused(case, split):
    log("fused middle layer", split)
    c = case
    o = c["o"]
    pts = o.th_plaintexts(c["diags"], *split, c["delta"])
    keys = _keys(c, split)
    ref = o.lt_th(c["level"], c["ct"], split, pts, keys)
    dpts = [None if f is None else H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    dct = [H.to_device(c["ct"][0]), H.to_device(c["ct"][1])]
    alone = _single(c, split, dpts, dkeys, dct)
    assert np.array_equal(alone, ref)
    P = gpu_params(c["prm"])
    pkeys = {r: H.ckks_pack(P, k) for r, k in dkeys.items()}
    ppts = [None if f is None else H.ckks_pack(P, f) for f in dpts]
    assert np.array_equal(_single(c, split, dpts, pkeys, dct), alone)
    assert np.array_equal(_single(c, split, ppts, pkeys, dct), alone)
    assert np.array_equal(_single(c, split, ppts, dkeys, dct), alone)
    pair = _shared_pair(c, split, dpts, dkeys, dct)
    assert np.array_equal(pair[0], alone) and np.array_equal(pair[1], alone)
    z = o.decrypt_slots(alone, c["delta"] * c["delta"] / c["prm"].q[c["level"]])
    assert np.abs(z - W.matvec(c["diags"], c["v"])).max() <= 5e-3


def test_fused_many_accumulators_every_limb_kind_packed():
    """A fused launch with 8 accumulators ((1, 2, 8)) over a chain holding
    all three kinds of limb: integer-path primes (50 bits), FP64-path primes
    stored at full width (42 and 44 bits) and narrow ones (35 bits, packed
    in 5 bytes).  With this many accumulators the packed kernels run the
    wide FP64-path limbs on the integer body; every layout equals the
    oracle's Algorithm 2 bit for bit."""
    log("fused, 8 accumulators, mixed limb kinds")
    two_n = 1 << 13
    p50 = W.ntt_primes(50, 3, two_n)
    prm = W.Params(log_n=12, q=(p50[0], W.ntt_primes(42, 1, two_n)[0], W.ntt_primes(35, 1, two_n)[0],
                                W.ntt_primes(44, 1, two_n)[0]),
                   p=(p50[1], p50[2]), dnum=2, log_delta=30, h=64)
    o = O.Oracle(prm)
    o.keygen(29)
    delta = 2.0 ** prm.log_delta
    level = prm.max_level
    split = (1, 2, 8)
    diags = W.banded_diagonals(41, prm.slots, range(16))
    ct = o.encrypt(level, W.input_vector(41, prm.slots), delta, seed=43)
    pts = o.th_plaintexts(diags, *split, delta)
    keys = {r: o.rotkey(r) for r in W.th_rotations(*split)}
    ref = o.lt_th(level, ct, split, pts, keys)
    c = dict(prm=prm, level=level, delta=delta)
    dpts = [None if f is None else H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    dct = [H.to_device(ct[0]), H.to_device(ct[1])]
    assert np.array_equal(_single(c, split, dpts, dkeys, dct), ref)
    P = gpu_params(prm)
    pkeys = {r: H.ckks_pack(P, k) for r, k in dkeys.items()}
    ppts = [None if f is None else H.ckks_pack(P, f) for f in dpts]
    assert np.array_equal(_single(c, split, dpts, pkeys, dct), ref)
    assert np.array_equal(_single(c, split, ppts, pkeys, dct), ref)
    assert np.array_equal(_single(c, split, ppts, dkeys, dct), ref)


@pytest.mark.parametrize("split,drop", [((1, 33, 2), 0), ((1, 34, 2), 5), ((2, 33, 2), 0), ((4, 17, 4), 0),
                                        ((4, 17, 3), 4), ((3, 12, 2), 7)])
def test_fused_launch_table_edges(case, split, drop):
    """Launches at the edges of the launch tables (32 keys, 64 terms, one more
    of either), inner steps of 1 to 4, with every diagonal and with every
    drop-th one absent, against the oracle's Algorithm 2, plain and packed."""
    log("fused launch tables", split, drop)
    c = case
    o, prm = c["o"], c["prm"]
    n = split[0] * split[1] * split[2]
    diags = {d: z for d, z in W.banded_diagonals(47, prm.slots, range(n)).items() if not drop or d % drop}
    pts = o.th_plaintexts(diags, *split, c["delta"])
    keys = _keys(c, split)
    ref = o.lt_th(c["level"], c["ct"], split, pts, keys)
    dpts = [None if f is None else H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    dct = [H.to_device(c["ct"][0]), H.to_device(c["ct"][1])]
    assert np.array_equal(_single(c, split, dpts, dkeys, dct), ref)
    P = gpu_params(prm)
    pkeys = {r: H.ckks_pack(P, k) for r, k in dkeys.items()}
    ppts = [None if f is None else H.ckks_pack(P, f) for f in dpts]
    assert np.array_equal(_single(c, split, ppts, pkeys, dct), ref)
    assert np.array_equal(_single(c, split, dpts, pkeys, dct), ref)


@pytest.mark.parametrize("split", [(6, 3, 2), (3, 4, 2), (8, 4, 3), (4, 6, 5), (2, 12, 8)])
def test_onfly_workspace_is_the_same_for_packed_keys(case, split):
    """The workspace is asked for without keys, so the fused launches of
    diagonals encoded on the fly must take the same workspace whether the keys
    are packed or not: the size asked for serves both, with equal results."""
    import torch
    log("fused, on the fly, packed keys", split)
    c = case
    prm, level = c["prm"], c["level"]
    P = gpu_params(prm)
    n = split[0] * split[1] * split[2]
    z = [torch.from_numpy(np.ascontiguousarray(d)).to("cuda")
         for d in W.banded_diagonals(53, prm.slots, range(n)).values()]
    dkeys = {r: H.to_device(k) for r, k in _keys(c, split).items()}
    pkeys = {r: H.ckks_pack(P, k) for r, k in dkeys.items()}
    dct = [H.to_device(c["ct"][0]), H.to_device(c["ct"][1])]
    wsb = H.ckks_lt_workspace_size(P, level, split, z, H.CKKS_LT_TH_BSGS, onfly=True)
    got = []
    for keys in (dkeys, pkeys):
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        o0, o1 = H.empty((level, prm.n)), H.empty((level, prm.n))
        H.ckks_lt_eval(P, level, c["delta"], dct[0], dct[1], split, z, c["delta"], keys, H.CKKS_LT_TH_BSGS, o0, o1,
                       ws, wsb, onfly=True)
        torch.cuda.synchronize()
        got.append(np.stack([H.to_host(o0), H.to_host(o1)]))
    assert np.array_equal(got[0], got[1])
    zd = c["o"].decrypt_slots(got[0], c["delta"] * c["delta"] / prm.q[level])
    ref = W.matvec(W.banded_diagonals(53, prm.slots, range(n)), c["v"])
    assert np.abs(zd - ref).max() <= 5e-3 * n / 16


@pytest.mark.parametrize("split,missing", [((4, 9, 1), (33, 34)), ((4, 9, 2), (4, 40, 68)), ((3, 7, 2), (3, 24)),
                                           ((5, 5, 1), (24,)), ((4, 33, 1), (64, 128))])
def test_fused_rotations_with_a_missing_term(case, split, missing):
    """Rotations some of whose terms have no diagonal in any block (groups of
    unequal size, split over launches), against the oracle's Algorithm 2."""
    log("fused, missing terms", split, missing)
    c = case
    o, prm = c["o"], c["prm"]
    inner = split[0] * split[1]
    gone = {m % inner for m in missing}
    diags = {d: z for d, z in W.banded_diagonals(59, prm.slots, range(inner * split[2])).items() if d % inner not in gone}
    pts = o.th_plaintexts(diags, *split, c["delta"])
    keys = _keys(c, split)
    ref = o.lt_th(c["level"], c["ct"], split, pts, keys)
    P = gpu_params(prm)
    dpts = [None if f is None else H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    dct = [H.to_device(c["ct"][0]), H.to_device(c["ct"][1])]
    assert np.array_equal(_single(c, split, dpts, dkeys, dct), ref)
    ppts = [None if f is None else H.ckks_pack(P, f) for f in dpts]
    assert np.array_equal(_single(c, split, ppts, {r: H.ckks_pack(P, k) for r, k in dkeys.items()}, dct), ref)
