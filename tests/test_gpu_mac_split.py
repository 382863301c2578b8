"""The separate multiply-accumulate on small rings, where a launch splits its
accumulators over more workgroups (8, 6 and 4 do, odd counts do not): splits
with more than 8 accumulators, whose second launch holds each remaining count,
plain and packed, and plain BSGS, against the oracle."""
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
    o.keygen(61)
    delta = 2.0 ** prm.log_delta
    ct = o.encrypt(prm.max_level, W.input_vector(61, prm.slots), delta, seed=61)
    return prm, o, delta, ct


def _run(prm, delta, ct, split, pts, keys, algo):
    import torch
    P, level = gpu_params(prm), prm.max_level
    wsb = H.ckks_lt_workspace_size(P, level, split, pts, algo)
    ws = torch.empty(max(wsb, 8), dtype=torch.uint8, device="cuda")
    o0, o1 = H.empty((level, prm.n)), H.empty((level, prm.n))
    H.ckks_lt_eval(P, level, delta, H.to_device(ct[0]), H.to_device(ct[1]), split, pts, delta, keys, algo, o0, o1, ws,
                   wsb)
    torch.cuda.synchronize()
    return np.stack([H.to_host(o0), H.to_host(o1)])


@pytest.mark.parametrize("n3", [9, 10, 11, 12, 13, 14, 15, 16])
def test_th_accumulator_counts(case, n3):
    prm, o, delta, ct = case
    split = (2, 2, n3)
    log("mac split, TH", split)
    diags = W.banded_diagonals(67, prm.slots, range(4 * n3 - 1))
    pts = o.th_plaintexts(diags, *split, delta)
    keys = {r: o.rotkey(r) for r in W.th_rotations(*split)}
    ref = o.lt_th(prm.max_level, ct, split, pts, keys)
    P = gpu_params(prm)
    dpts = [None if f is None else H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    assert np.array_equal(_run(prm, delta, ct, split, dpts, dkeys, H.CKKS_LT_TH_BSGS), ref)
    ppts = [None if f is None else H.ckks_pack(P, f) for f in dpts]
    pkeys = {r: H.ckks_pack(P, k) for r, k in dkeys.items()}
    assert np.array_equal(_run(prm, delta, ct, split, ppts, pkeys, H.CKKS_LT_TH_BSGS), ref)


@pytest.mark.parametrize("n2", [4, 6, 8])
def test_bsgs_accumulator_counts(case, n2):
    prm, o, delta, ct = case
    split = (3, n2)
    log("mac split, BSGS", split)
    diags = W.banded_diagonals(71, prm.slots, range(3 * n2))
    pts = o.bsgs_plaintexts(diags, *split, delta)
    keys = {r: o.rotkey(r) for r in W.bsgs_rotations(*split)}
    ref = o.lt_bsgs(prm.max_level, ct, split, pts, keys)
    dpts = [None if f is None else H.to_device(f) for f in pts]
    dkeys = {r: H.to_device(k) for r, k in keys.items()}
    assert np.array_equal(_run(prm, delta, ct, split, dpts, dkeys, H.CKKS_LT_BSGS), ref)
