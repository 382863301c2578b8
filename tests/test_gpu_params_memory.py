"""A parameter set holds the tables that its kernels read and no more."""
import pytest

import paper_2605_17222_amd as H
import workload as W
from gpu_common import log

pytestmark = pytest.mark.gpu


def _table_bytes(prm):
    """Twiddles (powers and Shoup words both ways on integer primes; on FP64 primes
    the powers of the one kernel, or of the column pass and the row pass's factors),
    the encoder's tables, the basis-conversion plans."""
    n, log_n = prm.n, prm.log_n
    row = log_n // 2
    col = log_n - row
    fp_words = 2 * n if log_n <= 13 else 2 * 2 ** col + 2 * (2 ** row + 2 * 2 ** col * row)
    words = sum(fp_words if q < 2 ** 46 else 4 * n for q in prm.q + prm.p)
    plans = len(prm.q) * (3 + -(-len(prm.q) // prm.alpha))
    return 8 * words + n // 2 * 36 + plans * 24 * 1024


def test_tables_are_what_the_kernels_read():
    import torch
    log("parameter tables")
    prm = W.params_n16()
    make = lambda: H.ckks_params_create(prm.log_n, prm.q, prm.p, prm.dnum)
    first = make()  # the library's code and its own memory are on the device
    torch.cuda.synchronize()
    sets, free = [], torch.cuda.mem_get_info()[0]
    for _ in range(4):
        sets.append(make())
    used = (free - torch.cuda.mem_get_info()[0]) / len(sets)
    # each of a set's 7 allocations rounded up to 2 MiB at most
    assert used <= _table_bytes(prm) + 7 * 2 ** 21, (used, _table_bytes(prm))
    del first, sets
