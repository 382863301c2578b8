"""The predictor's memory words against the fused middle layer's launches, formed
here term by term as the library packs them (64 terms, 32 keys and 256 plaintexts
a launch, terms of a rotation next to each other)."""
import math
import os

import pytest

import paper_2605_17222_amd as H

LOG_N, LEVEL, ALPHA = 16, 24, 9
LQ, K, BETA = 25, 34, 3
KEY = 2 * BETA * K


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(H.LIB_PATH):
        from paper_2605_17222_amd import build
        build.build()


def _middle_words(n1, n2, n3):
    terms, words, first = [(j, i) for j in range(n2) for i in range(n1)], 0, True
    while terms:
        launch, keys = [], set()
        while terms and len(launch) < min(64, 256 // n3):
            j, _ = terms[0]
            if j and j not in keys:
                if len(keys) == 32:
                    break
                keys.add(j)
            launch.append(terms.pop(0))
        rotated = [i for j, i in launch if j]
        sets = len(set(rotated))
        words += len(keys) * KEY + 2 * K * (len(launch) - len(rotated))
        words += (sets + (len(rotated) - sets) / 4) * (BETA + 1) * K  # gathered again: a quarter
        words += 2 * n3 * K * (1 if first else 2)
        first = False
    return words + n1 * n2 * n3 * K


@pytest.mark.parametrize("split", [(1, 8, 4), (4, 4, 4), (1, 16, 4), (1, 33, 1), (1, 34, 1), (1, 65, 2), (4, 16, 4),
                                   (4, 32, 4), (2, 16, 8), (1, 32, 8), (1, 64, 8), (4, 32, 8), (4, 13, 1), (3, 7, 3),
                                   (16, 16, 8), (1, 100, 5), (5, 9, 7)])
def test_fused_layer_words_are_its_launches(split):
    n1, n2, n3 = split
    got = H.ckks_lt_predict(LOG_N, LEVEL, ALPHA, H.CKKS_LT_TH_BSGS, split, n1 * n2 * n3, rates=(0.0, 0.0, 1.0, 0.0))
    words = _middle_words(*split)
    if n1 > 1:
        words += BETA * K + (n1 - 1) * KEY + (n1 - 1) * 2 * K + LQ
    if n3 > 1:
        words += (n3 - 1) * (BETA * K + KEY + K) + 4 * K
    # (a last launch may read fewer digit sets than the others, and a launch that
    # ends between two rotations be taken for one that ends inside a rotation)
    assert math.isclose(got, words * 8 * 2 ** LOG_N, rel_tol=0.02)
