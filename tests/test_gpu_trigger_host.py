"""llma_find_trigger from host lists: the forms its copy takes (one workgroup, many; buffers a thread keeps, buffers of one
call) around their limits, calls of several sizes in turn, and several threads at once, against the oracle.  Exact."""
import threading

import numpy as np
import pytest

from oracle import docs_from_flat, match_ngrams

pytestmark = pytest.mark.gpu


def lookup(seed, y_len, ref_len, docs):
    rng = np.random.RandomState(seed)
    y, ref = rng.randint(0, 4000, y_len).astype(np.int32), rng.randint(0, 4000, ref_len).astype(np.int32)
    if ref_len > 8 and y_len >= 3:
        at = rng.randint(0, ref_len - 4)
        ref[at:at + 3] = y[-3:]
    offs = np.concatenate([[0], np.sort(rng.randint(0, ref_len + 1, docs - 1)), [ref_len]]).astype(np.int32)
    return y, ref, offs


def check(args, n):
    import paper_2304_04487_amd as llma
    y, ref, offs = args
    assert llma.llma_find_trigger(y, ref, offs, n) == match_ngrams(y.tolist(), docs_from_flat(ref, offs), n), (len(y), len(ref), len(offs), n)


# (output tokens, reference tokens, documents).  One span (4096 positions) or two; lists of 32768 words in one workgroup, and of 32769;
# 2^18 words with result and keys, the most a thread keeps, and four more; beyond that in pieces of 131070 words: a list that ends with
# a piece, one that ends a word later, one of many pieces.  Mostly no multiple of four words.
SIZES = [(1, 1, 1), (3, 5, 2), (700, 4096, 3), (701, 4097, 3), (28600, 4090, 77), (28600, 4090, 78), (28601, 4091, 80), (300, 20001, 9),
         (250000, 12000, 5), (249980, 12100, 7), (254130, 8000, 5), (254131, 8000, 5), (131070, 131060, 9), (131070, 131061, 9),
         (262200, 100, 1), (40, 900001, 12), (5, 3, 1)]


@pytest.mark.parametrize("n", [1, 3])
def test_sizes_in_turn(n):
    for i, size in enumerate(SIZES):
        check(lookup(i, *size), n)


def test_threads():
    work = [[lookup(100 * t + i, 40 + 13 * t, 50 + 811 * t * (i + 1), 1 + t) for i in range(6)] for t in range(6)]
    errors = []

    def run(items):
        try:
            for _ in range(5):
                for args in items:
                    check(args, 2)
        except BaseException as e:                 # noqa: B036
            errors.append(e)

    threads = [threading.Thread(target=run, args=(items,)) for items in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[0]
