"""The extreme keys of the GPU tests (extreme_keys.py) are live: with the oracle,
the arranged steps reach the largest sums, and every key changes every output."""
import numpy as np
import pytest

import extreme_keys as X
from oracle import oracle as O

KSK = np.zeros((O.N, 8, 4, O.n + 1), np.uint32)


def _keys(bk):
    return O.Keys(np.zeros(O.n, np.uint32), np.zeros(O.N, np.uint32), bk, KSK)


def test_words_split_at_their_ends():
    lows = {X.split(int(w))[1] for a, b in X.CASES.values() for w in np.concatenate([a, b])}
    assert {-8, 7} <= lows or X.KEY_SHIFT != 4
    assert {min(lows), max(lows)} == {-(1 << (X.KEY_SHIFT - 1)), (1 << (X.KEY_SHIFT - 1)) - 1}
    assert list(O.decompose_arr(np.array([(-2 * X.MU) & 0xFFFFFFFF], np.uint32))[0]) == [-64, -64, -64]


@pytest.mark.parametrize("name", ["lows down", "lows up", "A down B up", "A up B down", "hi apart"])
def test_arranged_steps_reach_the_largest_sums(name):
    """After the two arranged steps A and B hold MU plus, per coefficient k, six
    rows of digits -64 times a constant word w: -64 * 6 * (2 k + 2 - 1024) * w.
    The low parts' sum is then +-6 * 1024 * 64 * lo at the ends."""
    got = O.blind_rotate(_keys(X.keys(name)), X.rows()[0], X.MU)
    k = np.arange(O.N, dtype=np.int64)
    for c in range(2):
        w = int(X.CASES[name][c][0])
        want = (X.MU + (-64 * 6 * (2 * k + 2 - O.N)) * w) % 2**32
        assert np.array_equal(got[c], want.astype(np.uint32)), c


@pytest.mark.parametrize("name", list(X.CASES))
def test_every_key_changes_every_output(name):
    rows = X.rows()
    keys, zero = _keys(X.keys(name)), _keys(np.zeros((O.n, 6, 2, O.N), np.uint32))
    out = [O.bootstrap_wo_ks(keys, r, X.MU) for r in rows]
    for r, o in zip(rows, out):
        assert not np.array_equal(o, O.bootstrap_wo_ks(zero, r, X.MU))
    assert len({o.tobytes() for o in out}) == len(out)
