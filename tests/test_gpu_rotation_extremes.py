"""Every blind-rotation kernel with keys and digits at the edges of the exactness
argument (extreme_keys.py; test_rotation_extremes.py shows that they get there),
word for word against the oracle (tolerance: none)."""
import functools
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import extreme_keys as X
from oracle import oracle as O

pytestmark = pytest.mark.gpu

KSK = np.zeros((O.N, 8, 4, O.n + 1), np.uint32)


@functools.lru_cache(maxsize=1)
def _expected(name):
    bk = X.keys(name)
    keys = O.Keys(np.zeros(O.n, np.uint32), np.zeros(O.N, np.uint32), bk, KSK)
    with ThreadPoolExecutor(O.default_threads()) as ex:
        return bk, list(ex.map(lambda r: O.bootstrap_wo_ks(keys, r, X.MU), X.rows()))


@pytest.mark.parametrize("waves,rpb", [(1, 4), (1, 8), (2, 2), (4, 1)])
@pytest.mark.parametrize("name", list(X.CASES))
def test_words_equal_the_oracle(name, waves, rpb):
    from paper_2506_12761_amd import vlp
    bk, want = _expected(name)
    print("extreme digits", name, waves, rpb, flush=True)
    rows = X.rows()
    with vlp.Context(0) as ctx:
        ks = ctx.load_keys(bk, KSK)
        t = vlp.vlp_get_tuning(ctx.ctx)
        vlp.vlp_set_tuning(ctx.ctx, rpb, 1, t.ks_gates_per_block, waves)
        out = ctx.empty(len(rows), O.N + 1)
        vlp.vlp_bootstrap(ctx.ctx, ks, ctx.tensor(rows), out, X.MU, len(rows))
        ctx.sync()
        got = ctx.to_host(out)
    for b in range(len(rows)):
        assert np.array_equal(got[b], want[b]), (name, b)
