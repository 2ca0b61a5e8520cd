"""The double-precision blind rotation at the edges of its dispatch and of its
exactness argument, word for word against the oracle (tolerance: none)."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from oracle import oracle as O
import synth

pytestmark = pytest.mark.gpu


def _oracle(keys, rows, mu=O.MU):
    with ThreadPoolExecutor(O.default_threads()) as ex:
        return list(ex.map(lambda c: O.bootstrap_wo_ks(keys, c, mu), rows))


@pytest.fixture(scope="module")
def uniform():
    from paper_2506_12761_amd import vlp
    bk, ksk = synth.uniform_keys(31)
    keys = O.Keys(np.zeros(O.n, np.uint32), np.zeros(O.N, np.uint32), bk, ksk)
    with vlp.Context(0) as ctx:
        yield vlp, ctx, ctx.load_keys(bk, ksk), keys


@pytest.mark.parametrize("per_cu,extra", [(0, 1), (1, -1), (1, 0), (1, 1), (2, 0), (2, 1), (4, 0), (4, 1), (6, 0), (6, 1), (8, 0), (8, 3)])
def test_round_boundaries(uniform, per_cu, extra):
    """Batches on both sides of every line of the automatic choice (rotations
    per CU): the last rotation, the first of each round and a sample."""
    vlp, ctx, ks, keys = uniform
    cus = ctx.torch.cuda.get_device_properties(0).multi_processor_count
    B = per_cu * cus + extra
    print("round boundary", B, flush=True)
    rows = synth.uniform_ciphertexts(B, "edge", (B,))
    out = ctx.empty(B, O.N + 1)
    vlp.vlp_bootstrap(ctx.ctx, ks, ctx.tensor(rows), out, O.MU, B)
    ctx.sync()
    got = ctx.to_host(out)
    at = sorted({0, B - 1, B // 2} | {k * cus for k in (1, 2, 4, 6, 8) if k * cus < B})
    for b, want in zip(at, _oracle(keys, [rows[b] for b in at])):
        assert np.array_equal(got[b], want), (B, b)


def _wave(f):
    """Key words +-2^31 (as far as 32 bits go) whose signs follow one frequency."""
    s = np.cos(np.pi * (2 * f + 1) * np.arange(O.N) / O.N)
    return np.where(s >= 0, 0x7FFFFFFF, 0x80000000).astype(np.uint32)


@pytest.mark.parametrize("name,words", [
    ("min", np.full(O.N, 0x80000000, np.uint32)),
    ("max", np.full(O.N, 0x7FFFFFFF, np.uint32)),
    ("low split", np.full(O.N, (20 * 107374182 - 10) % 2**32, np.uint32)),
    ("wave 0", _wave(0)),
    ("wave 301", _wave(301)),
])
@pytest.mark.parametrize("waves,rpb", [(1, 4), (2, 2), (4, 1)])
def test_extreme_keys(name, words, waves, rpb):
    """Keys of the largest magnitude, constant or concentrated in one
    frequency, where the sums and the rounding errors are largest: every
    kernel still rounds to the exact products."""
    from paper_2506_12761_amd import vlp
    bk = np.broadcast_to(words, (O.n, 6, 2, O.N)).copy()
    bk[1::2] = (0 - bk[1::2].astype(np.int64)).astype(np.uint32)  # alternate in sign from step to step
    ksk = np.zeros((O.N, 8, 4, O.n + 1), np.uint32)
    keys = O.Keys(np.zeros(O.n, np.uint32), np.zeros(O.N, np.uint32), bk, ksk)
    rows = synth.uniform_ciphertexts(77, "extreme", (5,))
    rows[1, :] = 0x80000000
    rows[2, : O.n // 2] = 0
    print("extreme key", name, waves, flush=True)
    with vlp.Context(0) as ctx:
        ks = ctx.load_keys(bk, ksk)
        t = vlp.vlp_get_tuning(ctx.ctx)
        vlp.vlp_set_tuning(ctx.ctx, rpb, 1, t.ks_gates_per_block, waves)
        out = ctx.empty(len(rows), O.N + 1)
        vlp.vlp_bootstrap(ctx.ctx, ks, ctx.tensor(rows), out, 1 << 31, len(rows))
        ctx.sync()
        got = ctx.to_host(out)
    for b, want in enumerate(_oracle(keys, list(rows), 1 << 31)):
        assert np.array_equal(got[b], want), (name, b)
