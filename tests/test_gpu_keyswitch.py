"""Key switching at the edges of its tiles (32 and 64 gates share a key that
the wavefronts split, 128 and 256 share a workgroup) and with key words at the
edges of the signed byte split, word for word against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from paper_2506_12761_amd import vlp
    bk, ksk = synth.uniform_keys(41)
    edge = np.array([0x00000000, 0x7F7F7F7F, 0x80808080, 0xFFFFFFFF, 0x7FFFFFFF, 0x80000000, 0x00000080, 0x0000FF7F],
                    np.uint32)
    ksk[512:] = edge[synth.stream(41, "edge").integers(0, len(edge), ksk[512:].shape)]
    keys = O.Keys(np.zeros(O.n, np.uint32), np.zeros(O.N, np.uint32), bk, ksk)
    with vlp.Context(0) as ctx:
        yield vlp, ctx, ctx.load_keys(bk, ksk), keys


@pytest.mark.parametrize("B", [1, 31, 32, 33, 64, 65, 128, 129, 256, 257])
def test_tile_edges(gpu, B):
    vlp, ctx, ks, keys = gpu
    rows = synth.uniform_u32(synth.stream(B, "ks"), (B, O.N + 1))
    rows[0] = 0xFFFF7FFF  # every digit 3, the largest before the rounding wraps
    rows[B - 1, : O.N // 2] = 0xFFFF8000  # rounds up past 2^32: every digit 0
    out = ctx.tensor(synth.uniform_u32(synth.stream(B, "dirty"), (B, O.n + 1)))
    vlp.vlp_keyswitch(ctx.ctx, ks, ctx.tensor(rows), out, B)
    ctx.sync()
    got = ctx.to_host(out)
    for b in range(B) if B <= 40 else sorted({0, 1, 31, 32, 63, B // 2, B - 2, B - 1}):
        assert np.array_equal(got[b], O.keyswitch(keys, rows[b])), (B, b)
