"""Rounds of blind rotations with two clients' keys, where workgroups on idle
CUs read the keys ahead (two, one or none of them): the words are those of each
program run alone."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from paper_2506_12761_amd import vlp
    with vlp.Context(0) as ctx:
        yield vlp, ctx, [ctx.load_keys(*synth.uniform_keys(seed)) for seed in (51, 52)]


def _programs(vlp, ctx, ks, rotations, seed):
    """CoV programs whose first levels hold `rotations` blind rotations together."""
    progs, keep = [], []
    while rotations:
        l = min(64, rotations)
        M = rotations // l
        shape = vlp.make_shape("cov", M, l, 0, 1)
        q, loc = (ctx.tensor(synth.uniform_ciphertexts(seed + len(progs), n, s)) for n, s in (("q", (l,)), ("loc", (M, l))))
        v = ctx.empty(M, vlp.CT_n)
        progs.append(vlp.vlp_program_create(ctx.ctx, ks, shape, q, loc, None, None, v))
        keep.append((q, loc, v))
        assert vlp.vlp_program_level_counts(ctx.ctx, progs[-1], 0)["blind_rotations"] == M * l
        rotations -= M * l
    return progs, keep


def _two_clients(vlp, ctx, keysets, rotations):
    parts = [_programs(vlp, ctx, ks, n, 61 + 10 * i) for i, (ks, n) in
             enumerate(zip(keysets, (rotations // 2, rotations - rotations // 2)))]
    return [p for progs, _ in parts for p in progs], [k for _, keep in parts for k in keep]


@pytest.mark.parametrize("per_cu,idle", [(1, 3), (1, 1), (2, 4), (2, 2), (2, 0)])  # two, one and no CUs idle
def test_merged_round_equals_each_program_alone(gpu, per_cu, idle):
    vlp, ctx, keysets = gpu
    cus = ctx.torch.cuda.get_device_properties(0).multi_processor_count
    print("two keys", per_cu * cus - idle, flush=True)
    progs, keep = _two_clients(vlp, ctx, keysets, per_cu * cus - idle)
    while vlp.vlp_step(ctx.ctx, progs):
        pass
    merged = [ctx.to_host(v).copy() for _, _, v in keep]
    for p, (_, _, v), want in zip(progs, keep, merged):
        ctx.zero(v)
        vlp.vlp_program_reset(ctx.ctx, p)
        vlp.vlp_program_run(ctx.ctx, p)
        ctx.sync()
        assert np.array_equal(ctx.to_host(v), want)
    for p in progs:
        vlp.vlp_program_destroy(ctx.ctx, p)
