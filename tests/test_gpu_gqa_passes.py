"""Grouped-query products whose passes read the cache together against the same passes one call after the other, limb for limb: groups
of two, four and eight (one, one and two turns), one to sixteen terms a sum, one to eight sums, calls that the rule leaves a pass at a time,
and a cache with more sums or terms than the joint form takes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _random(B, ctx, level, seed):
    ct = B.Ct(ctx, level)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    limbs = ct.buf[: 2 * (level + 1) * ctx.n].view(2, level + 1, ctx.n)
    for i, q in enumerate(ctx.moduli()[: level + 1]):
        limbs[:, i].random_(0, int(q), generator=gen)
    ct.d = B.cm_ct(ct.buf.data_ptr(), level, 2, ctx.scale)
    return ct


@pytest.mark.parametrize("group,dim,r_i,unrolled", [(2, 16, 2, True), (4, 16, 16, False), (8, 16, 4, True), (4, 8, 1, False), (2, 32, 1, True),
                                                    (4, 32, 32, True)])
def test_joint_passes_match_single_ones(group, dim, r_i, unrolled):
    from paper_2602_11470_amd import binding as B
    _check(B, B.config1(), 2, 3, group, dim, r_i, unrolled)


@pytest.mark.parametrize("lv,r_i", [(2, 2), (3, 16), (6, 4)])
def test_joint_passes_match_single_ones_on_the_large_ring(lv, r_i):
    """Three, four and seven limbs: the single passes' sums are formed in one, two and three launches."""
    from paper_2602_11470_amd import binding as B
    _check(B, B.llama_ring(8, 4), 32, lv, 2, 16, r_i, True)


@pytest.mark.parametrize("heads,group,dim,r_i,lv", [(8, 2, 64, 16, 4), (32, 4, 16, 16, 4), (32, 4, 8, 2, 7), (32, 4, 16, 4, 2)])
def test_joint_passes_on_the_large_ring(heads, group, dim, r_i, lv):
    """Where the large ring takes the joint form: two passes over four sums of sixteen terms; four passes, one sum and four sums."""
    from paper_2602_11470_amd import binding as B
    _check(B, B.llama_ring(9, 4), heads, lv, group, dim, r_i, True)


@pytest.mark.parametrize("group,dim,r_i", [(2, 16, 8), (2, 64, 16), (2, 8, 8), (4, 8, 8), (4, 64, 8)])
def test_joint_passes_of_a_small_launch(group, dim, r_i):
    from paper_2602_11470_amd import binding as B
    _check(B, B.config1(), 2, 3, group, dim, r_i, True)


def _check(B, ctx, heads, lv, group, dim, r_i, unrolled):
    try:
        kv = ctx.kv_create(heads, dim, lv, r_i=r_i, unrolled_ladders=unrolled, key_index=True)
        t = ctx.S // (heads * dim)
        run = t // group
        for k in range(dim):
            kv.load(B.CM_SV, k, _random(B, ctx, lv, 100 + k))
            kv.load(B.CM_KV_INDEX, k, _random(B, ctx, lv, 300 + k))
        kv.set_tokens(t)
        gqa = ctx.gqa(kv, group)
        keys = ctx.keygen_rotations(ctx.keygen_secret(1), sorted(set(kv.steps()) | set(gqa.steps())), 2, with_relin=True)
        q = _random(B, ctx, lv + 1, 7)
        rep = q
        for i in range(run.bit_length() - 1):
            rep = ctx.add(rep, ctx.rotate(keys, rep, -(1 << i)))
        got = ctx.gqa_qk(keys, gqa, q)
        for d in range(group):
            x = ctx.level_drop(rep, lv) if d == 0 else ctx.rope_apply(keys, ctx.inner_rot(t, d * run, lv + 1), rep)
            assert np.array_equal(ctx.ct_export(got[d]), ctx.ct_export(ctx.vmm_kv(keys, kv, B.CM_QK_GROUP, x))), d
        scores = [_random(B, ctx, lv, 20 + d) for d in range(group)]
        acc = None
        for d in range(group):
            y = ctx.vmm_kv(keys, kv, B.CM_SV_GROUP, scores[d])
            y = ctx.level_drop(y, lv - 2) if d == 0 else ctx.rope_apply(keys, ctx.inner_rot(t, (group - d) * run, lv - 1), y)
            y.d.scale = ctx.scale
            acc = y if acc is None else ctx.add(acc, y)
        for i in range(run.bit_length() - 1):
            acc = ctx.add(acc, ctx.rotate(keys, acc, 1 << i))
        assert np.array_equal(ctx.ct_export(ctx.gqa_sv(keys, gqa, scores)), ctx.ct_export(acc))
    finally:
        ctx.close()
