"""Row pass and inner product in one launch at n = 65536 against the oracle, limb for limb: one digit up to seven (and nine, which
take separate launches), integer and FP64 ciphertext limbs, a rotation (digits through the Galois map before they are raised),
a relinearisation and a product whose giant steps are summed (digits through the map afterwards); several outputs with one key in
runs of which the last is shorter, seven digits with several outputs, and a sum of more giant steps than one launch holds."""
import numpy as np
import pytest

from oracle import params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q,n_p,alpha,bits,levels", [
    (9, 1, 1, (50, 49, 60), (8, 6, 0)),
    (4, 2, 2, (61, 61, 61), (3,)),
    (4, 2, 2, (50, 49, 60), (3, 1)),
])
def test_key_switches_match_the_oracle(n_q, n_p, alpha, bits, levels):
    from oracle import ckks, packing, vmm
    from paper_2602_11470_amd import binding as B
    n = 65536
    gctx = B.Context(n, n_q, n_p, alpha, *bits, 2.0 ** 40, hamming=64)
    try:
        mods = [int(x) for x in gctx.moduli()]
        octx = ckks.Context(params.Params(n=n, q=mods[:n_q], p=mods[n_q:], alpha=alpha, scale=2.0 ** 40, hamming=64))
        osk, gsk = octx.keygen_secret(3), gctx.keygen_secret(3)
        plan = packing.make_plan(octx.S, 512, 512, 2)
        steps = sorted(set(vmm.unrolled_steps(plan) + [1, -3])) if n_q == 4 and bits[0] == 50 else [1, -3]
        okeys, gkeys = octx.keygen_rotations(osk, steps, 4, with_relin=True), gctx.keygen_rotations(gsk, steps, 4, with_relin=True)
        rng = np.random.default_rng(n_q)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), 2.0 ** 40)

        def same(o, g):
            assert np.array_equal(gctx.ct_export(g), octx.canonical(o))

        for level in levels:
            o = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
            g = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
            for st in (1, -3):
                same(octx.rotate(o, st, okeys), gctx.rotate(gkeys, g, st))
            if level:
                same(octx.relinearize(octx.mul_ct(o, o), okeys), gctx.relinearize(gkeys, gctx.mul_ct(g, g)))
        if len(steps) > 2:
            cs = rng.integers(-(1 << 40), 1 << 40, (plan.r_i * plan.r_o, n))
            level = levels[0]
            o = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
            g = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
            od = [[octx.pt_from_coeffs_ext(cs[j * plan.r_o + k], level, 2.0 ** 40) for k in range(plan.r_o)] for j in range(plan.r_i)]
            gplan = gctx.vmm_plan(512, 512, level=level, r_i=plan.r_i, coeffs=cs, unrolled_ladders=True)
            same(vmm.vmm_pt_unrolled(octx, okeys, plan, o, od), gctx.vmm_pt(gkeys, gplan, g))
    finally:
        gctx.close()


@pytest.mark.parametrize("n_q,n_p,alpha", [
    (10, 2, 2),           # level 8: five digits, eleven limbs, seven outputs in runs of four and three
    (5, 1, 1),            # level 3: four digits, five limbs, runs of two, the last of one
    (8, 1, 1),            # level 6: seven digits, more than a wave keeps draws of: every output by itself
])
def test_several_outputs_with_one_key_match_the_oracle(n_q, n_p, alpha):
    """q K^T over seven key ciphertexts: their relinearisations are one launch."""
    from oracle import ckks, packing, vmm
    from paper_2602_11470_amd import binding as B
    gctx = B.Context(65536, n_q, n_p, alpha, 50, 49, 60, 2.0 ** 40, hamming=64)
    try:
        mods = [int(x) for x in gctx.moduli()]
        octx = ckks.Context(params.Params(n=65536, q=mods[:n_q], p=mods[n_q:], alpha=alpha, scale=2.0 ** 40, hamming=64))
        H, E, nk, lv = 64, 8, 7, n_q - 2
        lay = packing.KvLayout(octx.S, H, E)
        kv = gctx.kv_create(H, E, lv, unrolled_ladders=True, shared_dims=E)
        osk, gsk = octx.keygen_secret(1), gctx.keygen_secret(1)
        steps = vmm.qk_shared_steps(lay, E)
        okeys, gkeys = octx.keygen_rotations(osk, steps, 2, with_relin=True), gctx.keygen_rotations(gsk, steps, 2, with_relin=True)
        rng = np.random.default_rng(n_q)

        def enc(seed):
            c = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), 2.0 ** 40)
            return octx.encrypt(osk, octx.pt_from_coeffs(c, lv, 2.0 ** 40), seed), gctx.encrypt(gsk, gctx.pt_from_coeffs(c, lv, 2.0 ** 40), seed)

        m0 = np.zeros(octx.S)
        m0[:H * lay.t] = 1
        base = octx.encode_coeffs(m0, float(mods[lv - 1]))
        kv.set_mask(0, base)
        idx = octx.q_idx(lv - 1)
        masks = [ckks.Pt(octx.ntt(octx.automorphism_coeff(octx.from_i64(base, idx), idx, octx.galois(-c * H * lay.t)), idx), lv - 1,
                         float(mods[lv - 1])) for c in range(E)]
        okc = []
        for c in range(nk):
            o, g = enc(100 + c)
            okc.append(o)
            kv.load(B.CM_QK, c, g)
        kv.set_tokens(nk * lay.t)
        oq, gq = enc(10)
        want = vmm.qk_scores_shared(octx, okeys, lay, oq, okc, masks, E)
        assert np.array_equal(gctx.ct_export(gctx.vmm_kv(gkeys, kv, B.CM_QK, gq)), octx.canonical(want))
    finally:
        gctx.close()


def test_more_giant_steps_than_one_launch_sums_match_the_oracle():
    """31 rotated sums of four digits and a first component each are 155 terms: a launch of 24 and one of 7."""
    from oracle import ckks, packing, vmm
    from paper_2602_11470_amd import binding as B
    gctx = B.Context(65536, 5, 1, 1, 50, 49, 60, 2.0 ** 40, hamming=64)
    try:
        mods = [int(x) for x in gctx.moduli()]
        octx = ckks.Context(params.Params(n=65536, q=mods[:5], p=mods[5:], alpha=1, scale=2.0 ** 40, hamming=64))
        plan, level = packing.make_plan(octx.S, 1024, 1024, 1), 3
        assert plan.r_o == 32
        osk, gsk = octx.keygen_secret(3), gctx.keygen_secret(3)
        steps = sorted(set(vmm.unrolled_steps(plan)))
        okeys, gkeys = octx.keygen_rotations(osk, steps, 4), gctx.keygen_rotations(gsk, steps, 4)
        rng = np.random.default_rng(31)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), 2.0 ** 40)
        cs = rng.integers(-(1 << 40), 1 << 40, (32, 65536))
        ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
        gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
        want = vmm.vmm_pt_unrolled(octx, okeys, plan, ox, [[octx.pt_from_coeffs_ext(c, level, 2.0 ** 40) for c in cs]])
        got = gctx.vmm_pt(gkeys, gctx.vmm_plan(1024, 1024, level=level, r_i=1, coeffs=cs, unrolled_ladders=True), gx)
        assert np.array_equal(gctx.ct_export(got), octx.canonical(want))
    finally:
        gctx.close()


@pytest.mark.parametrize("level", [6, 3])
def test_sums_of_integer_limbs_match_the_oracle(level):
    """Three giant steps under 61-bit primes: eight limbs fill the chip and are joined, five are not."""
    from oracle import ckks, packing, vmm
    from paper_2602_11470_amd import binding as B
    gctx = B.Context(65536, 7, 1, 1, 61, 61, 61, 2.0 ** 40, hamming=64)
    try:
        mods = [int(x) for x in gctx.moduli()]
        octx = ckks.Context(params.Params(n=65536, q=mods[:7], p=mods[7:], alpha=1, scale=2.0 ** 40, hamming=64))
        plan = packing.make_plan(octx.S, 512, 512, 2)
        osk, gsk = octx.keygen_secret(3), gctx.keygen_secret(3)
        steps = sorted(set(vmm.unrolled_steps(plan)))
        okeys, gkeys = octx.keygen_rotations(osk, steps, 4), gctx.keygen_rotations(gsk, steps, 4)
        rng = np.random.default_rng(level)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), 2.0 ** 40)
        cs = rng.integers(-(1 << 40), 1 << 40, (plan.r_i * plan.r_o, 65536))
        ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
        gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
        od = [[octx.pt_from_coeffs_ext(cs[j * plan.r_o + k], level, 2.0 ** 40) for k in range(plan.r_o)] for j in range(plan.r_i)]
        got = gctx.vmm_pt(gkeys, gctx.vmm_plan(512, 512, level=level, r_i=plan.r_i, coeffs=cs, unrolled_ladders=True), gx)
        assert np.array_equal(gctx.ct_export(got), octx.canonical(vmm.vmm_pt_unrolled(octx, okeys, plan, ox, od)))
    finally:
        gctx.close()
