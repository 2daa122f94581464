"""ModDown and rescale in one conversion against the oracle, limb for limb: the rotary embedding (two sets of special limbs in one
conversion) and a product that ends in a rotation or a ModDown, over the special-prime counts the conversion is instantiated for,
FP64 and integer moduli on either side, both ring sizes and the lowest level."""
import numpy as np
import pytest

from oracle import params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_q,n_p,alpha,q0_bits,qi_bits,p_bits,levels", [
    (4096, 4, 1, 1, 50, 40, 60, (3, 1)),
    (4096, 4, 2, 2, 58, 54, 60, (3, 1)),                 # 128-bit sums
    (4096, 4, 3, 2, 50, 49, 61, (3,)),                   # seven terms of 128-bit sums; two sets do not fit
    (4096, 4, 4, 2, 50, 49, 50, (3,)),                   # special primes below 2^50, two sets of four
    (4096, 3, 6, 2, 50, 49, 60, (2,)),                   # two sets do not fit, one set of six in one
    (4096, 3, 5, 2, 50, 49, 50, (2,)),                   # one set of five in one
    (4096, 3, 6, 2, 58, 54, 60, (2,)),                   # one set of six in one, 128-bit sums
    (65536, 3, 1, 1, 50, 50, 60, (2, 1)),
    (65536, 4, 2, 2, 50, 49, 60, (3,)),
    (65536, 3, 2, 2, 55, 52, 60, (2,)),
    (65536, 5, 4, 4, 50, 50, 60, (4,)),
    (65536, 5, 4, 4, 50, 49, 50, (4,)),
])
def test_embedding_and_product_match_the_oracle(n, n_q, n_p, alpha, q0_bits, qi_bits, p_bits, levels):
    from oracle import ckks, packing, vmm
    from paper_2602_11470_amd import binding as B
    gctx = B.Context(n, n_q, n_p, alpha, q0_bits, qi_bits, p_bits, 2.0 ** 40, hamming=64)
    try:
        mods = [int(x) for x in gctx.moduli()]
        prm = params.Params(n=n, q=mods[:n_q], p=mods[n_q:], alpha=alpha, scale=2.0 ** 40, hamming=64)
        octx = ckks.Context(prm)
        osk, gsk = octx.keygen_secret(3), gctx.keygen_secret(3)
        rng = np.random.default_rng(n + n_p)
        heads, dim, d = 16, 16, octx.S // (16 if n == 4096 else 64)          # eight diagonals
        lay = packing.KvLayout(octx.S, heads, dim)
        plan = packing.make_plan(octx.S, d, d, 8 if n == 4096 else 4)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), 2.0 ** 40)
        steps = sorted(set(vmm.unrolled_steps(plan) + plan.all_steps() + [lay.rope_step, -lay.rope_step]))
        okeys, gkeys = octx.keygen_rotations(osk, steps, 4), gctx.keygen_rotations(gsk, steps, 4)
        coeffs = rng.integers(-(1 << 40), 1 << 40, (max(3, plan.r_i * plan.r_o), n))
        for level in levels:
            ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
            gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
            oy = vmm.rope(vmm.CkksOps(octx, okeys), lay, ox, [octx.pt_from_coeffs(c, level, float(mods[level])) for c in coeffs[:3]])
            gy = gctx.rope_apply(gkeys, gctx.rope(heads, dim, level, 1, 0, coeffs=coeffs[:3]), gx)
            assert np.array_equal(gctx.ct_export(gy), octx.canonical(oy)), level
            for form in ("plain", "unrolled"):
                if n > 4096 and (form == "plain" or n_p < 4):
                    continue
                cs = coeffs[:plan.r_i * plan.r_o]
                gplan = gctx.vmm_plan(d, d, level=level, r_i=plan.r_i, coeffs=cs, unrolled_ladders=form == "unrolled")
                conv = octx.pt_from_coeffs if form == "plain" else octx.pt_from_coeffs_ext
                od = [[conv(cs[j * plan.r_o + k], level, prm.scale) for k in range(plan.r_o)] for j in range(plan.r_i)]
                if form == "plain":
                    oy = vmm.vmm_pt(vmm.CkksOps(octx, okeys), plan, ox, od)
                else:
                    oy = vmm.vmm_pt_unrolled(octx, okeys, plan, ox, od)
                assert np.array_equal(gctx.ct_export(gctx.vmm_pt(gkeys, gplan, gx)), octx.canonical(oy)), (level, form)
    finally:
        gctx.close()


@pytest.mark.parametrize("n,n_q,n_p,alpha", [(4096, 4, 2, 2), (65536, 5, 4, 4)])
def test_embedding_with_stored_key_halves_matches_the_oracle(n, n_q, n_p, alpha):
    from oracle import ckks, packing, vmm
    from paper_2602_11470_amd import binding as B
    gctx = B.Context(n, n_q, n_p, alpha, 50, 49, 60, 2.0 ** 40, hamming=64)
    try:
        gctx.set_option(B.CM_OPT_EVK_STORED_A, 1)
        mods = [int(x) for x in gctx.moduli()]
        octx = ckks.Context(params.Params(n=n, q=mods[:n_q], p=mods[n_q:], alpha=alpha, scale=2.0 ** 40, hamming=64))
        osk, gsk = octx.keygen_secret(3), gctx.keygen_secret(3)
        rng = np.random.default_rng(n)
        level, lay = n_q - 1, packing.KvLayout(octx.S, 16, 16)
        steps = [lay.rope_step, -lay.rope_step]
        okeys, gkeys = octx.keygen_rotations(osk, steps, 4), gctx.keygen_rotations(gsk, steps, 4)
        xc, coeffs = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), 2.0 ** 40), rng.integers(-(1 << 40), 1 << 40, (3, n))
        ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
        gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, 2.0 ** 40), 5)
        want = vmm.rope(vmm.CkksOps(octx, okeys), lay, ox, [octx.pt_from_coeffs(c, level, float(mods[level])) for c in coeffs])
        got = gctx.rope_apply(gkeys, gctx.rope(16, 16, level, 1, 0, coeffs=coeffs), gx)
        assert np.array_equal(gctx.ct_export(got), octx.canonical(want))
    finally:
        gctx.close()
