"""n = 4096, digits of one prime and one special prime: conversions that do the inverse transform of their source themselves against
the oracle, limb for limb, with as many targets as they take (363: three giant steps of 11 digits) and more (847: seven), sources below
2^50 and above, one digit only, and special primes of 50, 58 and 61 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q,level,bits,r_i", [
    (11, 10, (50, 50, 60), 8), (11, 10, (50, 50, 60), 4), (5, 1, (50, 40, 60), 8), (5, 4, (58, 58, 58), 8), (5, 4, (50, 45, 50), 8),
    (4, 3, (61, 61, 61), 8), (4, 3, (50, 58, 60), 16),
])
def test_products_match_the_oracle(n_q, level, bits, r_i):
    from oracle import ckks, packing, params, vmm
    from paper_2602_11470_amd import binding as B
    n, d = 4096, 256
    gctx = B.Context(n, n_q, 1, 1, *bits, 2.0 ** 40, hamming=64)
    try:
        mods = [int(q) for q in gctx.moduli()]
        prm = params.Params(n=n, q=mods[:n_q], p=mods[n_q:], alpha=1, scale=2.0 ** 40, hamming=64)
        octx = ckks.Context(prm)
        plan = packing.make_plan(octx.S, d, d, r_i)
        rng = np.random.default_rng(level + r_i)
        coeffs = rng.integers(-(1 << 62), 1 << 62, (plan.r_i * plan.r_o, n))
        gplan = gctx.vmm_plan(d, d, level=level, r_i=r_i, coeffs=coeffs, raised_sums=True, direct_giants=True)
        odiags = [[octx.pt_from_coeffs_ext(coeffs[j * plan.r_o + k], level, prm.scale) for k in range(plan.r_o)] for j in range(plan.r_i)]
        osk, gsk = octx.keygen_secret(1), gctx.keygen_secret(1)
        steps = vmm.direct_giant_steps(plan)
        okeys, gkeys = octx.keygen_rotations(osk, steps, 2), gctx.keygen_rotations(gsk, gplan.steps(), 2)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), prm.scale)
        ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, prm.scale), 3)
        gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, prm.scale), 3)
        oy, gy = vmm.vmm_pt_direct_giants(octx, okeys, plan, ox, odiags), gctx.vmm_pt(gkeys, gplan, gx)
        assert np.array_equal(gctx.ct_export(gy), octx.canonical(oy))
    finally:
        gctx.close()
