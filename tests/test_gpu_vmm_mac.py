"""The multiply-accumulate kernel of the packed product against the oracle, limb for limb: packed and unpacked limbs (moduli of 50,
below 60 and up to 61 bits), baby-step counts below and above a group of eight and around a staging pass of sixteen, giant-step
counts below and above what a workgroup takes at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [(50, 49, 60), (60, 58, 60), (61, 61, 61)])
@pytest.mark.parametrize("d,r_i", [(256, 1), (256, 2), (256, 4), (256, 32), (512, 8), (1024, 8), (1024, 16)])
def test_products_match_the_oracle(bits, d, r_i):
    from oracle import ckks, packing, params, vmm
    from paper_2602_11470_amd import binding as B
    n = 4096
    gctx = B.Context(n, 3, 1, 1, *bits, 2.0 ** 40, hamming=64)
    try:
        mods = [int(q) for q in gctx.moduli()]
        prm = params.Params(n=n, q=mods[:3], p=mods[3:], alpha=1, scale=2.0 ** 40, hamming=64)
        octx = ckks.Context(prm)
        plan = packing.make_plan(octx.S, d, d, r_i)
        rng = np.random.default_rng(d + r_i)
        coeffs = rng.integers(-(1 << 62), 1 << 62, (plan.r_i * plan.r_o, n))
        gplan = gctx.vmm_plan(d, d, level=2, r_i=r_i, coeffs=coeffs)
        odiags = [[octx.pt_from_coeffs(coeffs[j * plan.r_o + k], 2, prm.scale) for k in range(plan.r_o)] for j in range(plan.r_i)]
        osk, gsk = octx.keygen_secret(1), gctx.keygen_secret(1)
        okeys, gkeys = octx.keygen_rotations(osk, plan.all_steps(), 2), gctx.keygen_rotations(gsk, gplan.steps(), 2)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), prm.scale)
        ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, 2, prm.scale), 3)
        gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, 2, prm.scale), 3)
        oy, gy = vmm.vmm_pt(vmm.CkksOps(octx, okeys), plan, ox, odiags), gctx.vmm_pt(gkeys, gplan, gx)
        assert np.array_equal(gctx.ct_export(gy), octx.canonical(oy))
    finally:
        gctx.close()


@pytest.mark.parametrize("n_q,d,r_i", [(3, 256, 8), (3, 512, 16), (18, 256, 8), (18, 512, 16), (18, 512, 8)])
def test_rounds_of_a_workgroup_match_the_oracle(n_q, d, r_i):
    """Four, eight and sixteen giant steps; with 18 primes more items (18 x 64) than workgroups at once: a second, partly filled round,
    for sixteen giant steps (512 workgroups) a third."""
    from oracle import ckks, packing, params, vmm
    from paper_2602_11470_amd import binding as B
    n, level, alpha = 4096, n_q - 1, 1 if n_q < 16 else 2
    gctx = B.Context(n, n_q, alpha, alpha, 50, 49, 60, 2.0 ** 40, hamming=64)
    try:
        mods = [int(q) for q in gctx.moduli()]
        prm = params.Params(n=n, q=mods[:n_q], p=mods[n_q:], alpha=alpha, scale=2.0 ** 40, hamming=64)
        octx = ckks.Context(prm)
        plan = packing.make_plan(octx.S, d, d, r_i)
        rng = np.random.default_rng(d + r_i)
        coeffs = rng.integers(-(1 << 62), 1 << 62, (plan.r_i * plan.r_o, n))
        gplan = gctx.vmm_plan(d, d, level=level, r_i=r_i, coeffs=coeffs)
        odiags = [[octx.pt_from_coeffs(coeffs[j * plan.r_o + k], level, prm.scale) for k in range(plan.r_o)] for j in range(plan.r_i)]
        osk, gsk = octx.keygen_secret(1), gctx.keygen_secret(1)
        okeys, gkeys = octx.keygen_rotations(osk, plan.all_steps(), 2), gctx.keygen_rotations(gsk, gplan.steps(), 2)
        xc = octx.encode_coeffs(rng.uniform(-1, 1, octx.S), prm.scale)
        ox = octx.encrypt(osk, octx.pt_from_coeffs(xc, level, prm.scale), 3)
        gx = gctx.encrypt(gsk, gctx.pt_from_coeffs(xc, level, prm.scale), 3)
        oy, gy = vmm.vmm_pt(vmm.CkksOps(octx, okeys), plan, ox, odiags), gctx.vmm_pt(gkeys, gplan, gx)
        assert np.array_equal(gctx.ct_export(gy), octx.canonical(oy))
    finally:
        gctx.close()
