"""The blocked, packed weight plaintexts: every stored diagonal reads back as it was encoded, and the product is that of the
matrix, for baby-step counts below, at and above the eight words of a packed group and around the 32 of a staging pass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ring", ["50+40", "58+54"])
@pytest.mark.parametrize("d,r_i,form", [(64, 1, "plain"), (64, 2, "plain"), (256, 4, "raised"), (256, 8, "plain"), (256, 16, "raised"),
                                        (256, 32, "plain"), (512, 64, "raised"), (512, 128, "plain")])
def test_diagonals_and_product(ring, d, r_i, form):
    from paper_2602_11470_amd import binding as B, inputs
    gctx = B.config1() if ring == "50+40" else B.Context(4096, 4, 2, 1, 58, 54, 60, 2.0 ** 50)
    try:
        level, scale = gctx.L, gctx.scale
        x, W = inputs.vmm_inputs(3, d, d, "uniform", 0.05)
        raised = form == "raised"
        plan = gctx.vmm_plan(d, d, W=W, level=level, r_i=r_i, raised_sums=raised)
        m = plan.r_i * plan.r_o
        rng = np.random.default_rng(r_i)
        coeffs = rng.integers(-(1 << 55), 1 << 55, (m, gctx.n))
        stored = gctx.vmm_plan(d, d, level=level, r_i=r_i, coeffs=coeffs, raised_sums=raised)
        mods = [int(q) for q in gctx.moduli()]
        mods = mods[:level + 1] + (mods[gctx.L + 1:] if raised else [])
        for idx in (0, 1 % m, m // 2, m - 1):
            j, k = divmod(idx, plan.r_o)
            got = stored.diag_export(j, k)
            for l, q in enumerate(mods):
                want = np.array([int(c) % q for c in coeffs[idx][:512]], dtype=np.uint64)
                assert np.array_equal(got[l][:512], want), (idx, l)
        sk = gctx.keygen_secret(1)
        keys = gctx.keygen_rotations(sk, plan.steps(), 2)
        t = gctx.S // d
        slots = np.zeros(gctx.S)
        slots[::t] = x
        y = gctx.vmm_pt(keys, plan, gctx.encrypt(sk, gctx.encode(slots, level, scale), 3))
        assert np.abs(gctx.decrypt(sk, y).real[::t] - x @ W).max() < 1e-4
    finally:
        gctx.close()
