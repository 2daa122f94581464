"""A cache append forms its masked products in runs as long as the cache's work area allows: every ciphertext of the cache and
of its key index equals the two-step form's, for caches that make one short run, several whole ones and a remainder."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,dim,r_i,level", [(4, 8, 8, 3), (8, 32, 4, 3), (8, 64, 1, 2), (8, 128, 1, 3), (4, 128, 128, 2)])
def test_appends_equal_the_two_step_form(heads, dim, r_i, level):
    from paper_2602_11470_amd import binding as B
    gctx = B.config1()
    try:
        rng = np.random.default_rng(dim + r_i)
        sk = gctx.keygen_secret(1)
        enc = lambda seed: gctx.encrypt(sk, gctx.encode(rng.normal(size=gctx.S), level + 1), seed)
        new = [(enc(2 * i + 5), enc(2 * i + 6)) for i in range(2)]
        caches, keys = [], None
        for two_step in (False, True):
            kv = gctx.kv_create(heads, dim, level, r_i=r_i, key_index=True)
            keys = keys or gctx.keygen_rotations(sk, kv.steps(), 2, with_relin=True)
            gctx.set_option(B.CM_OPT_TWO_STEP_MASKS, two_step)
            kv.append_group(keys, *new[0])
            kv.append(keys, *new[1])
            caches.append(kv)
        a, b = caches
        assert a.tokens() == b.tokens()
        for k in range(dim):
            assert np.array_equal(a.export(B.CM_SV, k), b.export(B.CM_SV, k)), k
            assert np.array_equal(a.export(B.CM_KV_INDEX, k), b.export(B.CM_KV_INDEX, k)), k
    finally:
        gctx.close()
