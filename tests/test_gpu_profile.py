"""The work units of the kernel-family timing: every limb is counted in the one family that holds all of its passes, so that a
family's milliseconds over its units are the time of a limb."""
import pytest

pytestmark = pytest.mark.gpu

NTT_FWD, NTT_INV, BASE_CONV, MODDOWN_FINISH = 0, 1, 2, 4


@pytest.mark.parametrize("n,n_q,n_p,alpha", [(4096, 5, 2, 2), (65536, 5, 2, 2), (65536, 7, 3, 3)])
def test_units_of_a_rotation_and_a_rescale(n, n_q, n_p, alpha):
    import numpy as np
    import torch
    from paper_2602_11470_amd import binding as B
    ctx = B.Context(n, n_q, n_p, alpha, 50, 49, 60, 2.0 ** 40, hamming=64)
    try:
        sk = ctx.keygen_secret(1)
        keys = ctx.keygen_rotations(sk, [3], 2)

        def profiled(call):
            call()                                                   # the level's tables are made by a first call
            torch.cuda.synchronize()
            ctx.profile_enable(True)
            call()
            torch.cuda.synchronize()
            got = [ctx.profile_get(f) for f in range(8)]
            ctx.profile_enable(False)
            return got

        for level in (n_q - 1, n_q - 2):
            ct = ctx.encrypt(sk, ctx.encode(np.ones(4), level), 5)
            got = profiled(lambda: ctx.rotate(keys, ct, 3))
            ext = level + 1 + n_p
            raised = sum(ext - min(alpha, level + 1 - s) for s in range(0, level + 1, alpha))      # a ragged last digit converts more
            assert got[BASE_CONV][:2] == (2, raised + 2 * (level + 1))
            assert got[BASE_CONV][2] > 0
            assert got[NTT_FWD] == (0, 0, 0) and got[MODDOWN_FINISH] == (0, 0, 0)
            assert got[NTT_INV][:2] == (2, level + 1 + 2 * n_p)
            got = profiled(lambda: ctx.rescale(ct))
            assert got[NTT_FWD][:2] == (1, 2 * level) and got[NTT_FWD][2] > 0
            assert got[NTT_INV][:2] == (1, 2) and got[BASE_CONV] == (0, 0, 0)
    finally:
        ctx.close()
