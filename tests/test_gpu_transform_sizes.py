"""Transforms of 65536-word limbs around the limb counts where another pass takes over (8 limbs of columns, 16 of forward rows,
64 of inverse rows and of rows with a ModDown tail, 256 for reads past the caches), under FP64, integer and 61-bit moduli (no
bit of a word to spare: folded after every stage): against the oracle, and a batch of hoisted rotations against one hoisted
rotation at a time."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [(50, 49, 60), (61, 51, 61)])
@pytest.mark.parametrize("limbs", [1, 8, 9, 16, 17, 64, 65, 257])
def test_limb_counts_match_the_oracle(limbs, bits):
    import torch
    from oracle import ckks, params
    from paper_2602_11470_amd import binding as B
    n = 65536
    qs = params.scan_primes(bits[0], n, 1) + params.scan_primes(bits[1], n, 1)
    ps = [p for p in params.scan_primes(bits[2], n, 2) if p not in qs][:1]
    mods = qs + ps
    gctx = B.Context(n, 2, 1, 1, *bits, 2.0 ** 30)
    try:
        assert [int(x) for x in gctx.moduli()] == mods
        octx = ckks.Context(params.Params(n=n, q=qs, p=ps, alpha=1, scale=2.0 ** 30))
        rng = np.random.default_rng(limbs)
        # rows 0 .. 2 random under each modulus, rows 3 .. 5 the largest residue throughout
        a = np.stack([rng.integers(0, q, n, dtype=np.uint64) for q in mods] + [np.full(n, q - 1, dtype=np.uint64) for q in mods])
        a[0, :64], a[2, 100:300], a[2, -1] = mods[0] - 1, mods[2] - 1, 0
        i = np.arange(n)
        brev = sum(((i >> b) & 1) << (15 - b) for b in range(16))
        want = octx.ntt(a.copy(), [0, 1, 2] * 2)[:, brev]
        rows = [(5 * k + limbs) % 6 for k in range(limbs)]
        idx = [r % 3 for r in rows]
        dev = torch.from_numpy(a[rows].view(np.int64)).cuda()
        gctx.ntt(dev, idx)
        assert np.array_equal(dev.cpu().numpy().view(np.uint64), want[rows])
        gctx.ntt(dev, idx, inverse=True)
        assert np.array_equal(dev.cpu().numpy().view(np.uint64), a[rows])
        # the largest residues as evaluation words: the inverse stages' own worst case
        ones = torch.from_numpy(a[[3 + i for i in idx]].view(np.int64)).cuda()
        gctx.ntt(ones, idx, inverse=True)
        gctx.ntt(ones, idx)
        assert np.array_equal(ones.cpu().numpy().view(np.uint64), a[[3 + i for i in idx]])
    finally:
        gctx.close()


@pytest.mark.parametrize("level", [1, 2, 3, 4, 7])
def test_eight_hoisted_rotations_equal_one_at_a_time(level):
    """2 (level + 1) limbs with a tail for one rotation, eight times as many for eight: 32 to 128; raises of 2 to 16 limbs."""
    from paper_2602_11470_amd import binding as B
    gctx = B.Context(65536, 8, 4, 4, 50, 49, 60, 2.0 ** 40, hamming=64)
    try:
        sk = gctx.keygen_secret(3)
        steps = [1, 2, 3, 5, 7, 11, -4, 100]
        keys = gctx.keygen_rotations(sk, steps, 4)
        x = np.random.default_rng(level).normal(size=gctx.S)
        ct = gctx.encrypt(sk, gctx.encode(x, level), 9)
        for st, got in zip(steps, gctx.rotate_hoisted(keys, ct, steps)):
            assert np.array_equal(gctx.ct_export(got), gctx.ct_export(gctx.rotate_hoisted(keys, ct, [st])[0])), st
            assert np.abs(gctx.decrypt(sk, got).real - np.roll(x, -st)).max() < 1e-4
    finally:
        gctx.close()
