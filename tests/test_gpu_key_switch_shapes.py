"""Key switching against the oracle over the digit counts and digit sizes the kernels are instantiated for: one to nine digits,
one to eight primes a digit, FP64 and integer moduli, both ring sizes (limb for limb)."""
import numpy as np
import pytest

from oracle import params

pytestmark = pytest.mark.gpu


def _both(n, n_q, n_p, alpha, q0_bits, qi_bits, p_bits):
    from oracle import ckks
    from paper_2602_11470_amd import binding as B
    qs = params.scan_primes(q0_bits, n, n_q) if q0_bits == qi_bits else \
        params.scan_primes(q0_bits, n, 1) + params.scan_primes(qi_bits, n, n_q - 1)
    ps = [p for p in params.scan_primes(p_bits, n, n_p + n_q) if p not in qs][:n_p]
    gctx = B.Context(n, n_q, n_p, alpha, q0_bits, qi_bits, p_bits, 2.0 ** 40, hamming=64)
    prm = params.Params(n=n, q=qs, p=ps, alpha=alpha, scale=2.0 ** 40, hamming=64)
    assert [int(x) for x in gctx.moduli()] == prm.moduli
    return ckks.Context(prm), gctx


@pytest.mark.parametrize("n,n_q,n_p,alpha,q0_bits,qi_bits,p_bits,levels", [
    (4096, 9, 1, 1, 50, 40, 60, (8, 7, 5, 3, 2, 1, 0)),      # nine digits (more than a lane keeps) down to one
    (4096, 7, 4, 4, 50, 50, 60, (6, 3)),                     # four sources, a digit of three at the top
    (4096, 9, 8, 8, 50, 50, 60, (8, 4)),                     # eight sources
    (4096, 4, 2, 2, 58, 54, 60, (3, 1)),                     # no FP64 modulus: 128-bit sums in the conversion
    (4096, 4, 2, 2, 50, 40, 61, (3, 2)),                     # 61-bit special primes
    (4096, 9, 3, 7, 50, 50, 60, (8, 6)),                     # more sources in a raise than in a ModDown
    (4096, 5, 6, 2, 50, 49, 60, (4,)),                       # and fewer
    (4096, 5, 2, 2, 58, 49, 60, (4, 2, 1)),                  # a digit of one integer and one FP64 modulus
    (4096, 4, 2, 2, 40, 49, 60, (3, 1)),                     # a last modulus far above the first: reduced before it is transformed
    (65536, 3, 1, 1, 50, 50, 60, (2,)),
    (65536, 4, 2, 2, 50, 49, 60, (3, 2)),
    (65536, 9, 8, 8, 50, 50, 60, (8,)),
    (65536, 3, 2, 2, 55, 52, 60, (2,)),
    (65536, 8, 7, 7, 50, 49, 60, (7, 6)),                    # seven sources
    (65536, 4, 7, 2, 50, 49, 50, (3,)),                      # seven FP64 special primes, digits of two
    (65536, 6, 2, 5, 50, 49, 60, (5,)),
])
def test_key_switches_match_the_oracle(n, n_q, n_p, alpha, q0_bits, qi_bits, p_bits, levels):
    octx, gctx = _both(n, n_q, n_p, alpha, q0_bits, qi_bits, p_bits)
    try:
        osk, gsk = octx.keygen_secret(3), gctx.keygen_secret(3)
        steps = [1, -3] + [5 + i for i in range(9)]              # more than one chunk of the fan-out kernel
        okeys, gkeys = octx.keygen_rotations(osk, steps, 4, with_relin=True), gctx.keygen_rotations(gsk, steps, 4, with_relin=True)
        z = np.random.default_rng(6).uniform(-1, 1, octx.S)
        coeffs = octx.encode_coeffs(z, 2.0 ** 30)

        def same(o, g):
            assert np.array_equal(gctx.ct_export(g), octx.canonical(o))

        for level in levels:
            o = octx.encrypt(osk, octx.pt_from_coeffs(coeffs, level, 2.0 ** 30), 5)
            g = gctx.encrypt(gsk, gctx.pt_from_coeffs(coeffs, level, 2.0 ** 30), 5)
            same(octx.rotate(o, 1, okeys), gctx.rotate(gkeys, g, 1))
            h = octx.hoist(o)
            for st, got in zip(steps, gctx.rotate_hoisted(gkeys, g, steps)):
                same(octx.rotate_hoisted(o, h, st, okeys), got)
            if level < 1:
                continue
            o3, g3 = octx.mul_ct(o, o), gctx.mul_ct(g, g)
            same(octx.rescale(o3), gctx.rescale(g3))             # three components: rescaled without the fused tail
            orl, grl = octx.relinearize(o3, okeys), gctx.relinearize(gkeys, g3)
            same(orl, grl)
            same(octx.rescale(orl), gctx.rescale(grl))
    finally:
        gctx.close()


def test_masked_sums_of_32_copies_against_float64():
    """q K^T through the FP64 transform of length 32 (radix 8 x 4) with every key ciphertext there, the last one partly filled,
    and half of the rows written: scores against float64 (limbs are compared with the oracle's at 20 of 32 ciphertexts, where the
    shared-dim rotations are tested)."""
    from oracle import packing
    from paper_2602_11470_amd import binding as B, inputs
    gctx = B.config1()
    try:
        H, E, lv = 8, 32, gctx.L - 1
        lay = packing.KvLayout(gctx.S, H, E)
        nk = 32
        ntok = nk * lay.t - 3
        q, K, _, _ = inputs.attention_inputs(23, H, 2, E, ntok)
        q = q * 0.3
        sk = gctx.keygen_secret(1)
        enc = lambda v, seed: gctx.level_drop(gctx.encrypt(sk, gctx.encode(v, gctx.L), seed), lv)
        want = np.einsum("he,nhe->hn", q, K)
        for shared in (32, 16):                              # nk * shared >= 16 E: the transform
            kv = gctx.kv_create(H, E, lv, unrolled_ladders=True, shared_dims=shared)
            keys = gctx.keygen_rotations(sk, kv.steps(), 2, with_relin=True)
            for c in range(nk):
                kv.load(B.CM_QK, c, enc(lay.pack_k(K, c), 100 + c))
            kv.set_tokens(ntok)
            got = gctx.decrypt(sk, gctx.vmm_kv(keys, kv, B.CM_QK, enc(lay.pack_vec(q), 10))).real
            assert np.abs(lay.unpack_scores(got, ntok) - want).max() < 1e-4
    finally:
        gctx.close()
