"""Base conversions at their largest operands: every source word y_m = x_m (Q/q_m)^-1 is q_m - 1, so that a sum over the sources is
as large as it gets for the weights of that table.  A raise and a ModDown of such polynomials against Python integers, for each form of
the conversion: FP64 and cut weights below 2^50, 30-bit halves, 128-bit sums, one to eight sources, partial digits, and (n = 4096, one
source) the conversion that does the inverse transform of its source."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _prod(v):
    p = 1
    for x in v:
        p *= x
    return p


def _evaluate(ctx, columns, mods):
    """Evaluation form of the polynomials whose coefficients are all columns[i], under the moduli `mods`."""
    import torch
    a = np.repeat(np.array(columns, dtype=np.uint64)[:, None], ctx.n, axis=1)
    dev = torch.from_numpy(a.view(np.int64)).cuda()
    ctx.ntt(dev, mods)
    return dev


def _worst(qs):
    """Residues x_m of the source words whose y_m are all q_m - 1, and the integer their conversion stands for."""
    Q = _prod(qs)
    return [(-(Q // q)) % q for q in qs], sum((q - 1) * (Q // q) for q in qs)


CONTEXTS = [(8, 1, 1, (50, 40, 60)), (8, 1, 1, (50, 45, 50)), (5, 2, 2, (50, 49, 60)), (8, 4, 4, (50, 48, 60)), (8, 4, 4, (58, 58, 60)), (7, 3, 3, (61, 61, 61)),
            (9, 6, 6, (50, 50, 60)), (9, 7, 7, (50, 48, 50)), (10, 8, 8, (50, 50, 60)), (10, 8, 8, (54, 54, 54)), (6, 2, 2, (35, 35, 40))]


@pytest.mark.parametrize("n", [4096, 65536])
@pytest.mark.parametrize("n_q,n_p,alpha,bits", CONTEXTS)
def test_largest_words(n, n_q, n_p, alpha, bits):
    import torch
    from paper_2602_11470_amd import binding as B
    u64p = C.c_void_p
    raise_ = B.lib._Z8ks_raiseP6cm_ctxPKmiPmP12ihipStream_tmb
    raise_.argtypes = [u64p, u64p, C.c_int, u64p, C.c_void_p, C.c_ulong, C.c_bool]
    moddown = B.lib._Z12moddown_intoP6cm_ctxPmiPKmimS1_S3_P12ihipStream_tb
    moddown.argtypes = [u64p, u64p, C.c_int, u64p, C.c_int, C.c_ulong, u64p, u64p, C.c_void_p, C.c_bool]
    ctx = B.Context(n, n_q, n_p, alpha, *bits, 2.0 ** 30, hamming=64)
    try:
        mods = [int(q) for q in ctx.moduli()]
        for level in (n_q - 1, n_q // 2):
            ext, special = level + 1 + n_p, list(range(n_q, n_q + n_p))
            index = list(range(level + 1)) + special
            digits = [list(range(s, min(s + alpha, level + 1))) for s in range(0, level + 1, alpha)]
            # raise: own limbs as they are, the others the transform of sum_m y_m Q/q_m
            xs, want = [0] * (level + 1), []
            for D in digits:
                x, total = _worst([mods[i] for i in D])
                for i, v in zip(D, x):
                    xs[i] = v
                want += [x[D.index(i)] if i in D else total % mods[i] for i in index]
            d = _evaluate(ctx, xs, list(range(level + 1)))
            out = torch.zeros((len(digits) * ext, n), dtype=torch.int64, device="cuda")
            assert raise_(ctx.h, d.data_ptr(), level, out.data_ptr(), None, 0, False) == 0
            torch.cuda.synchronize()
            assert torch.equal(out, _evaluate(ctx, want, index * len(digits))), ("raise", level)
            # ModDown of (u, special limbs at their largest): (u - conv) P^-1, u the largest residue in one component and 0 in the other
            x, total = _worst([mods[i] for i in special])
            u = torch.empty((2, ext, n), dtype=torch.int64, device="cuda")
            for c, top in enumerate((1, 0)):
                u[c] = _evaluate(ctx, [(mods[i] - 1) * top for i in range(level + 1)] + x, index)
            got = torch.zeros((2, level + 1, n), dtype=torch.int64, device="cuda")
            assert moddown(ctx.h, u.data_ptr(), level, None, 0, 0, got.data_ptr(), None, None, False) == 0
            torch.cuda.synchronize()
            P = _prod(mods[i] for i in special)
            for c, top in enumerate((1, 0)):
                want = [((mods[i] - 1) * top - total) * pow(P, -1, mods[i]) % mods[i] for i in range(level + 1)]
                assert torch.equal(got[c], _evaluate(ctx, want, list(range(level + 1)))), ("ModDown", level, c)
    finally:
        ctx.close()
